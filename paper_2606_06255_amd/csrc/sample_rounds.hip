// RadiusFPS-G with certified multi-pick rounds (the default sampler), for a
// single cloud and for batches of clouds.
//
// A cloud is sampled by a team of G workgroups of eight wavefronts.  Rank r of
// the team owns the cloud's tiles t with (t - first tile) % G == r, and deals
// them to its wavefronts in turn (tiles of neighbouring voxels land on
// different workgroups, and there on different wavefronts, so the unpruned
// work near a new sample spreads).  Points (x, y, z, Dist_p, original index)
// and per-tile state (centre, radius, packed Dist_v key, filter row) stay in
// LDS for the whole cloud.  One exchange settles a whole round of selections:
//
//   L  lookahead: every wavefront proposes `steps` candidates of its own
//      tiles: it takes the largest tile key, notes the point and the
//      runner-up (the largest distance among its other points), applies the
//      candidate to its own tile only, in registers, and takes the largest
//      key again.  Its bound is the largest key left.  Applying a candidate
//      only lowers keys, so tiles it was not applied to keep keys that bound
//      their points from above;
//   X  exchange: a workgroup publishes its K largest candidates and a bound
//      that is at least every other key it holds;
//   M  merge: every workgroup runs the same deterministic merge.  S* is the
//      largest bound of the team: every point that was not published has its
//      key at or below it.  The candidates above S* are listed, and for each
//      the listed ones of no smaller distance that could lower it.  A
//      candidate none of those lowers keeps its distance until it is the
//      largest of all, so it is exactly one of the next selections of plain
//      FPS (the Sec. 3.1 rule; keys are unique).  One that is lowered fails:
//      its true key is at most its new distance and the other points of its
//      wavefront are bounded by its runner-up, so the bound rises to the
//      larger of the two and candidates at or below it leave;
//   A  apply: every wavefront applies the round's picks to its own tiles
//      (spherical test of 16 tiles by 16 picks at a time on the matrix cores,
//      strict update, tile-key resync), and starts its next lookahead without
//      a barrier.
//
// The largest candidate of a round always survives, so the loop terminates,
// and the output equals plain FPS bit for bit.  A candidate's order among the
// picks is its key order, which rank 0 of the team works out while the next
// exchange is in flight.
//
// What bounds a round (the bench's 1,048,576 points -> 65,536 picks, 256
// workgroups, 892 rounds of 10.8 us, 73 picks each): lookahead 1.9 us (a
// serial chain of wave maxima), exchange 3.6 us (2.4 of them are the bare
// exchange of the team's 32 KB, measured with nothing else in a round), list
// 1.0, conflicts 1.4, certification 1.3, picks 0.3, apply 1.1.  One lookahead per wavefront instead of one
// per workgroup removes the serial steps over all tiles of a workgroup (the
// largest term before: 16 steps on one list of tile keys), and the matrix
// cores take the pair tests, which were the next.  Sampling times before and
// after: 1,048,576 -> 65,536 15.5 -> 9.5 ms, 114,623 -> 28,655 Euclidean 10.1
// -> 5.6 ms, 80,000 -> 20,000 4.5 -> 2.8 ms; with a team size for every cloud,
// 32 clouds of 8k to 120k points 34.3 -> 8.9 ms.
//
// Exchange scopes: a team spread over the device stores through agent-scope
// atomics (coherent across XCDs); a team whose workgroups all sit on one XCD
// exchanges through that XCD's L2.  Both read past the L1 (sc1): every word
// carries the tag of its exchange, so a thread keeps reading its own 32-byte
// units until the words are there.
#include <type_traits>

#include "batch_teams.h"
#include "rfps_internal.h"
#include "round_layout.h"
#include "solo_cloud.h"

namespace rfps {

struct RoundArgs {
    IndexHeader *hdr;
    const float *xs, *ys, *zs;
    const uint32_t *orig, *inv;
    const uint32_t *tstart, *tcnt;
    const float *tcx, *tcy, *tcz, *trad;
    unsigned long long *board;
    unsigned long long *trace;
    int32_t *out_idx;
    float *out_d2;
    int32_t n, m, start;
    uint32_t flags;
    uint32_t lds_budget;
    // batched mode
    BatchCtl bc;
    BatchState *bstate;
    const uint32_t *tile_first;  // [batch+1]
    const int32_t *order;        // [batch] clouds by decreasing cost
    const uint32_t *cl_bb;       // [batch][6] boxes
};

// Value of lane l of v (l uniform).
__device__ __forceinline__ float lane_f32(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ uint32_t lane_u32(uint32_t v, int l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ unsigned long long lane_u64(unsigned long long v, int l)
{
    return ((unsigned long long)lane_u32((uint32_t)(v >> 32), l) << 32) | lane_u32((uint32_t)v, l);
}
__device__ __forceinline__ uint32_t uniform_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Plan of a single cloud: checks the capacity of the team of Gcap workgroups
// (R candidates) the caller's parameters stand for, then settles the shape
// the sampler runs with, in the header: G0 workgroups when the caller asked
// for a team, else by team_shape, enlarged until every share fits the
// sampler's LDS.  K0 as asked for, or 0.  One workgroup.
constexpr int kPlanBlock = 1024;
__global__ __launch_bounds__(kPlanBlock) void k_rounds_plan(IndexHeader *hdr, const uint32_t *__restrict__ tcnt,
                                                            unsigned long long *board, int m, int start,
                                                            int32_t *out_idx, float *out_d2, int Gall, int Gcap,
                                                            int G0, int K0, int R, uint32_t budget, uint32_t lds)
{
    __shared__ uint32_t s_tiles[kMaxGroups], s_pts[kMaxGroups];
    __shared__ uint32_t s_big, s_refused;
    const int tid = threadIdx.x;
    if (blockIdx.x) {
        // the slots a team of Gall workgroups may use
        const int words = 2 * Gall * kMaxSlotWords;
        for (int w = (blockIdx.x - 1) * kPlanBlock + tid; w < words; w += (gridDim.x - 1) * kPlanBlock)
            board[w] = 0ull;
        return;
    }
    if (tid == 0) {
        s_refused = 0u;
        hdr->last_m = (uint32_t)m;
        hdr->trace_n = 0;
        out_idx[0] = start;
        if (out_d2)
            out_d2[0] = INFINITY;
    }
    if (tid < kTeleFields)
        hdr->tele[tid] = 0;
    if (hdr->build_status) {
        if (tid == 0)
            hdr->sample_status = 0;
        return;
    }
    const uint32_t NT = hdr->n_tiles;
    TeamShape shape = team_shape(NT, (uint32_t)m);
    // shares of a team of G workgroups (tile t belongs to rank t % G)
    auto shares = [&](int G) {
        __syncthreads();
        if (tid < kMaxGroups)
            s_tiles[tid] = s_pts[tid] = 0u;
        if (tid == 0)
            s_big = 0u;
        __syncthreads();
        for (uint32_t t = tid; t < NT; t += kPlanBlock) {
            const uint32_t r = t % (uint32_t)G;
            atomicAdd(&s_tiles[r], 1u);
            atomicAdd(&s_pts[r], tcnt[t]);
        }
        __syncthreads();
    };
    shares(Gcap);
    if (tid < Gcap && !share_granted(s_tiles[tid], s_pts[tid], Gcap, R, budget))
        s_refused = 1u;
    __syncthreads();
    int G = G0;
    if (!G) {
        G = min(shape.G, Gall);
        for (;;) {
            shares(G);
            if (tid < G && rounds_lds_need(s_tiles[tid], s_pts[tid]) > lds)
                s_big = 1u;
            __syncthreads();
            if (!s_big || G >= Gcap)
                break;
            G = min(2 * G, Gcap);
        }
    }
    // a thread reads at most two units of an exchange unless the caller
    // asked for more candidates
    int K = K0;
    if (!K) {
        K = shape.K;
        while (K > 3 && G * (int)slot_units((uint32_t)K) > 2 * kRBlock)
            --K;
    }
    if (tid == 0) {
        hdr->sample_status = s_refused ? RFPS_ERR_CAPACITY : 0u;
        hdr->team_g = G;
        hdr->team_k = K;
        hdr->team_steps = shape.steps;
    }
}

// ---------------------------------------------------------------------------
// Exchange primitives for the scopes of a team.
// ---------------------------------------------------------------------------
enum class Scope { Agent, Xcd };

// A store to the board.  Inside an XCD it stays in that XCD's L2 (an ordinary
// store, written through the L1); reads past the L1 (sc1) find it there.  The
// bare exchange of 32 workgroups, 5 units each: 0.62 us; 1.94 with stores that
// go on to memory, as those between XCDs must.  32 clouds of 8k to 120k points
// in a batch: 9.7 -> 8.8 ms.
template <Scope S>
__device__ __forceinline__ void bstore(unsigned long long *p, unsigned long long v)
{
    if constexpr (S == Scope::Agent)
        st_agent(p, v);
    else
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Tags run through 1..65534 with the exchange counter: 0 is a cleared board,
// 65535 the abort tag, and a slot is rewritten every second exchange, so a
// stale word never carries the current tag.
constexpr uint32_t kAbortTag = 0xffffu;
__device__ __forceinline__ uint32_t tag_of(uint32_t epoch) { return epoch % 65534u + 1u; }

// A team's slots: rank r's slot of exchange e is at
// base + (e & 1) * par_words + r * slot_words.
struct Board {
    unsigned long long *base;
    uint32_t slot_words, par_words;
};

template <Scope S>
__device__ void publish_abort_tags(const Board &bd, int rank, int K)
{
    const uint32_t words = slot_units(K) * kUnit;
    for (uint32_t par = 0; par < 2; ++par)
        for (uint32_t w = 0; w < words; ++w)
            bstore<S>(bd.base + par * bd.par_words + rank * bd.slot_words + w, (unsigned long long)kAbortTag << 48);
}

// Reads one or two units (32 bytes each) past the L1, all loads in flight;
// each aligned 64-bit word is read whole.  Words come as (low, high) pairs.
__device__ __forceinline__ void load_unit(const unsigned long long *p, u32x4 &a, u32x4 &b)
{
    asm volatile("global_load_dwordx4 %0, %2, off sc1\n\t"
                 "global_load_dwordx4 %1, %2, off offset:16 sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(a), "=&v"(b)
                 : "v"(p)
                 : "memory");
}
__device__ __forceinline__ void load_unit2(const unsigned long long *p, const unsigned long long *q, u32x4 &a,
                                           u32x4 &b, u32x4 &c, u32x4 &d)
{
    asm volatile("global_load_dwordx4 %0, %4, off sc1\n\t"
                 "global_load_dwordx4 %1, %4, off offset:16 sc1\n\t"
                 "global_load_dwordx4 %2, %5, off sc1\n\t"
                 "global_load_dwordx4 %3, %5, off offset:16 sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(a), "=&v"(b), "=&v"(c), "=&v"(d)
                 : "v"(p), "v"(q)
                 : "memory");
}

// Payload of a candidate's unit: x, y, z, distance bits, ~original index and
// the runner-up's distance bits, 192 bits in four words of 48.
struct Cand {
    float x, y, z;
    uint32_t d, o, u;  // distance bits, ~original index, runner-up distance bits
};
__device__ __forceinline__ Cand unpack_cand(const u32x4 &a, const u32x4 &b)
{
    // a = words 0, 1 and b = words 2, 3 as (low, high) halves
    Cand c;
    c.x = __uint_as_float(a.x);
    c.y = __uint_as_float((a.y & 0xffffu) | (a.z << 16));
    c.z = __uint_as_float((a.z >> 16) | (a.w << 16));
    c.d = b.x;
    c.o = (b.y & 0xffffu) | (b.z << 16);
    c.u = (b.z >> 16) | (b.w << 16);
    return c;
}

// What every workgroup keeps in LDS besides its tiles and points.
struct __align__(16) RoundShared {
    u32x4 rec[kMaxRec][2];              // this workgroup's candidates of the round, packed
    float4 lq[kList];                   // listed candidates: coordinates, runner-up distance (bits)
    float4 lb[kList];                   // shifted coordinates and column term of the distance filter
    float ld[kList], lT[kList];         // distance, minus the row term of the filter
    unsigned long long lkey[kList];     // keys (0 in the padding of the last block)
    // conflict rows of the listed candidates (see conflict_pos), then, in the
    // same memory, the round's picks: coordinates, and shifted ones with the
    // column term
    union {
        unsigned long long adj[kList * kListWords];
        float4 pk[2 * kList];
    };
    unsigned long long pkey[kList];     // the picks' keys
    uint32_t prank[kList];              // and their ranks (0 between uses)
    unsigned long long rkey[kMaxRec];   // keys of rec
    // by parity of the round (cleared for the next one): the largest bound of
    // this workgroup's wavefronts, and of the whole team
    unsigned long long gb[2], sx[2];
    unsigned long long red2[kRWaves];
    unsigned long long wf[4], wo[4], wscur;  // certification of long lists: masks and bound
    uint32_t wmet[4];
    uint32_t scan[kRWaves];
    uint32_t cnt[kRWaves];              // candidates a wavefront lists, and whether one blurs the filter
    uint32_t abort, npick, cut_bin, cut_have;
    uint32_t hist[256];
};

// (and the few words the kernels add)
static_assert(sizeof(RoundShared) + 256 <= kRoundsStatic, "static LDS of the sampler");

// Bit b of word w of a conflict row stands for list position
// conflict_pos<NW>(w, b), NW words in use (64 NW positions): the layout the
// matrix cores' result registers give without any exchange between lanes.
// For more than 128 positions each quarter of a word holds qs row blocks, 3
// (up to 192 positions; 4 bits of the quarter stay unused) or 4.
template <int NW>
__device__ __forceinline__ int conflict_pos(int w, int b, int qs)
{
    if constexpr (NW == 1)
        return 16 * ((b >> 2) & 3) + 4 * (b >> 4) + (b & 3);
    else if constexpr (NW == 2)
        return 16 * ((b >> 2) & 7) + 4 * (2 * w + (b >> 5)) + (b & 3);
    else
        return ((b >> 2) & 3) < qs ? 16 * ((b >> 4) * qs + ((b >> 2) & 3)) + 4 * w + (b & 3) : kList;
}

// Per-thread telemetry accumulators.
struct RoundTele {
    unsigned long long tests = 0, pruned = 0, visited = 0, skipped = 0, updated = 0, resync = 0;
    unsigned long long ph[5] = {0, 0, 0, 0, 0};  // lookahead, exchange, merge, apply, exchange wait
    // finer clocks: merge list / conflicts / certification / picks, lookahead
    // steps after the first, exchange poll / rest, apply's point updates
    unsigned long long list = 0, conflicts = 0, walk = 0, picks = 0, later = 0, poll = 0, rest = 0, update = 0;
    unsigned long long apairs = 0, arekeys = 0;  // wavefront 0's apply: tile-pick pairs updated, tiles re-keyed
    unsigned long long above = 0, listed = 0, fails = 0;
    unsigned long long rounds = 0;
};

// What one team samples: tiles [tb, te) of the index, whose original indices
// start at point_base (subtracted from the output), m selections from the
// local start index, outputs at out_idx / out_d2 (already offset), and the
// origin the distance filter shifts to.
struct CloudJob {
    uint32_t tb, te, point_base;
    int32_t m, start;
    int32_t *out_idx;
    float *out_d2;
    float ox, oy, oz;
};

__device__ __forceinline__ float norm2(float x, float y, float z)
{
    const float xx = x * x, yy = y * y, zz = z * z;
    const float s = xx + yy;
    return s + zz;
}

// Largest key of the wave and the lowest lane that holds it (all lanes active).
__device__ __forceinline__ unsigned long long wave_max_key(unsigned long long v, int &at)
{
    const uint32_t hi = (uint32_t)(v >> 32), lo = (uint32_t)v;
    const uint32_t mhi = wave_max_u32(hi);
    unsigned long long tie = ballot64(hi == mhi);
    if (tie & (tie - 1)) {  // several lanes hold the largest high half
        const uint32_t mlo = wave_max_u32(hi == mhi ? lo : 0u);
        tie &= ballot64(lo == mlo);
    }
    at = __builtin_ctzll(tie);
    return ((unsigned long long)mhi << 32) | lane_u32(lo, at);
}

// Samples one cloud.  Every thread of every workgroup of the team calls it.
// `epoch` is the team's exchange counter: it only grows, so slots never need
// clearing between clouds.  NU: units a thread reads per exchange (the team's
// G (K + 1) units are dealt to kRBlock threads).  Returns false when an
// exchange failed (abort).
template <Scope S, int NU, bool E, bool T>
__device__ __forceinline__ bool sample_cloud(const RoundArgs &a, const CloudJob &job, const int rank, const int G, const int K,
                             const int steps, const Board &board, uint32_t &epoch, unsigned char *smem,
                             RoundShared &sh, RoundTele &tl, bool record_trace, bool clocks)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    // the wavefront index is uniform: as a scalar it keeps wave-strided loops
    // and their addressing off the exec mask
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint32_t span = job.te - job.tb;
    const int ntl = (span > (uint32_t)rank) ? (int)((span - 1 - rank) / G) + 1 : 0;
    constexpr bool euclid = E;  // Euclidean distances (RFPS_F_SQRT), a separate instantiation
    // counters, phase clocks and the exchange trace exist only in the
    // instrumented instantiation (T): the default kernels carry none of
    // their code
    const bool tele = T && (a.flags & RFPS_F_TELEMETRY) != 0;
    const bool count_skip = T && !(a.flags & RFPS_F_NO_POINT_SKIP);
    const bool trace = T && record_trace && tid == 0;
    clocks = T && clocks;
    const bool solo = G == 1;
    const int li = lane & (kBlk - 1), lg = lane / kBlk;  // column (or row) and group of a filter block's operands

    // ---- LDS layout (the plan checked that it fits) ----
    const int nws = (int)wave_slots((uint32_t)ntl);  // tile slots per wavefront
    const int nts = nws * kRWaves;
    float4 *tsph = reinterpret_cast<float4 *>(smem);                              // tile centres
    unsigned long long *tkey = reinterpret_cast<unsigned long long *>(tsph + nts);
    float *trow = reinterpret_cast<float *>(tkey + nts);  // the tile's filter: minus its row term
    float *trad = trow + nts;
    uint32_t *tmeta = reinterpret_cast<uint32_t *>(trad + nts);  // LDS offset | count << 16
    float4 *pq = reinterpret_cast<float4 *>(tmeta + nts);        // points: coordinates, ~original index (bits)

    // ---- prologue: tile metadata and LDS offsets (block prefix sum) ----
    for (int s = tid; s < nts; s += kRBlock) {
        tsph[s] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        tkey[s] = 0ull;
        trow[s] = INFINITY;  // a padding slot passes no filter
        trad[s] = 0.0f;
        tmeta[s] = 0u;
    }
    const int per = (ntl + kRBlock - 1) / kRBlock;
    const int l0 = tid * per, l1 = min(l0 + per, ntl);
    uint32_t cnt_sum = 0;
    for (int lt = l0; lt < l1; ++lt)
        cnt_sum += a.tcnt[job.tb + rank + (size_t)lt * G];
    uint32_t incl = cnt_sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        uint32_t o = __shfl_up(incl, off, kWave);
        if (lane >= off)
            incl += o;
    }
    if (lane == kWave - 1)
        sh.scan[wave] = incl;
    __syncthreads();
    uint32_t off = incl - cnt_sum, npl = 0;
    for (int q = 0; q < kRWaves; ++q) {
        off += q < wave ? sh.scan[q] : 0u;
        npl += sh.scan[q];
    }
    // tile lt belongs to wavefront lt % kRWaves: tiles of neighbouring voxels
    // go to different wavefronts as they go to different workgroups
    for (int lt = l0; lt < l1; ++lt) {
        const size_t t = job.tb + rank + (size_t)lt * G;
        const uint32_t c = a.tcnt[t];
        const int s = (lt % kRWaves) * nws + lt / kRWaves;
        tmeta[s] = off | (c << 16);
        tsph[s] = make_float4(a.tcx[t], a.tcy[t], a.tcz[t], 0.0f);
        trad[s] = a.trad[t];
        off += c;
    }
    float *pd = reinterpret_cast<float *>(pq + npl);
    // the carving must end inside the dynamic LDS the plan sized
    if (reinterpret_cast<unsigned char *>(pd + npl) - smem > (ptrdiff_t)a.lds_budget) {
        if (tid == 0) {
            set_status(&a.hdr->sample_status, RFPS_ERR_INTERNAL);
            // the rest of the team must not wait for this workgroup
            if (!solo)
                publish_abort_tags<S>(board, rank, K);
        }
        return false;
    }
    const int wb = wave * nws;  // this wavefront's tile slots: wb .. wb + ntw - 1
    const int ntw = ntl > wave ? (ntl - 1 - wave) / kRWaves + 1 : 0;

    // Key, threshold and filter row of tile slot s from each lane's distance d
    // and key low half o of its point (all lanes of the wave must call it).
    auto rekey = [&](int s, bool valid, float d, uint32_t o) {
        const float4 c = tsph[s];
        const float r = trad[s];
        int at;
        const unsigned long long kmax = wave_max_key(
            valid ? ((unsigned long long)__float_as_uint(d) << 32) | o : 0ull, at);
        const float thr = prune_threshold(r, key_d2(kmax));
        const float row = thr == 0.0f ? INFINITY
                                      : -filter_row(thr, norm2(c.x - job.ox, c.y - job.oy, c.z - job.oz));
        if (lane == 0) {
            tkey[s] = kmax;
            trow[s] = row;
        }
    };

    // Seed and initial update (Sec. 3.3)
    {
        const uint32_t p0 = a.inv[job.point_base + (uint32_t)job.start];
        const float sx = a.xs[p0], sy = a.ys[p0], sz = a.zs[p0];
        __syncthreads();
        for (int i = 0; i < ntw; ++i) {
            const uint32_t meta = tmeta[wb + i];
            const uint32_t ls = meta & 0xffffu, c = meta >> 16;
            const uint32_t gs = a.tstart[job.tb + rank + (size_t)(i * kRWaves + wave) * G];
            float dp = 0.0f;
            uint32_t op = 0;
            if ((uint32_t)lane < c) {
                const uint32_t q = gs + lane, p = ls + lane;
                const float x = a.xs[q], y = a.ys[q], z = a.zs[q];
                const float d0 = sqdist(x, y, z, sx, sy, sz);
                dp = euclid ? sqrt_class_top(d0) : d0;
                op = ~(a.orig[q] - job.point_base);
                pq[p] = make_float4(x, y, z, __uint_as_float(op));
                pd[p] = dp;
            }
            rekey(wb + i, (uint32_t)lane < c, dp, op);
        }
        if (tid == 0)
            sh.abort = 0;
        if (tid < kList)
            sh.prank[tid] = 0u;
        if (tid < 2)
            sh.gb[tid] = sh.sx[tid] = 0ull;
        __syncthreads();
    }

    // ---- this thread's units of every exchange ----
    const int units = (int)slot_units(K);
    const int total = solo ? kRWaves * steps : G * units;
    uint32_t upos[NU];            // word offset of its units on the board
    bool uin[NU], ubound[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int e = tid + u * kRBlock;
        const int g = e / units, s = e - g * units;
        uin[u] = e < total;
        ubound[u] = !solo && s == K;
        upos[u] = uin[u] ? g * board.slot_words + s * kUnit : 0u;
    }
    const unsigned long long below = lane ? (~0ull >> (kWave - lane)) : 0ull;

    unsigned long long t_mark = 0;
    int j = 1;
    uint32_t round = 0;
    int j_out = 1, n_out = 0, p_out = 0;  // the last round's outputs, written during the next exchange (rank 0)

    // Outputs of the last round (rank 0): a pick's position is its rank in key
    // order among the picks, of which only the first n_out count.  Every
    // wavefront counts the larger keys among its share of the picks, for all
    // of them; after a barrier the threads of write_out store the results.
    auto rank_out = [&]() {
        for (int i0 = 0; i0 < p_out; i0 += kWave) {
            const int i = i0 + lane;
            const unsigned long long ki = sh.pkey[i < p_out ? i : 0];
            uint32_t r = 0;
            // (positions past the picks hold older keys: masked)
            for (int q = wave; q < p_out; q += 4 * kRWaves)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int qv = q + v * kRWaves;
                    r += (sh.pkey[qv & (kList - 1)] > ki && qv < p_out) ? 1u : 0u;
                }
            if (i < p_out && r)
                atomicAdd(&sh.prank[i], r);
        }
    };
    auto write_out = [&](int t) {
        for (int i = t; i < p_out; i += kWave) {
            const int r = (int)sh.prank[i];
            sh.prank[i] = 0u;
            if (r < n_out) {
                const unsigned long long k = sh.pkey[i];
                job.out_idx[j_out + r] = (int32_t)key_orig(k);
                if (job.out_d2)
                    job.out_d2[j_out + r] = key_d2(k);
            }
        }
    };

    while (j < job.m) {
        ++round;
        ++epoch;
        if (clocks)
            t_mark = wall_clock64();
        // =============== L: lookahead of every wavefront on its own tiles ===============
        // A candidate is the largest key of the wavefront's tiles; it is then
        // applied to its own tile only, on a copy in registers (other tiles
        // keep their keys, which bound their points from above), and the next
        // step takes the largest key again.  A tile whose key was lowered by
        // its own candidate holds the lowered key in LDS until the lookahead
        // ends, when the true key is put back.
        {
            // (lane 0 stored the tile keys of the apply phase)
            wave_sync();
            unsigned long long t_step = 0;  // when the first step was done
            const int rb = wave * steps;
            unsigned long long bound = 0;
            // candidate s: lane p of the loaded tile (coordinates q, distance
            // bits db), with the largest distance of its wavefront's others u
            auto record = [&](int s, bool own, const float4 &q, uint32_t db, uint32_t u) {
                if (own) {
                    const uint32_t x = __float_as_uint(q.x), y = __float_as_uint(q.y), z = __float_as_uint(q.z),
                                   o = __float_as_uint(q.w);
                    sh.rec[rb + s][0] = u32x4{x, y & 0xffffu, (y >> 16) | (z << 16), z >> 16};
                    sh.rec[rb + s][1] = u32x4{db, o & 0xffffu, (o >> 16) | (u << 16), u >> 16};
                    sh.rkey[rb + s] = ((unsigned long long)db << 32) | o;
                }
            };
            // One step on a loaded tile (points q, distances d) whose largest
            // key is bk: lane p of it, the largest distance of the others, and
            // the tile's key once p is applied to it (d follows).
            auto step = [&](const float4 &q, float &d, bool valid, unsigned long long bk, int &p, uint32_t &rest,
                            unsigned long long &nk) {
                // key low halves are unique to their points
                const uint32_t o = __float_as_uint(q.w);
                p = __builtin_ctzll(ballot64(o == (uint32_t)bk) & ballot64(valid));
                const float cx = lane_f32(q.x, p), cy = lane_f32(q.y, p), cz = lane_f32(q.z, p);
                const uint32_t db = valid && lane != p ? __float_as_uint(d) : 0u;
                d = min_dist(d, sqdist(q.x, q.y, q.z, cx, cy, cz), euclid);
                const uint32_t nb = valid ? __float_as_uint(d) : 0u;
                rest = wave_max_u32(db);
                const uint32_t mh = wave_max_u32(nb);
                unsigned long long tie = ballot64(nb == mh) & ballot64(valid);
                if (tie & (tie - 1)) {
                    const uint32_t ml = wave_max_u32(((tie >> lane) & 1ull) ? o : 0u);
                    tie &= ballot64(o == ml);
                }
                nk = ((unsigned long long)mh << 32) | lane_u32(o, __builtin_ctzll(tie));
            };
            auto load = [&](uint32_t meta, float4 &q, float &d, bool &valid) {
                const uint32_t ls = meta & 0xffffu, cnt = meta >> 16;
                valid = (uint32_t)lane < cnt;
                const uint32_t pp = ls + (valid ? lane : 0);
                q = pq[pp];
                d = pd[pp];
            };
            if (ntw <= kWave) {
                // The usual case, a tile per lane: the keys the lookahead
                // lowers stay in registers.
                unsigned long long k1 = lane < ntw ? tkey[wb + lane] : 0ull, oth = 0;
                const uint32_t m1 = lane < ntw ? tmeta[wb + lane] : 0u;
                int h, ho = 0;
                unsigned long long bk = wave_max_key(k1, h);
                if (bk == 0) {
                    // a wavefront without points: no candidates, bound 0
                    if (lane < steps) {
                        sh.rkey[rb + lane] = 0ull;
                        sh.rec[rb + lane][0] = u32x4{0u, 0u, 0u, 0u};
                        sh.rec[rb + lane][1] = u32x4{0u, 0u, 0u, 0u};
                    }
                } else {
                    float4 q;
                    float d;
                    bool valid;
                    load(lane_u32(m1, h), q, d, valid);
                    oth = wave_max_key(lane == h ? 0ull : k1, ho);
                    float4 qn;  // the tile that comes next if another one does
                    float dn;
                    bool vn;
                    load(lane_u32(m1, ho), qn, dn, vn);
                    int ctile = -1;  // lane s: the tile of candidate s
                    for (int s = 0;;) {
                        int p;
                        uint32_t rest;
                        unsigned long long nk;
                        const uint32_t db = __float_as_uint(d);
                        step(q, d, valid, bk, p, rest, nk);
                        record(s, lane == p, q, db, max(rest, (uint32_t)(oth >> 32)));
                        bound = umax64(nk, oth);
                        if (lane == s)
                            ctile = h;
                        if (clocks && s == 0)
                            t_step = wall_clock64();
                        if (++s == steps)
                            break;
                        bk = bound;
                        if (nk < oth) {
                            // the next candidate comes from another tile
                            if (lane == h)
                                k1 = nk;
                            h = ho;
                            q = qn;
                            d = dn;
                            valid = vn;
                            oth = wave_max_key(lane == h ? 0ull : k1, ho);
                            if (s + 1 < steps)
                                load(lane_u32(m1, ho), qn, dn, vn);
                            unsigned long long mine = ballot64(ctile == h);
                            if (mine) {
                                wave_sync();  // the records are other lanes'
                                float least = INFINITY;
                                for (; mine; mine &= mine - 1) {
                                    const int c = __builtin_ctzll(mine);
                                    const Cand l = unpack_cand(sh.rec[rb + c][0], sh.rec[rb + c][1]);
                                    least = fminf(least, sqdist(q.x, q.y, q.z, l.x, l.y, l.z));
                                }
                                d = min_dist(d, least, euclid);
                            }
                        }
                    }
                }
            } else {
                unsigned long long bk, oth;  // the largest key, and the largest of the other tiles
                int bt;                      // the tile of bk
                uint32_t meta;               // and its points
                auto scan = [&]() {
                    unsigned long long k1 = 0, k2 = 0;
                    int i1 = 0;
                    uint32_t m1 = 0;
                    for (int i = lane; i < ntw; i += kWave) {
                        const unsigned long long k = tkey[wb + i];
                        const uint32_t m = tmeta[wb + i];
                        const bool top = k > k1;
                        k2 = top ? k1 : umax64(k, k2);
                        k1 = top ? k : k1;
                        i1 = top ? i : i1;
                        m1 = top ? m : m1;
                    }
                    int hl, ol;
                    bk = wave_max_key(k1, hl);
                    bt = __builtin_amdgcn_readlane(i1, hl);
                    meta = lane_u32(m1, hl);
                    oth = wave_max_key(lane == hl ? k2 : k1, ol);
                };
                scan();
                if (bk == 0) {
                    // a wavefront without points: no candidates, bound 0
                    if (lane < steps) {
                        sh.rkey[rb + lane] = 0ull;
                        sh.rec[rb + lane][0] = u32x4{0u, 0u, 0u, 0u};
                        sh.rec[rb + lane][1] = u32x4{0u, 0u, 0u, 0u};
                    }
                } else {
                    float4 q = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    float d = 0.0f;
                    bool valid = false;
                    int cur = -1;
                    int ctile = -1;               // lane q: the tile of candidate q
                    int svt = -1, nsv = 0;        // lane q: the q-th tile whose key was lowered,
                    unsigned long long svk = 0;   // and its true key
                    unsigned long long curk = 0;  // key of the loaded tile when it was taken
                    for (int s = 0;;) {
                        if (cur != bt) {
                            cur = bt;
                            curk = bk;
                            load(meta, q, d, valid);
                            unsigned long long mine = ballot64(ctile == bt);
                            wave_sync();  // the records are other lanes'
                            while (mine) {
                                const int c = __builtin_ctzll(mine);
                                mine &= mine - 1;
                                const Cand l = unpack_cand(sh.rec[rb + c][0], sh.rec[rb + c][1]);
                                d = min_dist(d, sqdist(q.x, q.y, q.z, l.x, l.y, l.z), euclid);
                            }
                        }
                        int p;
                        uint32_t rest;
                        unsigned long long nk;
                        const uint32_t db = __float_as_uint(d);
                        step(q, d, valid, bk, p, rest, nk);
                        record(s, lane == p, q, db, max(rest, (uint32_t)(oth >> 32)));
                        if (lane == s)
                            ctile = bt;
                        bound = umax64(nk, oth);
                        if (clocks && s == 0)
                            t_step = wall_clock64();
                        if (++s == steps)
                            break;
                        if (nk >= oth) {
                            bk = nk;
                        } else {
                            if (!ballot64(svt == cur)) {
                                if (lane == nsv) {
                                    svt = cur;
                                    svk = curk;
                                }
                                ++nsv;
                            }
                            wave_sync();  // the scan before has read the keys
                            if (lane == 0)
                                tkey[wb + cur] = nk;
                            wave_sync();
                            scan();
                        }
                    }
                    wave_sync();
                    if (lane < nsv)
                        tkey[wb + svt] = svk;
                }
            }
            if (clocks && t_step)
                tl.later += wall_clock64() - t_step;
            if (lane == 0)
                atomicMax(&sh.gb[round & 1u], bound);
        }
        __syncthreads();
        if (tid == 0)
            sh.gb[(round + 1u) & 1u] = 0ull;  // last read before this barrier
        if (clocks) {
            const unsigned long long t = wall_clock64();
            tl.ph[0] += t - t_mark;
            t_mark = t;
        }

        // =============== X: publish and read every slot ===============
        // A workgroup publishes its K largest candidates and a bound on every
        // other point's key: the largest of its wavefronts' bounds and of its
        // next candidate.  Every wavefront finds the ranks of its own
        // candidates and publishes those below K at their rank; the one that
        // owns the next candidate publishes the bound.  Every thread then
        // reads its own units of the whole team's slots into registers.
        const unsigned long long t_pub = trace ? wall_clock64() : 0ull;
        Cand cd[NU];
        unsigned long long ck[NU];  // candidate keys (0: none)
        unsigned long long smax;    // S*, the largest bound of the team
        float4 cb[NU];              // candidates' shifted coordinates and column term
        float ct[NU];               // and minus their row term
        unsigned long long cx[NU];  // lanes whose candidate is too far from the origin for the filter
        auto prepare = [&]() {
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const Cand &c = cd[u];
                float sx = c.x - job.ox, sy = c.y - job.oy, sz = c.z - job.oz;
                const float n2 = norm2(sx, sy, sz);
                if (!(n2 <= 1e36f))
                    sx = sy = sz = 0.0f;  // kept whatever the other point: no product may be NaN
                cb[u] = make_float4(sx, sy, sz, filter_col(n2));
                ct[u] = -filter_row(__uint_as_float(c.d), n2);
                cx[u] = ballot64(filter_blurred(n2, __uint_as_float(c.d), j));
            }
        };
        bool solo_out = false;      // outputs of the last round wait for a barrier
        if (!solo) {
            const uint32_t tag = tag_of(epoch);
            {
                const int nr = kRWaves * steps, c0 = wave * steps;
                const unsigned long long kq = lane < nr ? sh.rkey[lane] : 0ull;
                const unsigned long long gb = sh.gb[round & 1u];
                unsigned long long *slot = board.base + (epoch & 1u) * board.par_words + rank * board.slot_words;
                const unsigned long long tag64 = (unsigned long long)tag << 48;
                for (int s = 0; s < steps; ++s) {
                    const int c = c0 + s;
                    const unsigned long long w =
                        reinterpret_cast<const unsigned long long *>(sh.rec[c])[lane & (kUnit - 1)];
                    const unsigned long long kc = lane_u64(kq, c);
                    // equal keys (empty wavefronts, or one point repeated): by position
                    const int r = __popcll(ballot64(kq > kc) | (ballot64(kq == kc) & ((1ull << c) - 1ull)));
                    if (r < K && lane < kUnit)
                        bstore<S>(slot + r * kUnit + lane, tag64 | w);
                    if (r == K && lane < kUnit) {  // (there are at least 16 candidates, more than K)
                        const unsigned long long b = umax64(gb, kc);
                        bstore<S>(slot + K * kUnit + lane, tag64 | (lane == 0 ? b >> 32 : b & 0xffffffffull));
                    }
                }
            }
            if (rank == 0 && n_out)
                rank_out();
            const unsigned long long *sbase = board.base + (epoch & 1u) * board.par_words;
            unsigned long long b = 0;
            // The passes after the first are waiting.  (Of the whole first
            // wavefront: thread 0 reads its own workgroup's slot.)
            const bool timed_wave = T && ballot64(clocks) != 0ull;
            unsigned long long t_first = 0;
            bool lost = false;
            const uint32_t tagw = tag << 16;
            auto fresh = [&](const u32x4 &x, const u32x4 &y) {
                return ((((x.y ^ tagw) | (x.w ^ tagw)) | ((y.y ^ tagw) | (y.w ^ tagw))) >> 16) == 0u;
            };
            auto aborted = [&](const u32x4 &x) { return (x.y >> 16) == kAbortTag; };
            auto take = [&](int u, const u32x4 &x, const u32x4 &y) {
                cd[u] = unpack_cand(x, y);
                ck[u] = ubound[u] || !uin[u] ? 0ull : ((unsigned long long)cd[u].d << 32) | cd[u].o;
                if (ubound[u])
                    b = umax64(b, ((unsigned long long)x.x << 32) | x.z);
            };
            if constexpr (NU == 2) {
                // both units' loads in flight together
                bool p0 = uin[0], p1 = uin[1];
                ck[0] = ck[1] = 0ull;
                for (uint32_t spin = 0; p0 || p1; ++spin) {
                    if (timed_wave && spin == 1 && !t_first)
                        t_first = wall_clock64();
                    u32x4 x0, y0, x1, y1;
                    load_unit2(sbase + upos[0], sbase + upos[1], x0, y0, x1, y1);
                    if (p0 && fresh(x0, y0)) {
                        take(0, x0, y0);
                        p0 = false;
                    }
                    if (p1 && fresh(x1, y1)) {
                        take(1, x1, y1);
                        p1 = false;
                    }
                    if ((p0 && aborted(x0)) || (p1 && aborted(x1)) || spin >= kSpinLimit) {
                        lost = true;
                        break;
                    }
                }
            } else {
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    ck[u] = 0ull;
                    bool p0 = uin[u];
                    for (uint32_t spin = 0; p0; ++spin) {
                        if (timed_wave && spin == 1 && !t_first)
                            t_first = wall_clock64();
                        u32x4 x0, y0;
                        load_unit(sbase + upos[u], x0, y0);
                        if (fresh(x0, y0)) {
                            take(u, x0, y0);
                            p0 = false;
                        } else if (aborted(x0) || spin >= kSpinLimit) {
                            lost = true;
                            break;
                        }
                    }
                }
            }
            if (lost)
                sh.abort = 1;
            if (timed_wave && ballot64(t_first != 0ull)) {
                int first;
                const unsigned long long t0 = ~wave_max_key(t_first ? ~t_first : 0ull, first);
                if (clocks)
                    tl.ph[4] += wall_clock64() - t0;
            }
            if (clocks)
                tl.poll += wall_clock64() - t_mark;
            // what the list needs of this thread's candidates, while the
            // wavefront's bound is reduced
            prepare();
            int at;
            b = wave_max_key(b, at);
            if (lane == 0 && b)
                atomicMax(&sh.sx[round & 1u], b);
            __syncthreads();
            if (sh.abort) {
                if (tid == 0) {
                    set_status(&a.hdr->sample_status, RFPS_ERR_TIMEOUT);
                    publish_abort_tags<S>(board, rank, K);
                }
                return false;
            }
            if (rank == 0 && n_out && wave == kRWaves - 1)
                write_out(lane);
            smax = sh.sx[round & 1u];
            if (tid == 0)
                sh.sx[(round + 1u) & 1u] = 0ull;  // last read in the round before
        } else {
            if (n_out)
                rank_out();
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                ck[u] = 0ull;
                if (uin[u]) {
                    const int e = tid + u * kRBlock;
                    cd[u] = unpack_cand(sh.rec[e][0], sh.rec[e][1]);
                    ck[u] = sh.rkey[e];
                }
            }
            prepare();
            smax = sh.gb[round & 1u];
            solo_out = n_out != 0;
        }
        if (clocks) {
            const unsigned long long t = wall_clock64();
            tl.ph[1] += t - t_mark;
            tl.rest += t - t_mark;  // the poll's share is taken off below
            t_mark = t;
        }

        // =============== M: certified merge (whole workgroup) ===============
        // The candidates above S*, in the order of the units (the same in
        // every workgroup).  A candidate at distance 0 is never listed: when
        // nothing is left above distance 0, the loop ends below.  Positions
        // past kList are counted only.
        uint32_t L;
        bool blurred;  // some listed candidate is too far from the origin for the filter
        constexpr uint32_t kFarCount = 1u << 16;  // beside the counts, which stay below
        auto list_above = [&](unsigned long long lim) {
            uint32_t mine = 0;
            unsigned long long km[NU], far = 0;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                km[u] = ballot64(ck[u] > lim) & ballot64((ck[u] >> 32) != 0ull);
                mine += (uint32_t)__popcll(km[u]);
                far |= km[u] & cx[u];
            }
            if (lane == 0)
                sh.cnt[wave] = mine + (far ? kFarCount : 0u);
            __syncthreads();
            uint32_t base = 0;
            L = 0;
#pragma unroll
            for (int q = 0; q < kRWaves; ++q) {
                const uint32_t c = sh.cnt[q];
                base += q < wave ? c : 0u;
                L += c;
            }
            base %= kFarCount;
            blurred = L >= kFarCount;
            L %= kFarCount;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const uint32_t pos = base + (uint32_t)__popcll(km[u] & below);
                if (((km[u] >> lane) & 1ull) && pos < (uint32_t)kList) {
                    sh.lq[pos] = make_float4(cd[u].x, cd[u].y, cd[u].z, __uint_as_float(cd[u].u));
                    sh.lb[pos] = cb[u];
                    sh.ld[pos] = __uint_as_float(cd[u].d);
                    sh.lT[pos] = ct[u];
                    sh.lkey[pos] = ck[u];
                }
                base += (uint32_t)__popcll(km[u]);
            }
            __syncthreads();
        };
        list_above(smax);
        if (solo_out && wave == kRWaves - 1)
            write_out(lane);
        // scur: every listed key is above it, and every point left out of the
        // list has its true key at most it
        unsigned long long scur = smax;
        if (L == 0) {
            // The largest key is never a bound unless its distance is 0 (keys
            // of different points differ, and a candidate's own key falls to
            // distance 0 once it is applied), so every distance is 0: the
            // lowest index is selected for good (Sec. 3.1).
            unsigned long long mk = 0;
#pragma unroll
            for (int u = 0; u < NU; ++u)
                mk = umax64(mk, ck[u]);
            int at;
            mk = wave_max_key(mk, at);
            if (lane == 0)
                sh.red2[wave] = mk;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kRWaves; ++q)
                mk = umax64(mk, sh.red2[q]);
            if (mk == 0 || (mk >> 32) != 0) {
                // impossible by construction; a guard so that a violated
                // invariant ends the call
                if (tid == 0)
                    set_status(&a.hdr->sample_status, RFPS_ERR_INTERNAL);
                return false;
            }
            if (rank == 0) {
                for (int q = j + tid; q < job.m; q += kRBlock) {
                    job.out_idx[q] = (int32_t)key_orig(mk);
                    if (job.out_d2)
                        job.out_d2[q] = 0.0f;
                }
            }
            if (trace && round - 1 < (uint32_t)kTraceCap) {
                a.trace[2 * (size_t)(round - 1)] = t_pub;
                a.trace[2 * (size_t)(round - 1) + 1] =
                    wall_clock64() | ((unsigned long long)min(job.m - j, 0xffff) << 48);
            }
            n_out = 0;
            break;
        }
        if (T && clocks)
            tl.above += L;
        if (L > (uint32_t)kList) {
            // Too many for one round: find a key with at most kList (and at
            // least half as many) candidates above it, by 256-bin histograms
            // of the keys' range, narrowed to the bin that holds the edge.
            unsigned long long hm = 0;
#pragma unroll
            for (int u = 0; u < NU; ++u)
                hm = umax64(hm, ck[u]);
            int at;
            hm = wave_max_key(hm, at);
            if (lane == 0)
                sh.red2[wave] = hm;
            __syncthreads();
            unsigned long long hi = 0;
#pragma unroll
            for (int q = 0; q < kRWaves; ++q)
                hi = umax64(hi, sh.red2[q]);
            unsigned long long lo = umax64(smax, 0xffffffffull) + 1ull;  // keys of the range: lo .. hi
            uint32_t have = 0;                                           // candidates above the range
            for (;;) {
                const int bits = 64 - __clzll((long long)((hi - lo) | 1ull));
                const int shift = bits > 8 ? bits - 8 : 0;
                __syncthreads();
                if (tid < 256)
                    sh.hist[tid] = 0;
                __syncthreads();
#pragma unroll
                for (int u = 0; u < NU; ++u)
                    if (ck[u] >= lo && ck[u] <= hi)
                        atomicAdd(&sh.hist[(uint32_t)((ck[u] - lo) >> shift)], 1u);
                __syncthreads();
                if (wave == 0) {
                    // the lowest bin such that it and those above hold at most kList - have
                    uint32_t c4[4], sum = 0;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        c4[v] = sh.hist[4 * lane + v];
                        sum += c4[v];
                    }
                    uint32_t suf = sum;
#pragma unroll
                    for (int o = 1; o < kWave; o <<= 1) {
                        const uint32_t v = (uint32_t)__shfl_down((int)suf, o, kWave);
                        suf += lane + o < kWave ? v : 0u;
                    }
                    uint32_t acc = suf - sum, bin = 256, tot = 0;
#pragma unroll
                    for (int v = 3; v >= 0; --v) {
                        acc += c4[v];
                        if (acc <= (uint32_t)kList - have) {
                            bin = 4 * lane + v;
                            tot = acc;
                        }
                    }
                    const uint32_t lowest = wave_min_u32(bin);
                    const unsigned long long own = ballot64(bin == lowest);
                    if (lane == __ffsll((long long)own) - 1) {
                        sh.cut_bin = lowest;
                        sh.cut_have = lowest < 256 ? tot : 0u;
                    }
                }
                __syncthreads();
                const uint32_t bin = sh.cut_bin;
                have += sh.cut_have;
                const unsigned long long edge = lo + ((unsigned long long)bin << shift);
                if (have >= (uint32_t)kList / 2 || shift == 0 || bin == 0) {
                    scur = edge - 1ull;
                    break;
                }
                hi = edge - 1ull;  // the bin below holds more than fit: narrow the range to it
                lo = edge - (1ull << shift);
            }
            __syncthreads();
            list_above(scur);
        }
        const int nb = (int)((L + kBlk - 1) / kBlk);
        unsigned long long t_sub = 0;
        if (clocks) {
            t_sub = wall_clock64();
            tl.list += t_sub - t_mark;
            tl.listed += L;
        }

        // Conflicts: for every listed candidate i, the set of listed
        // candidates q of no smaller distance that may lower it.  The matrix
        // cores test 16 x 16 blocks of pairs with a margin that keeps every
        // true conflict (filter_row); the certification checks the kept ones
        // it meets exactly, ties of the distance included.  Columns are i: a
        // lane holds one i and four q per block, so it collects its part of
        // the row of i without exchange.
        {
            // Where the cloud's extent is far beyond its distances (a point
            // or a part far from the rest), the filter's terms cancel and it
            // keeps every pair, of which a pass of the certification clears
            // one a candidate.  Such a round checks its pairs here, a
            // wavefront taking a word of a row at a time.  (Every workgroup
            // has the same list and so decides alike: the passes, and with
            // them the bound, depend on what the rows hold.)  A room of 80,000
            // points and one 12 km away, per round: certification 40 us by the
            // filter's rows; conflicts 3.5 and certification 0.8 by these.
            // Whole call 24.6 -> 11.6 ms.
            auto exact_conflicts = [&]() {
                const int nw = L <= kWave ? 1 : L <= 2 * kWave ? 2 : 4, qs = nb <= 12 ? 3 : 4;
#pragma unroll 1
                for (int w = 0; w < nw; ++w) {
                    const int q = nw == 1   ? conflict_pos<1>(w, lane, qs)
                                  : nw == 2 ? conflict_pos<2>(w, lane, qs)
                                            : conflict_pos<4>(w, lane, qs);
                    const bool in = q < (int)L;
                    const float4 c = sh.lq[in ? q : 0];
                    const unsigned long long kq = in ? sh.lkey[q] : 0ull;
#pragma unroll 2
                    for (int i = wave; i < (int)L; i += kRWaves) {
                        const float4 p = sh.lq[i];
                        const float d = sh.ld[i];
                        const float t = min_dist(d, sqdist(p.x, p.y, p.z, c.x, c.y, c.z), euclid);
                        const unsigned long long row = ballot64(t < d) & ballot64(kq > sh.lkey[i]);
                        if (lane == 0)
                            sh.adj[i * nw + w] = row;
                    }
                }
            };
            // NP wavefronts split the row blocks (QS each, kept in registers)
            // and the others the columns: what a wavefront reads of LDS is
            // what bounds this phase (1.4 us for lists of about 150; 2.4 with
            // the row data read again for every block).  A lane stores the
            // bits of its row blocks at once.  Row blocks past the list give
            // bits of positions past it, which no live mask holds.
            const float *lbf = reinterpret_cast<const float *>(sh.lb);
            auto conflicts = [&](auto qs_c, auto np_c) {
                constexpr int QS = decltype(qs_c)::value, NP = decltype(np_c)::value;
                const int part = wave & (NP - 1);
                if (part * QS >= nb)
                    return;
                float av[QS];
                float4 dr[QS];
#pragma unroll
                for (int v = 0; v < QS; ++v) {
                    const int rb = part * QS + v;
                    av[v] = lbf[(rb * kBlk + li) * 4 + lg];
                    dr[v] = *reinterpret_cast<const float4 *>(&sh.ld[rb * kBlk + 4 * lg]);
                }
                for (int cb = wave / NP; cb < nb; cb += kRWaves / NP) {
                    const int i = cb * kBlk + li;
                    const float bv = lbf[i * 4 + lg];
                    const float bv2 = lg == 3 ? 1.0f : -2.0f * bv;
                    const float ti = sh.lT[i];
                    // the next value below the distance: q of the same
                    // distance give a negative difference too
                    const float di = __uint_as_float(__float_as_uint(sh.ld[i]) - 1u);
                    f32x4 dd[QS];
#pragma unroll
                    for (int v = 0; v < QS; ++v)
                        dd[v] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[v], bv2, f32x4{ti, ti, ti, ti}, 0, 0, 0);
                    // a pair is kept when both terms are negative: their
                    // common sign bit goes into the row
                    uint32_t acc = 0;
                    auto put = [&](float x, float dq) {
                        acc = __builtin_amdgcn_alignbit(acc, __float_as_uint(x) & __float_as_uint(di - dq), 31);
                    };
#pragma unroll
                    for (int v = QS - 1; v >= 0; --v) {
                        put(dd[v][3], dr[v].w);
                        put(dd[v][2], dr[v].z);
                        put(dd[v][1], dr[v].y);
                        put(dd[v][0], dr[v].x);
                    }
                    // a candidate and itself
                    const int v = cb - part * QS;
                    if (v >= 0 && v < QS)
                        acc &= lg == li / 4 ? ~(1u << (4 * v + li % 4)) : ~0u;
                    if constexpr (QS <= 2)
                        reinterpret_cast<uint8_t *>(sh.adj)[(i * 4 + lg) * NP + part] = (uint8_t)acc;
                    else
                        reinterpret_cast<uint16_t *>(sh.adj)[(i * 4 + lg) * NP + part] = (uint16_t)acc;
                }
            };
            const std::integral_constant<int, 4> c4{};
            if (blurred)
                exact_conflicts();
            else if (nb <= 4)
                conflicts(std::integral_constant<int, 2>(), std::integral_constant<int, 2>());
            else if (nb <= 8)
                conflicts(std::integral_constant<int, 2>(), c4);
            else if (nb <= 12)
                conflicts(std::integral_constant<int, 3>(), c4);
            else
                conflicts(c4, c4);
        }
        __syncthreads();
        if (clocks) {
            const unsigned long long t = wall_clock64();
            tl.conflicts += t - t_sub;
            t_sub = t;
        }

        // Certification, in registers, on wavefront 0 for lists of up to 128
        // and on four wavefronts for longer ones (a pass over four rows per
        // lane on one wavefront took 3.1 us a round, split over four 1.7;
        // two rows do not pay for the two barriers).  Lane l holds the listed
        // candidates at conflict_pos(w, l) with their conflict rows.  A live
        // candidate with no live one in its row is free: it is a pick if the
        // round gets that far.  One that a free candidate lowers has failed:
        // its true key is at most its distance to that candidate, and the
        // other points of its wavefront are bounded by its runner-up, so the
        // bound rises to the larger of the two.  Failed candidates and every
        // key at or below the bound leave, and so on until every live
        // candidate is free.  (The live candidate with the largest key that is
        // not free always has a free one in its row, so every pass ends one or
        // clears a pair that is no conflict; a failed candidate the sequence
        // would not have reached has its key, and so both of its terms, below
        // the bound already.)
        if (wave == 0) {
            auto walk = [&](auto nw_c) {
                constexpr int NW = decltype(nw_c)::value;
                const int qs = nb <= 12 ? 3 : 4;
                unsigned long long s[NW][NW], key[NW], lv[NW];
                float4 q[NW];
#pragma unroll
                for (int k = 0; k < NW; ++k) {
                    const int i = conflict_pos<NW>(k, lane, qs);
                    const bool in = (uint32_t)i < L;
                    lv[k] = ballot64(in);
                    const int ii = in ? i : 0;
#pragma unroll
                    for (int w = 0; w < NW; ++w)
                        s[k][w] = sh.adj[ii * NW + w];
                    q[k] = sh.lq[ii];
                    key[k] = sh.lkey[ii];
                }
                uint32_t nfail = 0;
                bool ties = false;  // the last pass ended nothing: mutual ties
                for (;;) {
                    unsigned long long f[NW], fr[NW], any = 0;
#pragma unroll
                    for (int k = 0; k < NW; ++k) {
                        unsigned long long acc = 0;
#pragma unroll
                        for (int w = 0; w < NW; ++w)
                            acc |= s[k][w] & lv[w];
                        f[k] = ballot64(acc != 0ull) & lv[k];
                        any |= f[k];
                    }
                    if (!any)
                        break;
#pragma unroll
                    for (int k = 0; k < NW; ++k)
                        fr[k] = ties ? lv[k] : lv[k] & ~f[k];
                    unsigned long long b = 0, met = 0;
#pragma unroll
                    for (int k = 0; k < NW; ++k) {
                        // the first free candidate of its row (the list has one
                        // order in every workgroup, so all find the same bound)
                        int at = 0, aw = -1;
                        unsigned long long bit = 0;
#pragma unroll
                        for (int w = NW - 1; w >= 0; --w) {
                            const unsigned long long h = s[k][w] & fr[w];
                            if (h) {
                                at = conflict_pos<NW>(w, __ffsll((long long)h) - 1, qs);
                                bit = h & (0ull - h);
                                aw = w;
                            }
                        }
                        bool fails = false;
                        const bool meets = ((f[k] >> lane) & 1ull) && aw >= 0;
                        if (meets) {
                            const float4 p = sh.lq[at];
                            const float d = key_d2(key[k]);
                            const float t = min_dist(d, sqdist(q[k].x, q[k].y, q[k].z, p.x, p.y, p.z), euclid);
                            // a pair within the filter's margin, or a tie of
                            // the distance with the smaller key, is no conflict
                            const bool real = t < d && sh.lkey[at] > key[k];
                            fails = real && !ties;
#pragma unroll
                            for (int w = 0; w < NW; ++w)
                                s[k][w] &= (!real && aw == w) ? ~bit : ~0ull;
                            const unsigned long long kt =
                                ((unsigned long long)__float_as_uint(t) << 32) | (uint32_t)key[k];
                            // the runner-up's key is below this one's
                            const unsigned long long ku =
                                ((unsigned long long)__float_as_uint(q[k].w) << 32) | 0xffffffffull;
                            const unsigned long long kb = umax64(kt, ku < key[k] ? ku : key[k] - 1ull);
                            b = fails ? umax64(b, kb) : b;
                        }
                        const unsigned long long om = ballot64(fails);
                        lv[k] &= ~om;
                        met |= ballot64(meets);
                        nfail += (uint32_t)__popcll(om);
                    }
                    // no free candidate in any row: only ties of the distance
                    // hold the largest of them back; clear those next
                    ties = met == 0ull;
                    int at;
                    scur = umax64(scur, wave_max_key(b, at));
#pragma unroll
                    for (int k = 0; k < NW; ++k)
                        lv[k] &= ballot64(key[k] > scur);
                }
                if (clocks) {
                    const unsigned long long t = wall_clock64();
                    tl.walk += t - t_sub;
                    t_sub = t;
                }
                // the picks, in any order, for the apply phase and the outputs
                uint32_t n = 0;
#pragma unroll
                for (int k = 0; k < NW; ++k) {
                    const uint32_t pos = n + (uint32_t)__popcll(lv[k] & below);
                    if ((lv[k] >> lane) & 1ull) {
                        sh.pk[pos] = q[k];
                        sh.pk[kList + pos] = sh.lb[conflict_pos<NW>(k, lane, qs)];
                        sh.pkey[pos] = key[k];
                    }
                    n += (uint32_t)__popcll(lv[k]);
                }
                // padding of the last block: columns that pass no filter
                if (lane < kBlk && n + lane < (n + kBlk - 1) / kBlk * kBlk)
                    sh.pk[kList + n + lane] = make_float4(0.0f, 0.0f, 0.0f, INFINITY);
                if (lane == 0)
                    sh.npick = n;
                if (clocks)
                    tl.fails += nfail;
            };
            if (L <= kWave)
                walk(std::integral_constant<int, 1>());
            else if (L <= 2 * kWave)
                walk(std::integral_constant<int, 2>());
        }
        if (L > 2 * kWave) {
            // The same for longer lists, on four wavefronts: wavefront w takes
            // the candidates of word w, and masks and bound meet in LDS.
            const int qs = nb <= 12 ? 3 : 4;
            const int w4 = wave & 3;
            unsigned long long s[4], key[4], lv[4];
            float4 q = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            const int own = conflict_pos<4>(w4, lane, qs);
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int i = conflict_pos<4>(w, lane, qs);
                lv[w] = ballot64((uint32_t)i < L);
                key[w] = sh.lkey[(uint32_t)i < L ? i : 0];
                s[w] = sh.adj[((uint32_t)own < L ? own : 0) * 4 + w];
            }
            q = sh.lq[(uint32_t)own < L ? own : 0];
            const unsigned long long k0 = w4 == 0 ? key[0] : w4 == 1 ? key[1] : w4 == 2 ? key[2] : key[3];
            uint32_t nfail = 0;
            bool ties = false;
            for (;;) {
                if (wave < 4) {
                    const unsigned long long acc = (s[0] & lv[0]) | (s[1] & lv[1]) | (s[2] & lv[2]) | (s[3] & lv[3]);
                    const unsigned long long f = ballot64(acc != 0ull) &
                                                 (w4 == 0 ? lv[0] : w4 == 1 ? lv[1] : w4 == 2 ? lv[2] : lv[3]);
                    if (lane == 0)
                        sh.wf[wave] = f;
                    if (tid == 0)
                        sh.wscur = 0ull;
                }
                __syncthreads();
                unsigned long long f[4], fr[4];
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    f[w] = lane_u64(sh.wf[w], 0);
                if (!(f[0] | f[1] | f[2] | f[3]))
                    break;
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    fr[w] = ties ? lv[w] : lv[w] & ~f[w];
                if (wave < 4) {
                    int at = 0, aw = -1;
                    unsigned long long bit = 0;
#pragma unroll
                    for (int w = 3; w >= 0; --w) {
                        const unsigned long long h = s[w] & fr[w];
                        if (h) {
                            at = conflict_pos<4>(w, __builtin_ctzll(h), qs);
                            bit = h & (0ull - h);
                            aw = w;
                        }
                    }
                    unsigned long long b = 0;
                    bool fails = false;
                    const unsigned long long fo = w4 == 0 ? f[0] : w4 == 1 ? f[1] : w4 == 2 ? f[2] : f[3];
                    const bool meets = ((fo >> lane) & 1ull) && aw >= 0;
                    if (meets) {
                        const float4 p = sh.lq[at];
                        const float d = key_d2(k0);
                        const float t = min_dist(d, sqdist(q.x, q.y, q.z, p.x, p.y, p.z), euclid);
                        const bool real = t < d && sh.lkey[at] > k0;
                        fails = real && !ties;
#pragma unroll
                        for (int w = 0; w < 4; ++w)
                            s[w] &= (!real && aw == w) ? ~bit : ~0ull;
                        const unsigned long long kt = ((unsigned long long)__float_as_uint(t) << 32) | (uint32_t)k0;
                        const unsigned long long ku = ((unsigned long long)__float_as_uint(q.w) << 32) | 0xffffffffull;
                        const unsigned long long kb = umax64(kt, ku < k0 ? ku : k0 - 1ull);
                        b = fails ? kb : 0ull;
                    }
                    const unsigned long long om = ballot64(fails), met = ballot64(meets);
                    int mat;
                    b = wave_max_key(b, mat);
                    if (lane == 0) {
                        sh.wo[wave] = om;
                        sh.wmet[wave] = met ? 1u : 0u;
                        if (b)
                            atomicMax(&sh.wscur, b);
                    }
                }
                __syncthreads();
                scur = umax64(scur, sh.wscur);
                ties = (sh.wmet[0] | sh.wmet[1] | sh.wmet[2] | sh.wmet[3]) == 0u;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const unsigned long long om = lane_u64(sh.wo[w], 0);
                    nfail += (uint32_t)__popcll(om);
                    lv[w] &= ~om & ballot64(key[w] > scur);
                }
                __syncthreads();
            }
            if (clocks) {
                const unsigned long long t = wall_clock64();
                tl.walk += t - t_sub;
                t_sub = t;
            }
            // the picks, in any order, for the apply phase and the outputs
            uint32_t n = 0, base = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                base += w < w4 ? (uint32_t)__popcll(lv[w]) : 0u;
                n += (uint32_t)__popcll(lv[w]);
            }
            if (wave < 4) {
                const unsigned long long lo = w4 == 0 ? lv[0] : w4 == 1 ? lv[1] : w4 == 2 ? lv[2] : lv[3];
                const uint32_t pos = base + (uint32_t)__popcll(lo & below);
                if ((lo >> lane) & 1ull) {
                    sh.pk[pos] = q;
                    sh.pk[kList + pos] = sh.lb[own];
                    sh.pkey[pos] = k0;
                }
                if (wave == 0 && lane < kBlk && n + lane < (n + kBlk - 1) / kBlk * kBlk)
                    sh.pk[kList + n + lane] = make_float4(0.0f, 0.0f, 0.0f, INFINITY);
                if (tid == 0)
                    sh.npick = n;
                if (clocks)
                    tl.fails += nfail;
            }
        }
        if (clocks)
            tl.picks += wall_clock64() - t_sub;
        __syncthreads();
        const int PN = (int)sh.npick;  // picks certified; the last round may need fewer
        const int P = min(PN, job.m - j);
        if (P == 0) {
            // impossible by construction (the largest key is always free);
            // kept as a guard so a violated invariant cannot spin forever
            if (tid == 0)
                set_status(&a.hdr->sample_status, RFPS_ERR_INTERNAL);
            return false;
        }
        if (trace && round - 1 < (uint32_t)kTraceCap) {
            a.trace[2 * (size_t)(round - 1)] = t_pub;
            a.trace[2 * (size_t)(round - 1) + 1] = wall_clock64() | ((unsigned long long)P << 48);
        }
        if (clocks) {
            const unsigned long long t = wall_clock64();
            tl.ph[2] += t - t_mark;
            t_mark = t;
        }
        j_out = j;
        n_out = P;
        p_out = PN;
        j += P;
        if (j >= job.m)
            break;

        // =============== A: apply the round's picks to the true state ===============
        // Every wavefront takes its own tiles, so that its next lookahead
        // needs no barrier.  The matrix cores test blocks of 16 tiles by 16
        // picks (filter_row of the pruning threshold); a tile some pick
        // passes is updated with the picks of the block (the minimum over
        // picks does not depend on their order) and re-keyed.
        {
            const float osh = lg == 0 ? job.ox : lg == 1 ? job.oy : job.oz;
            const float *sf = reinterpret_cast<const float *>(tsph);
            const float *bf = reinterpret_cast<const float *>(sh.pk + kList);
            const int npb = (P + kBlk - 1) / kBlk;
            for (int rb = 0; rb < ntw; rb += kBlk) {
                const float av = sf[(wb + rb + li) * 4 + lg];
                const float av2 = lg == 3 ? 1.0f : -2.0f * (av - osh);
                const float4 t4 = *reinterpret_cast<const float4 *>(&trow[wb + rb + 4 * lg]);
                if (tele && lane == 0)
                    tl.tests += (unsigned long long)P * (unsigned long long)min(kBlk, ntw - rb);
                for (int cb = 0; cb < npb; ++cb) {
                    const float bv = bf[(cb * kBlk + li) * 4 + lg];
                    const f32x4 dd =
                        __builtin_amdgcn_mfma_f32_16x16x4f32(av2, bv, f32x4{t4.x, t4.y, t4.z, t4.w}, 0, 0, 0);
                    unsigned long long mr[4] = {ballot64(!(dd[0] >= 0.0f)), ballot64(!(dd[1] >= 0.0f)),
                                                ballot64(!(dd[2] >= 0.0f)), ballot64(!(dd[3] >= 0.0f))};
                    // (a tile that is never skipped passes the padding too)
                    const unsigned long long cols = ballot64(cb * kBlk + li < P);
                    if (tele) {
                        int kept = 0;
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            kept += __popcll(mr[r] & cols & ballot64(rb + 4 * lg + r < ntw));
                        if (lane == 0)
                            tl.pruned += (unsigned long long)(min(kBlk, P - cb * kBlk) * min(kBlk, ntw - rb) - kept);
                    }
                    if (!(mr[0] | mr[1] | mr[2] | mr[3]))
                        continue;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        unsigned long long m = mr[r] & cols;
                        while (m) {
                            const int g = __builtin_ctzll(m) >> 4;
                            uint32_t f = (uint32_t)(m >> (16 * g)) & 0xffffu;
                            m &= ~(0xffffull << (16 * g));
                            const int s = wb + rb + 4 * g + r;
                            const uint32_t meta = uniform_u32(tmeta[s]);
                            const uint32_t ls = meta & 0xffffu, cnt = meta >> 16;
                            const bool valid = (uint32_t)lane < cnt;
                            const uint32_t pp = ls + (valid ? lane : 0);
                            const float4 q = pq[pp];
                            float d = pd[pp];
                            const float d0 = d;
                            const unsigned long long t_upd = clocks ? wall_clock64() : 0ull;
                            if (clocks)
                                tl.apairs += (unsigned long long)__popc(f);
                            if (tele && lane == 0)
                                tl.visited += (unsigned long long)__popc(f) * cnt;
                            // (the class top of the smallest distance is the
                            // smallest class top)
                            float least = INFINITY;
                            while (f) {
                                const int kk = cb * kBlk + __builtin_ctz(f);
                                f &= f - 1;
                                const float4 s4 = sh.pk[kk];
                                if (tele && count_skip && valid) {
                                    const float dx = q.x - s4.x, dy = q.y - s4.y, dz = q.z - s4.z;
                                    const float dn = fminf(d, least);
                                    tl.skipped += (dx * dx >= dn || dy * dy >= dn || dz * dz >= dn) ? 1 : 0;
                                }
                                least = fminf(least, sqdist(q.x, q.y, q.z, s4.x, s4.y, s4.z));
                            }
                            d = min_dist(d, least, euclid);
                            const bool changed = valid && d < d0;
                            const unsigned long long um = ballot64(changed);
                            if (tele && lane == 0) {
                                tl.updated += (unsigned long long)__popcll(um);
                                tl.resync += um != 0;
                            }
                            if (um) {
                                if (changed)
                                    pd[pp] = d;
                                rekey(s, valid, d, __float_as_uint(q.w));
                                if (clocks)
                                    ++tl.arekeys;
                            }
                            if (clocks)
                                tl.update += wall_clock64() - t_upd;
                        }
                    }
                }
            }
        }
        if (clocks) {
            const unsigned long long t = wall_clock64();
            tl.ph[3] += t - t_mark;
        }
    }
    if (rank == 0 && n_out) {
        __syncthreads();
        rank_out();
        __syncthreads();
        if (wave == 0)
            write_out(lane);
    }
    tl.rounds += round;
    __syncthreads();  // LDS is reused by the next cloud
    return true;
}

// Adds the per-thread telemetry of a workgroup to the header counters.
__device__ __forceinline__ void flush_telemetry(IndexHeader *hdr, const RoundTele &tl, bool clocks)
{
    const int lane = threadIdx.x & (kWave - 1);
    const unsigned long long v[6] = {tl.tests, tl.pruned, tl.visited, tl.skipped, tl.updated, tl.resync};
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        unsigned long long s = v[q];
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1)
            s += __shfl_xor(s, o, kWave);
        if (lane == 0 && s)
            atomicAdd(&hdr->tele[2 + q], s);
    }
    if (clocks) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            atomicAdd(&hdr->tele[kTeleTicksLookahead + q], tl.ph[q]);
        atomicAdd(&hdr->tele[kTeleTicksWait], tl.ph[4]);
        // (the fields between, of phases the sampler no longer has, stay 0)
        const int at[7] = {0, 1, 2, 3, 5, 6, 7};
        const unsigned long long fine[7] = {tl.list, tl.conflicts, tl.walk, tl.picks, tl.later, tl.poll, tl.rest - tl.poll};
#pragma unroll
        for (int q = 0; q < 7; ++q)
            atomicAdd(&hdr->tele[kTeleSub + at[q]], fine[q]);
        atomicAdd(&hdr->tele[kTeleMergeStats + 0], tl.above);
        atomicAdd(&hdr->tele[kTeleMergeStats + 1], tl.listed);
        atomicAdd(&hdr->tele[kTeleMergeStats + 2], tl.fails);
        atomicAdd(&hdr->tele[kTeleMergeStats + 3], tl.ph[3]);
        atomicAdd(&hdr->tele[kTeleMergeStats + 5], tl.update);
        atomicAdd(&hdr->tele[kTeleMergeStats + 6], tl.apairs);
        atomicAdd(&hdr->tele[kTeleMergeStats + 7], tl.arekeys);
    }
}

// ---------------------------------------------------------------------------
// Single cloud: one team made of the whole grid, agent-scope exchange.
// ---------------------------------------------------------------------------
template <int NU, bool E, bool T>
__device__ __forceinline__ void rounds_single(const RoundArgs &a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ RoundShared sh;
    __shared__ uint32_t s_status;
    const int tid = threadIdx.x;
    IndexHeader *hdr = a.hdr;
    if (tid == 0)
        s_status = hdr->build_status | hdr->sample_status;
    __syncthreads();
    const int G = hdr->team_g, K = hdr->team_k, steps = hdr->team_steps;
    if (s_status || (int)blockIdx.x >= G)
        return;
    const bool timed = T && (a.flags & (RFPS_F_TELEMETRY | RFPS_F_CLOCKS)) != 0;
    const bool clocks = timed && blockIdx.x == 0 && tid == 0;
    CloudJob job;
    job.tb = 0;
    job.te = hdr->n_tiles;
    job.point_base = 0;
    job.m = a.m;
    job.start = a.start;
    job.out_idx = a.out_idx;
    job.out_d2 = a.out_d2;
    job.ox = (float)hdr->origin[0];
    job.oy = (float)hdr->origin[1];
    job.oz = (float)hdr->origin[2];
    uint32_t epoch = 0;
    RoundTele tl;
    const bool trace = (a.flags & RFPS_F_TRACE) != 0 && blockIdx.x == 0;
    const uint32_t words = slot_units((uint32_t)K) * kUnit;
    const Board board = {a.board, words, (uint32_t)G * words};
    bool ok;
    if (NU == 2 && G * (int)slot_units((uint32_t)K) <= kRBlock)
        ok = sample_cloud<Scope::Agent, 1, E, T>(a, job, blockIdx.x, G, K, steps, board, epoch, smem, sh, tl, trace,
                                                 clocks);
    else
        ok = sample_cloud<Scope::Agent, NU, E, T>(a, job, blockIdx.x, G, K, steps, board, epoch, smem, sh, tl, trace,
                                                  clocks);
    if (timed && ok) {
        flush_telemetry(hdr, tl, clocks);  // the counters stay 0 without RFPS_F_TELEMETRY
        if (blockIdx.x == 0 && tid == 0) {
            atomicAdd(&hdr->tele[0], (unsigned long long)(a.m > 1 ? a.m - 2 : 0));
            atomicAdd(&hdr->tele[1], (unsigned long long)hdr->n_tiles);
            atomicAdd(&hdr->tele[kTeleExchanges], tl.rounds);
            hdr->tele[kTeleTeam] = (unsigned long long)G | ((unsigned long long)K << 16);
        }
    }
    if (blockIdx.x == 0 && tid == 0)
        hdr->trace_n = (uint32_t)tl.rounds;
}

// Squared distances (the default) and Euclidean distances are separate
// kernels, and so are the instrumented ones (RFPS_F_TELEMETRY or
// RFPS_F_TRACE): the default kernel carries no code of either.  Its machine
// code is close to the instruction cache's size, and compiling the
// instrumentation out of it shortens a round measurably.
#define RFPS_ROUNDS_KERNEL(NAME, ...)                                                                         \
    __global__ __launch_bounds__(kRBlock)                                                                     \
        __attribute__((amdgpu_waves_per_eu(kRBlock / 256, kRBlock / 256))) void NAME(RoundArgs a)             \
    {                                                                                                         \
        __VA_ARGS__(a);                                                                                       \
    }
RFPS_ROUNDS_KERNEL(k_rfps_rounds, rounds_single<2, false, false>)
RFPS_ROUNDS_KERNEL(k_rfps_rounds_wide, rounds_single<5, false, false>)
RFPS_ROUNDS_KERNEL(k_rfps_rounds_euclid, rounds_single<2, true, false>)
RFPS_ROUNDS_KERNEL(k_rfps_rounds_wide_euclid, rounds_single<5, true, false>)
RFPS_ROUNDS_KERNEL(k_rfps_rounds_tele, rounds_single<2, false, true>)
RFPS_ROUNDS_KERNEL(k_rfps_rounds_wide_tele, rounds_single<5, false, true>)
RFPS_ROUNDS_KERNEL(k_rfps_rounds_euclid_tele, rounds_single<2, true, true>)
RFPS_ROUNDS_KERNEL(k_rfps_rounds_wide_euclid_tele, rounds_single<5, true, true>)


// ---------------------------------------------------------------------------
// Batches: teams of T workgroups, all on one XCD (found from the hardware
// XCC id at run time), exchange through that XCD's L2.  The plan gives every
// cloud a team size (a power of two, a level) and orders the clouds by
// decreasing size and cost; batch_teams.h says how the teams take them.
// Measured against one team of a whole XCD per cloud: 64 clouds of 512 to
// 4,096 points 2.18 -> 0.78 ms (0.52 with small clouds in one workgroup and a
// shorter build), 32 clouds of 8k to 120k points 16.1 -> 9.8 ms
// (then bound by the workgroups' time: the device is full until the end).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t xcc_id()
{
    return __builtin_amdgcn_s_getreg((20) | (0 << 6) | ((16 - 1) << 11)) & 0xffu;
}

// What a workgroup of a batch reaches of the device (see batch_teams.h).
template <bool E, bool I>
struct BatchIo {
    static constexpr uint32_t kSpins = kSpinLimit;
    const RoundArgs &a;
    const int me;  // this workgroup among all, by XCD and place in it
    unsigned char *const smem;
    RoundShared &sh;
    uint32_t &s_value;
    RoundTele &tl;
    unsigned long long led;  // rounds of the clouds this workgroup led
    uint32_t epoch;

    // Control words: for every level a post, then for every level a count.  A
    // team's are those of its first workgroup.
    __device__ __forceinline__ unsigned long long *control(int word, int T)
    {
        return a.board + (size_t)kMaxGroups * kBatchSlotWords + (size_t)word * kMaxGroups + (me & ~(T - 1));
    }
    __device__ __forceinline__ uint32_t next(int lev) { return atomicAdd(&a.bstate->next[lev], 1u); }
    __device__ __forceinline__ bool wanted(uint32_t q) { return a.bc.m[a.order[q]] >= 2; }
    __device__ __forceinline__ void post(int lev, int T, unsigned long long v)
    {
        bstore<Scope::Xcd>(control(lev, T), v);
    }
    __device__ __forceinline__ unsigned long long posted(int lev, int T) { return ld_agent(control(lev, T)); }
    // (nothing is handed over: a workgroup's reads have returned before it
    // arrives, and what it stores next waits for the count)
    __device__ __forceinline__ void arrive(int lev, int T)
    {
        __hip_atomic_fetch_add(control(kBatchLevels + lev, T), 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ unsigned long long arrived(int lev, int T)
    {
        return ld_agent(control(kBatchLevels + lev, T));
    }
    __device__ __forceinline__ uint32_t first(int lev) { return a.bstate->level_first[lev]; }
    template <class F>
    __device__ __forceinline__ uint32_t one(F f)
    {
        if (threadIdx.x == 0) {
            s_value = f();
            if (s_value == kNoCloud)
                set_status(&a.hdr->sample_status, RFPS_ERR_TIMEOUT);
        }
        __syncthreads();
        const uint32_t v = s_value;
        __syncthreads();
        return v;
    }
    __device__ __forceinline__ bool sample(int lev, int T, int rank, uint32_t q)
    {
        const BatchCtl &bc = a.bc;
        const int c = a.order[q];
        if (!I && T == 1) {
            const uint32_t p = (uint32_t)bc.offsets[c];  // the cloud's place in the input and among the sorted points
            const SoloJob solo = {a.xs,
                                  a.ys,
                                  a.zs,
                                  a.inv + p,
                                  bc.offsets[c + 1] - bc.offsets[c],
                                  bc.m[c],
                                  bc.starts ? bc.starts[c] : 0,
                                  a.out_idx + bc.out_offsets[c],
                                  a.out_d2 ? a.out_d2 + bc.out_offsets[c] : nullptr};
            solo_any<E>(solo, smem);
            return true;
        }
        CloudJob job;
        job.tb = a.tile_first[c];
        job.te = a.tile_first[c + 1];
        job.point_base = (uint32_t)bc.offsets[c];
        job.m = bc.m[c];
        job.start = bc.starts ? bc.starts[c] : 0;
        job.out_idx = a.out_idx + bc.out_offsets[c];
        job.out_d2 = a.out_d2 ? a.out_d2 + bc.out_offsets[c] : nullptr;
        const uint32_t *bb = a.cl_bb + 6 * (size_t)c;
        job.ox = 0.5f * ord2f(bb[0]) + 0.5f * ord2f(bb[3]);
        job.oy = 0.5f * ord2f(bb[1]) + 0.5f * ord2f(bb[4]);
        job.oz = 0.5f * ord2f(bb[2]) + 0.5f * ord2f(bb[5]);
        // a workgroup's two slots lie side by side, so a team's slots are the
        // slots of the teams it splits into.  K never falls from a level to
        // the next (k_batch_levels): every word a team reads is rewritten at
        // every second exchange of its members, whatever team they were in.
        const Board board = {a.board + (size_t)(me - rank) * kBatchSlotWords, (uint32_t)kBatchSlotWords,
                             (uint32_t)kMaxSlotWords};
        const unsigned long long r0 = tl.rounds;
        if (!sample_cloud<Scope::Xcd, 1, E, I>(a, job, rank, T, (int)a.bstate->level_k[lev], kBatchSteps, board, epoch,
                                               smem, sh, tl, false, false))
            return false;
        led += rank == 0 ? tl.rounds - r0 : 0ull;
        return true;
    }
};

template <bool E, bool I>
__device__ __forceinline__ void rounds_batched(const RoundArgs &a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ RoundShared sh;
    __shared__ uint32_t s_status, s_xcc, s_xrank, s_value, s_ok;
    const int tid = threadIdx.x;
    IndexHeader *hdr = a.hdr;
    const BatchCtl &bc = a.bc;
    BatchState *st = a.bstate;
    if (tid == 0) {
        s_status = hdr->build_status | hdr->sample_status;
        s_ok = 0;
        if (!s_status) {
            // join the workgroups of this XCD, then wait until all have joined
            const uint32_t x = xcc_id();
            s_xcc = x;
            s_xrank = x < kMaxXcds ? atomicAdd(&st->xcd_count[x], 1u) : 0xffffffffu;
            // release / acquire: a workgroup that sees every join also sees
            // every XCD count bumped before it
            __hip_atomic_fetch_add(&st->joined, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            uint32_t spin = 0;
            while (__hip_atomic_load(&st->joined, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < gridDim.x &&
                   ++spin < kSpinLimit) {
            }
            if (spin >= kSpinLimit || x >= kMaxXcds) {
                set_status(&hdr->sample_status, RFPS_ERR_TIMEOUT);
            } else if (__hip_atomic_load(&st->xcd_count[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) !=
                       (uint32_t)bc.per_xcd) {
                // the teams assume per_xcd workgroups on every XCD
                set_status(&hdr->sample_status, RFPS_ERR_UNSUPPORTED);
            } else {
                s_ok = 1;
            }
        }
    }
    __syncthreads();
    if (s_status || !s_ok)
        return;
    RoundTele tl;
    BatchIo<E, I> io = {a, (int)s_xcc * bc.per_xcd + (int)s_xrank, smem, sh, s_value, tl, 0ull, 0u};
    if (!walk_levels(io, bc.per_xcd, (int)s_xrank))
        return;
    if (I && (a.flags & RFPS_F_TELEMETRY) != 0) {
        flush_telemetry(hdr, tl, false);
        if (tid == 0)
            atomicAdd(&hdr->tele[kTeleExchanges], io.led);
    }
}

RFPS_ROUNDS_KERNEL(k_rfps_rounds_batched, rounds_batched<false, false>)
RFPS_ROUNDS_KERNEL(k_rfps_rounds_batched_euclid, rounds_batched<true, false>)
RFPS_ROUNDS_KERNEL(k_rfps_rounds_batched_tele, rounds_batched<false, true>)
RFPS_ROUNDS_KERNEL(k_rfps_rounds_batched_euclid_tele, rounds_batched<true, true>)
#undef RFPS_ROUNDS_KERNEL

// ---------------------------------------------------------------------------
// Exchange floor: G workgroups run `rounds` exchanges with nothing else in a
// round.  Each publishes W epoch-tagged words and reads every word of every
// slot until all carry the epoch, with agent-scope stores and loads as the
// sampler's exchange between XCDs.  Workgroup 0 records the
// wall-clock ticks of the whole loop in out[0]; an expired wait records
// RFPS_ERR_TIMEOUT in *status and ends the workgroup.  The launcher clears
// the slots and out[0..1] first.
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_exchange_clear(unsigned long long *board, int words,
                                                           unsigned long long *out)
{
    const int t0 = blockIdx.x * blockDim.x + threadIdx.x;
    for (int w = t0; w < words; w += gridDim.x * blockDim.x)
        board[w] = 0ull;
    if (t0 < 2)
        out[t0] = 0ull;
}

// NW: words per thread (G * W <= kBlock * NW), all of a thread's words in
// flight at once
template <int NW>
__global__ __launch_bounds__(kBlock) void k_exchange_probe(unsigned long long *board, int G, int W, int rounds,
                                                           unsigned long long *out, uint32_t *status)
{
    const int tid = threadIdx.x, rank = blockIdx.x;
    const int total = G * W;
    __shared__ uint32_t s_abort;
    if (tid == 0)
        s_abort = 0;
    __syncthreads();
    const unsigned long long t0 = wall_clock64();
    for (uint32_t epoch = 1; epoch <= (uint32_t)rounds; ++epoch) {
        unsigned long long *sbase = board + (size_t)(epoch & 1u) * G * kMaxSlotWords;
        if (tid < W)
            bstore<Scope::Agent>(sbase + (size_t)rank * kMaxSlotWords + tid,
                                 ((unsigned long long)epoch << 32) | (uint32_t)(rank * W + tid));
        unsigned long long pend = 0;
#pragma unroll
        for (int r = 0; r < NW; ++r)
            pend |= (tid + kBlock * r < total) ? (1ull << r) : 0ull;
        for (uint32_t spin = 0; pend && spin < kSpinLimit; ++spin) {
            unsigned long long x[NW];
#pragma unroll
            for (int r = 0; r < NW; ++r) {
                const int e = tid + kBlock * r;
                x[r] = ((pend >> r) & 1ull) ? ld_agent(sbase + (size_t)(e / W) * kMaxSlotWords + e % W)
                                            : 0ull;
            }
#pragma unroll
            for (int r = 0; r < NW; ++r)
                if (((pend >> r) & 1ull) && (uint32_t)(x[r] >> 32) == epoch)
                    pend &= ~(1ull << r);
        }
        if (pend)
            s_abort = 1;
        __syncthreads();
        if (s_abort) {
            if (tid == 0)
                set_status(status, RFPS_ERR_TIMEOUT);
            return;
        }
    }
    if (rank == 0 && tid == 0)
        out[0] = wall_clock64() - t0;
}

hipError_t launch_exchange_probe(unsigned long long *board, int G, int W, int rounds, unsigned long long *out,
                                 uint32_t *status, hipStream_t s)
{
    if (G < 1 || G > kMaxGroups || W < 1 || W > kMaxSlotWords || 2 * G * kMaxSlotWords > kBoardWords || rounds < 1)
        return hipErrorInvalidValue;
    const int per = (G * W + kBlock - 1) / kBlock;  // words per thread
    k_exchange_clear<<<64, kBlock, 0, s>>>(board, 2 * G * kMaxSlotWords, out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    void *args[] = {&board, &G, &W, &rounds, &out, &status};
    // unused dynamic LDS of more than half a compute unit's keeps one
    // workgroup per compute unit, as in the sampler
    const void *fn = per <= 2    ? reinterpret_cast<const void *>(k_exchange_probe<2>)
                     : per <= 16 ? reinterpret_cast<const void *>(k_exchange_probe<16>)
                     : per <= 32 ? reinterpret_cast<const void *>(k_exchange_probe<32>)
                                 : reinterpret_cast<const void *>(k_exchange_probe<64>);
    constexpr int kOnePerCu = 96 * 1024;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kOnePerCu);
    if (e != hipSuccess)
        return e;
    return launch_persistent(fn, G, args, kOnePerCu, s);
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
static const void *rounds_fn(const SampleLaunch &L, bool batched, bool wide_slots)
{
    const int e = (L.flags & RFPS_F_SQRT) != 0, t = (L.flags & (RFPS_F_TELEMETRY | RFPS_F_TRACE | RFPS_F_CLOCKS)) != 0;
#define RFPS_FN(K) reinterpret_cast<const void *>(K)
    static const void *const one[2][2] = {{RFPS_FN(k_rfps_rounds), RFPS_FN(k_rfps_rounds_tele)},
                                          {RFPS_FN(k_rfps_rounds_euclid), RFPS_FN(k_rfps_rounds_euclid_tele)}};
    static const void *const wide[2][2] = {{RFPS_FN(k_rfps_rounds_wide), RFPS_FN(k_rfps_rounds_wide_tele)},
                                           {RFPS_FN(k_rfps_rounds_wide_euclid), RFPS_FN(k_rfps_rounds_wide_euclid_tele)}};
    static const void *const many[2][2] = {
        {RFPS_FN(k_rfps_rounds_batched), RFPS_FN(k_rfps_rounds_batched_tele)},
        {RFPS_FN(k_rfps_rounds_batched_euclid), RFPS_FN(k_rfps_rounds_batched_euclid_tele)}};
#undef RFPS_FN
    if (batched)
        return many[e][t];
    return wide_slots ? wide[e][t] : one[e][t];
}

static RoundArgs round_args(const IndexView &v, int m, int start, const SampleLaunch &L, int32_t *out_idx,
                            float *out_d2)
{
    RoundArgs a;
    a.hdr = v.hdr;
    a.xs = v.xs;
    a.ys = v.ys;
    a.zs = v.zs;
    a.orig = v.orig;
    a.inv = v.inv;
    a.tstart = v.tstart;
    a.tcnt = v.tcnt;
    a.tcx = v.tcx;
    a.tcy = v.tcy;
    a.tcz = v.tcz;
    a.trad = v.trad;
    a.board = v.board;
    a.trace = v.trace;
    a.out_idx = out_idx;
    a.out_d2 = out_d2;
    a.n = v.n;
    a.m = m;
    a.start = start;
    a.flags = L.flags;
    a.lds_budget = 0;
    a.cl_bb = nullptr;
    a.bc = BatchCtl{};
    a.bstate = nullptr;
    a.tile_first = nullptr;
    a.order = nullptr;
    return a;
}

hipError_t launch_rfps_rounds(const IndexView &v, int m, int start, const SampleLaunch &L, int32_t *out_idx,
                              float *out_d2, hipStream_t s)
{
    RoundArgs a = round_args(v, m, start, L, out_idx, out_d2);
    a.lds_budget = rounds_dynamic((uint32_t)L.max_lds);
    // at most K + 1 units of a slot from every workgroup the launch may use
    const int most = L.G * (int)slot_units((uint32_t)(L.K ? L.K : 3));
    if (!a.lds_budget || L.K > kRWaves || most > 5 * kRBlock)
        return hipErrorInvalidValue;
    k_rounds_plan<<<5, kPlanBlock, 0, s>>>(v.hdr, v.tcnt, v.board, m, start, out_idx, out_d2, L.G, L.Gcap, L.fixed_g ? L.G : 0, L.K, L.R,
                                           L.lds_budget, a.lds_budget);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || m <= 1)
        return e;
    const void *fn = rounds_fn(L, false, most > 2 * kRBlock);
    void *args[] = {&a};
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)a.lds_budget);
    if (e != hipSuccess)
        return e;
    return launch_persistent(fn, L.G, args, a.lds_budget, s, kRBlock);
}

// Batched plan, one workgroup per cloud: finds the cloud's tiles, checks the cloud's capacity for a
// team of bc.team_size workgroups, finds the smallest team whose shares fit
// the sampler's LDS (bc.team_size itself when the caller asked for it), and
// writes the cloud's first output (its start, at distance +inf).  The counters
// the sampler does not keep are set by the first workgroup.
constexpr int kBatchPlanBlock = 256;
static_assert(kMaxGroups * (kBatchSlotWords + 2 * kBatchLevels) <= kBoardWords, "a batch's slots and control words");
static_assert(kBatchSlotWords == 2 * kMaxSlotWords && (kBatchK + 1) * kUnit <= kMaxSlotWords, "a slot's units");
__global__ __launch_bounds__(kBatchPlanBlock) void k_batch_plan(IndexHeader *hdr, const uint32_t *__restrict__ tstart,
                                                                const uint32_t *__restrict__ tcnt, BatchCtl bc,
                                                                uint32_t *__restrict__ tile_first,
                                                                int R, uint32_t budget, uint32_t lds, bool solo,
                                                                uint32_t *cl_team,
                                                                int32_t *out_idx, float *out_d2)
{
    // tiles and points by tile number modulo the largest team: a smaller
    // team's shares are sums of them
    __shared__ uint32_t s_tiles[kMaxGroups], s_pts[kMaxGroups], s_big[kBatchLevels], s_tile[2];
    if (hdr->build_status)
        return;
    const int tid = threadIdx.x, c = blockIdx.x, X = bc.per_xcd, T = bc.team_size;
    if (tid < 2 * kWave) {
        // The cloud's tiles: the sorted points of a cloud are its range of the
        // input, so its first tile starts there (64 probes a step).
        const int lane = tid & (kWave - 1), w = tid / kWave;
        const uint32_t p = (uint32_t)bc.offsets[c + w];
        uint32_t lo = 0, hi = hdr->n_tiles;  // the first tile that starts at p or later
        while (lo < hi) {
            const uint32_t step = (hi - lo + kWave - 1) / kWave, q = lo + lane * step;
            const uint32_t f = (uint32_t)__popcll(ballot64(q < hi && tstart[q < hi ? q : lo] < p));
            const uint32_t nlo = f ? lo + (f - 1) * step + 1 : lo;
            hi = min(lo + f * step, hi);
            lo = nlo;
        }
        if (lane == 0) {
            s_tile[w] = lo;
            tile_first[c + w] = lo;  // (twice, the same)
        }
    }
    s_tiles[tid] = s_pts[tid] = 0u;
    if (tid < kBatchLevels)
        s_big[tid] = 0u;
    __syncthreads();
    const uint32_t tb = s_tile[0], te = s_tile[1];
    for (uint32_t t = tb + tid; t < te; t += kBatchPlanBlock) {
        atomicAdd(&s_tiles[(t - tb) % (uint32_t)X], 1u);
        atomicAdd(&s_pts[(t - tb) % (uint32_t)X], tcnt[t]);
    }
    __syncthreads();
    for (int lev = 0; lev < kBatchLevels && (X >> lev) > 0; ++lev) {
        const int t = X >> lev;
        if (tid >= t)
            continue;
        uint32_t tiles = 0, pts = 0;
        for (int r = tid; r < X; r += t) {
            tiles += s_tiles[r];
            pts += s_pts[r];
        }
        if (t == T && !share_granted(tiles, pts, T, R, budget))
            set_status(&hdr->sample_status, RFPS_ERR_CAPACITY);
        if (solo && t == 1 ? pts > (uint32_t)kSoloPoints : pts > 65535u || rounds_lds_need(tiles, pts) > lds)
            s_big[lev] = 1u;
    }
    __syncthreads();
    if (tid == 0) {
        int lev = 0;
        if (bc.fixed_team)
            while ((X >> lev) > T)
                ++lev;
        else
            for (int q = 1; q < kBatchLevels && (X >> q) > 0; ++q)
                lev = s_big[q] ? lev : q;
        cl_team[c] = (uint32_t)lev;
        const uint32_t o = bc.out_offsets[c];
        out_idx[o] = bc.starts ? bc.starts[c] : 0;
        if (out_d2)
            out_d2[o] = INFINITY;
        if (c == 0)
            hdr->tele[1] = hdr->n_tiles;
        if (bc.m[c] > 2)
            atomicAdd(&hdr->tele[0], (unsigned long long)(bc.m[c] - 2));
    }
}

// Team sizes and order of the clouds.  A smaller team spends less of the
// device on a cloud (a workgroup's lookahead and merge are the same for any
// share), so with more clouds than the device holds at once every cloud keeps
// its smallest team; otherwise the teams grow, the costliest clouds' first,
// until the device is full.  The clouds are then ordered by team, and inside
// a level by decreasing cost N_c m_c (ties by index).
//
// A cloud of up to kSoloPoints points is sampled by one workgroup in registers
// (solo_cloud.h).  Up to 4,096 points no team is faster; beyond, teams of two
// and four are not (8,192 -> 2,048: one workgroup 1.4 ms, teams of 2, 4, 8,
// 16: 2.0, 1.5, 1.2, 0.95).
//
// Measured, sampling time per cloud with the device full (room, 16,384 ->
// 4,096): teams of 4 52 us, 8 65, 16 96, 32 172; and latency of one cloud
// (4,096 -> 1,024): teams of 2 1.3 ms, 4 0.94, 8 0.76, 16 0.67, 32 0.62.
constexpr int kSoloBatch = 4096;
constexpr int kBatchOrderBlock = 1024;
__global__ __launch_bounds__(kBatchOrderBlock) void k_batch_levels(IndexHeader *hdr, BatchCtl bc, BatchState *st,
                                                                   const uint32_t *__restrict__ cl_team, int K,
                                                                   bool solo, int32_t *order)
{
    __shared__ unsigned long long s_key[kMaxBatch];
    __shared__ uint32_t s_sum, s_cnt[kBatchLevels];
    __shared__ unsigned long long s_pts;  // points of the largest level's clouds
    if (hdr->build_status)
        return;
    const int tid = threadIdx.x, B = bc.batch, X = bc.per_xcd;
    const uint32_t all = (uint32_t)(X * kMaxXcds);
    auto cost = [&](int c) {
        return (unsigned long long)(bc.offsets[c + 1] - bc.offsets[c]) * (unsigned long long)bc.m[c];
    };
    // level of a cloud whose smallest team is `least` and whose cost has the
    // logarithm f, teams holding 2^(e / 8) of cost per workgroup
    const int top = 31 - __builtin_clz((uint32_t)X);  // log2 of the largest team
    auto level_at = [&](uint32_t least, int n, float f, int e) {
        const int lev = max(0, min((int)least, top - (int)floorf(f - 0.125f * (float)e)));
        return solo && (int)least == top && (n <= kSoloBatch || lev > top - 3) ? top : lev;
    };
    auto points = [&](int c) { return bc.offsets[c + 1] - bc.offsets[c]; };
    int e = 8 * 64;
    if (!bc.fixed_team && B <= (int)all) {
        // the smallest such cost that leaves a place for every team, found by
        // the first wavefront
        if (tid < kWave) {
            constexpr int per = kMaxGroups / kWave;
            uint32_t least[per];
            int pts[per];
            float f[per];
#pragma unroll
            for (int q = 0; q < per; ++q) {
                const int c = q * kWave + tid;
                least[q] = c < B ? cl_team[c] : 0u;
                pts[q] = c < B ? points(c) : 0;
                f[q] = c < B ? log2f((float)cost(c)) : 0.0f;
            }
            int lo = 0, hi = e;  // hi: every cloud keeps its smallest team
            while (lo < hi) {
                const int mid = (lo + hi) / 2;
                uint32_t sum = 0;
#pragma unroll
                for (int q = 0; q < per; ++q)
                    sum += q * kWave + tid < B ? (uint32_t)(X >> level_at(least[q], pts[q], f[q], mid)) : 0u;
#pragma unroll
                for (int o = kWave / 2; o > 0; o >>= 1)
                    sum += (uint32_t)__shfl_xor((int)sum, o, kWave);
                if (sum <= all)
                    hi = mid;
                else
                    lo = mid + 1;
            }
            if (tid == 0)
                s_sum = (uint32_t)hi;
        }
        __syncthreads();
        e = (int)s_sum;
    }
    if (tid < kBatchLevels)
        s_cnt[tid] = 0u;
    if (tid == 0)
        s_pts = 0ull;
    __syncthreads();
    for (int c = tid; c < B; c += kBatchOrderBlock) {
        const unsigned long long v = cost(c);
        const int lev = level_at(cl_team[c], points(c), log2f((float)v), e);
        s_key[c] = ((unsigned long long)(kBatchLevels - lev) << 56) | v;
        atomicAdd(&s_cnt[lev], 1u);
        if (lev == 0)
            atomicAdd(&s_pts, (unsigned long long)(bc.offsets[c + 1] - bc.offsets[c]));
    }
    __syncthreads();
    for (int c = tid; c < B; c += kBatchOrderBlock) {
        const unsigned long long k = s_key[c];
        int rank = 0;
        for (int d = 0; d < B; ++d)
            rank += (s_key[d] > k) || (s_key[d] == k && d < c);
        order[rank] = c;
    }
    if (tid == 0) {
        uint32_t at = 0;
        for (int lev = 0; lev < kBatchLevels; ++lev) {
            st->level_first[lev] = at;
            at += s_cnt[lev];
            const unsigned long long groups = lev ? 1ull : (unsigned long long)max(s_cnt[0], 1u) * (unsigned)X;
            st->level_k[lev] = (uint32_t)(K ? K : batch_k(lev, s_pts / groups));
        }
        st->level_first[kBatchLevels] = at;
    }
}

hipError_t launch_rfps_rounds_batched(const IndexView &v, const SampleLaunch &L, int32_t *out_idx,
                                      float *out_d2, hipStream_t s)
{
    const uint32_t lds = rounds_dynamic((uint32_t)L.max_lds);
    if (!lds || L.K > kBatchK || v.bc.per_xcd * kMaxXcds > kMaxGroups || v.bc.per_xcd >> (kBatchLevels - 1) > 1)
        return hipErrorInvalidValue;
    // (the counters of the instrumented kernel are the team sampler's)
    const bool solo = (L.flags & RFPS_F_TELEMETRY) == 0 && solo_lds(kSoloPoints) <= lds;
    k_batch_plan<<<v.bc.batch, kBatchPlanBlock, 0, s>>>(v.hdr, v.tstart, v.tcnt, v.bc, v.tile_first, L.R, L.lds_budget, lds, solo,
                                                        v.cl_team, out_idx, out_d2);
    k_batch_levels<<<1, kBatchOrderBlock, 0, s>>>(v.hdr, v.bc, v.bstate, v.cl_team, L.K, solo, v.order);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    const void *fn = rounds_fn(L, true, false);
    RoundArgs a = round_args(v, 0, 0, L, out_idx, out_d2);
    a.bc = v.bc;
    a.bstate = v.bstate;
    a.tile_first = v.tile_first;
    a.order = v.order;
    a.cl_bb = v.cl_bb;
    a.lds_budget = lds;
    void *args[] = {&a};
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)a.lds_budget);
    if (e != hipSuccess)
        return e;
    e = launch_persistent(fn, L.G, args, a.lds_budget, s, kRBlock);
    if (e != hipSuccess)
        return e;
    return launch_sample_finalize(v.hdr, v.bc.m_total, out_idx, out_d2, s);
}

}  // namespace rfps
