// Spherical-voxel index builder (Sec. 3.2; the GPU steps of Algorithm 2):
// bounding box, voxel size L (eq. voxel_size), clamped voxel id
// V_id = v_z n^2 + v_y n + v_x, stable LSD radix sort of (V_id, original
// index), gather to structure-of-arrays coordinates, split of the active
// voxels into tiles of at most T points and an enclosing sphere per tile.
//
// All kernels are launched by rfps_api.hip on the caller's stream; counts
// that only the device knows (K voxels, NT tiles) stay in the index header.
//
// What bounds a build is its launches: below half a million points every
// kernel runs for 2 to 8 us, as long as a launch takes to follow another.  So
// every kernel does what it can with what the one before left in memory: the
// keys come with the histogram of the first digit, a scatter sums the
// histograms of the blocks before it instead of waiting for a scan, and two
// kernels turn the sorted keys into tiles.  Two digits take 7 launches (25
// before), and up to 4,096 points take 2.  Measured from call to completion:
// 1,024 points 113 -> 38 us, 80,000 140 -> 68, 1,048,576 353 -> 178.
#include <algorithm>
#include <utility>

#include "rfps_internal.h"

namespace rfps {

// Exclusive prefix sum over a workgroup of BLOCK threads.
template <int BLOCK = kBlock>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *wsum /*[BLOCK / kWave]*/,
                                                         uint32_t &total)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        uint32_t o = __shfl_up(incl, off, kWave);
        if (lane >= off)
            incl += o;
    }
    if (lane == kWave - 1)
        wsum[w] = incl;
    __syncthreads();
    uint32_t woff = 0;
    total = 0;
#pragma unroll
    for (int q = 0; q < BLOCK / kWave; ++q) {
        woff += q < w ? wsum[q] : 0u;
        total += wsum[q];
    }
    __syncthreads();
    return woff + incl - v;
}

// Largest and smallest coordinates and a flag over a workgroup; every thread
// gets them.
struct Box {
    float mn[3], mx[3];
    bool bad;
};
template <int BLOCK>
__device__ __forceinline__ Box block_box(Box v, float (*s)[8] /*[BLOCK / kWave][8]*/)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const bool bad = __any(v.bad);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        v.mn[a] = wave_min_f32(v.mn[a]);
        v.mx[a] = wave_max_f32(v.mx[a]);
    }
    if (lane == 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            s[w][a] = v.mn[a];
            s[w][3 + a] = v.mx[a];
        }
        s[w][6] = bad ? 1.0f : 0.0f;
    }
    __syncthreads();
    float any = 0.0f;
#pragma unroll
    for (int q = 0; q < BLOCK / kWave; ++q) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            v.mn[a] = fminf(v.mn[a], s[q][a]);
            v.mx[a] = fmaxf(v.mx[a], s[q][3 + a]);
        }
        any = fmaxf(any, s[q][6]);
    }
    v.bad = any != 0.0f;
    return v;
}

// Bounding box of the cloud, one part per workgroup (eight floats: lower and
// upper corner, whether a coordinate is not finite).  At most kBoxParts, so
// that a thread of the next kernel reads one.
constexpr int kBoxParts = kBlock;
__global__ __launch_bounds__(kBlock) void k_bbox(const float *__restrict__ xyz, int n, float *__restrict__ parts)
{
    __shared__ float s_box[kWavesPerBlock][8];
    Box b = {{INFINITY, INFINITY, INFINITY}, {-INFINITY, -INFINITY, -INFINITY}, false};
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float v = xyz[3 * (size_t)i + a];
            b.bad |= !isfinite(v);
            b.mn[a] = fminf(b.mn[a], v);
            b.mx[a] = fmaxf(b.mx[a], v);
        }
    }
    b = block_box<kBlock>(b, s_box);
    if (threadIdx.x == 0) {
        float *p = parts + 8 * (size_t)blockIdx.x;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            p[a] = b.mn[a];
            p[3 + a] = b.mx[a];
        }
        p[6] = b.bad ? 1.0f : 0.0f;
    }
}

// Where a histogram keeps the count of digit d in block b: rows of 256 digits
// (scatters that sum the blocks themselves read whole rows), or, for the
// prefix sum over all of it, rows of blocks.
__device__ __forceinline__ size_t hist_at(int d, int b, int nblk, bool rows)
{
    return rows ? (size_t)b * 256 + d : (size_t)d * nblk + b;
}

// Voxel edge L = alpha * max(E) / n_vox with alpha = 1 + 1e-4 (eq. voxel_size);
// a cloud of identical points gets L = 1 (one voxel).  The range shells (if
// any) are centred on the bounding-box centre.
struct Grid {
    double pmin[3], origin[3], L;
};
__device__ __forceinline__ Grid grid_of(const float *lo, const float *hi, bool failed, uint32_t n_vox)
{
    Grid g;
    double E = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        g.pmin[a] = (double)lo[a];
        g.origin[a] = 0.5 * ((double)lo[a] + (double)hi[a]);
        const double e = (double)hi[a] - (double)lo[a];
        E = e > E ? e : E;
    }
    const double alpha = 1.0 + 1e-4;
    // a failed build still gets a finite edge: the keys are then meaningless
    // but every index computed from them stays in range
    g.L = (E > 0.0 && E < INFINITY && !failed) ? alpha * E / (double)n_vox : 1.0;
    return g;
}
// What a build leaves in the header beside the counts (first threads of one
// workgroup).
__device__ __forceinline__ void begin_header(IndexHeader *hdr, const Box &b, const Grid &g, double shell_inv,
                                             uint32_t shell_cap)
{
    if (threadIdx.x == 0) {
        hdr->build_status = b.bad ? RFPS_ERR_NONFINITE : 0u;
        hdr->sample_status = 0;
        for (int a = 0; a < 3; ++a) {
            hdr->bb[a] = f2ord(b.mn[a]);
            hdr->bb[3 + a] = f2ord(b.mx[a]);
            hdr->pmin[a] = g.pmin[a];
            hdr->origin[a] = g.origin[a];
        }
        hdr->L = g.L;
        hdr->shell_inv = shell_inv;
        hdr->shell_cap = shell_cap;
        hdr->trace_n = 0;
    }
    if (threadIdx.x < kTeleFields)
        hdr->tele[threadIdx.x] = 0;
}

// Threads of the sort's workgroups: a radix tile of 2,048 keys on 16
// wavefronts (two keys a thread), since FP64 keys and the digit matches are
// chains of dependent operations that only more wavefronts overlap (61 tiles:
// key kernel 6 us against 12 with 256 threads, scatter 7.6 against 11).
constexpr int kSortBlock = 1024;
constexpr int kSortItems = kRadixTile / kSortBlock;
constexpr int kSortWaves = kSortBlock / kWave;

// Grid, voxel key of every point, the identity payload and the histogram of
// the first digit.  Every workgroup forms the grid from the parts of the box;
// the first one resets the header and records it.
__global__ __launch_bounds__(kSortBlock) void k_voxel_key(const float *__restrict__ xyz, int n,
                                                          const float *__restrict__ parts, int n_parts,
                                                          IndexHeader *hdr, int n_vox, double shell_inv,
                                                          uint32_t shell_cap, uint32_t *__restrict__ key,
                                                          uint32_t *__restrict__ val, uint32_t *__restrict__ hist,
                                                          int nblk, bool rows)
{
    __shared__ float s_box[kSortWaves][8];
    __shared__ uint32_t h[256];
    const int tid = threadIdx.x;
    Box b = {{INFINITY, INFINITY, INFINITY}, {-INFINITY, -INFINITY, -INFINITY}, false};
    if (tid < n_parts) {
        const float *p = parts + 8 * (size_t)tid;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            b.mn[a] = p[a];
            b.mx[a] = p[3 + a];
        }
        b.bad = p[6] != 0.0f;
    }
    if (tid < 256)
        h[tid] = 0;
    b = block_box<kSortBlock>(b, s_box);
    const Grid g = grid_of(b.mn, b.mx, b.bad, (uint32_t)n_vox);
    if (blockIdx.x == 0)
        begin_header(hdr, b, g, shell_inv, shell_cap);
    const int base = blockIdx.x * kRadixTile;
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int i = base + r * kSortBlock + tid;
        if (i < n) {
            const uint32_t k = voxel_key(xyz[3 * (size_t)i], xyz[3 * (size_t)i + 1], xyz[3 * (size_t)i + 2], g.pmin,
                                         g.L, (uint32_t)n_vox, g.origin, shell_inv, shell_cap);
            key[i] = k;
            val[i] = (uint32_t)i;
            atomicAdd(&h[k & 255u], 1u);
        }
    }
    __syncthreads();
    if (tid < 256)
        hist[hist_at(tid, blockIdx.x, nblk, rows)] = h[tid];
}

// ---------------------------------------------------------------------------
// Stable LSD radix sort, 8 bits per pass.  Tile b covers keys
// [b*kRadixTile, (b+1)*kRadixTile).  `range` (batches): the keys are below
// *range; a pass with skip set has nothing to do when they have 16 bits.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool pass_skipped(const uint32_t *range, bool skip)
{
    return skip && *range <= 65536u;
}

__global__ __launch_bounds__(kSortBlock) void k_radix_hist(const uint32_t *__restrict__ keys, int n, int shift,
                                                           uint32_t *__restrict__ hist, int nblk, bool rows,
                                                           const uint32_t *range, bool skip)
{
    __shared__ uint32_t h[256];
    const int tid = threadIdx.x;
    if (pass_skipped(range, skip))
        return;
    if (tid < 256)
        h[tid] = 0;
    __syncthreads();
    const int base = blockIdx.x * kRadixTile;
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        int i = base + r * kSortBlock + tid;
        if (i < n)
            atomicAdd(&h[(keys[i] >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (tid < 256)
        hist[hist_at(tid, blockIdx.x, nblk, rows)] = h[tid];
}

// Ranks of a workgroup's keys among its keys of the same digit, stable in the
// order wavefront, item, lane: a wavefront counts its digits as it goes, the
// rank among equal digits of one item coming from eight ballots and the
// wavefront's count so far from LDS, so the items need no barrier.  wcnt is
// cleared before; after a barrier it holds the wavefronts' counts.
template <int ITEMS>
__device__ __forceinline__ void digit_ranks(const uint32_t *key, const bool *valid, int shift, uint32_t *cnt,
                                            uint32_t *rank)
{
    const int lane = threadIdx.x & (kWave - 1);
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t d = (key[r] >> shift) & 255u;
        const unsigned long long in = __ballot(valid[r]);
        uint32_t lo = (uint32_t)in, hi = (uint32_t)(in >> 32);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const uint32_t m = (uint32_t)((int32_t)(d << (31 - bit)) >> 31);  // all ones when the bit is set
            const unsigned long long ones = __ballot(m != 0u);
            lo &= ~((uint32_t)ones ^ m);
            hi &= ~((uint32_t)(ones >> 32) ^ m);
        }
        const unsigned long long peers = ((unsigned long long)hi << 32) | lo;
        const uint32_t at = (uint32_t)__popcll(peers & below);
        const uint32_t so_far = cnt[d];
        rank[r] = so_far + at;
        // all lanes have read before one of them stores, and the next item
        // reads what was stored
        wave_sync();
        if (valid[r] && at == 0)
            cnt[d] = so_far + (uint32_t)__popcll(peers);
        wave_sync();
    }
}
// Turns the wavefronts' counts into first positions: base of the digit plus
// the counts of the wavefronts before (thread d < 256 for digit d).
template <int WAVES>
__device__ __forceinline__ void digit_bases(uint32_t (*wcnt)[256], uint32_t base)
{
    const int d = threadIdx.x;
    uint32_t c[WAVES];
#pragma unroll
    for (int q = 0; q < WAVES; ++q)
        c[q] = wcnt[q][d];
#pragma unroll
    for (int q = 0; q < WAVES; ++q) {
        wcnt[q][d] = base;
        base += c[q];
    }
}

// Scatter with a stable rank.
//
// rows: the histogram is still one row of counts per block, and the block
// sums those before it (and all, for the digits before) itself.  For up to
// kDirectBlocks blocks, whose rows it reads 32 at a time in four groups of
// threads, that takes less than the three launches of a prefix sum over all
// of them (whole build of 250,000 points, 122 blocks: 68 us against 86; of
// 1,048,576, 512 blocks: 181 against 163).
constexpr int kDirectBlocks = 256;
__global__ __launch_bounds__(kSortBlock) void k_radix_scatter(const uint32_t *__restrict__ kin,
                                                              const uint32_t *__restrict__ vin,
                                                              uint32_t *__restrict__ kout,
                                                              uint32_t *__restrict__ vout, int n, int shift,
                                                              const uint32_t *__restrict__ hist, int nblk, bool rows,
                                                              const uint32_t *range, bool skip)
{
    __shared__ uint32_t wcnt[kSortWaves][256];
    __shared__ uint32_t s_all[4][256], s_before[4][256], wsum[kSortWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    if (pass_skipped(range, skip))
        return;
    const int me = blockIdx.x;
    // this wavefront's keys, all loads in flight
    const int first = me * kRadixTile + w * (kSortItems * kWave) + lane;
    uint32_t key[kSortItems], val[kSortItems], rank[kSortItems];
    bool valid[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int i = first + r * kWave;
        valid[r] = i < n;
        key[r] = valid[r] ? kin[i] : 0u;
        val[r] = valid[r] ? vin[i] : 0u;
    }
    for (int q = tid; q < kSortWaves * 256; q += kSortBlock)
        wcnt[0][q] = 0;
    uint32_t base = 0;
    if (rows) {
        uint32_t all = 0, before = 0;
        const int g = tid / 256, d = tid % 256;
        for (int q0 = 0; q0 < nblk; q0 += 4 * 8) {
            uint32_t c[8];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                c[q] = q0 + 4 * q + g < nblk ? hist[(size_t)(q0 + 4 * q + g) * 256 + d] : 0u;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                all += c[q];
                before += q0 + 4 * q + g < me ? c[q] : 0u;
            }
        }
        s_all[g][d] = all;
        s_before[g][d] = before;
        __syncthreads();
        all = before = 0;
        if (tid < 256) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                all += s_all[q][tid];
                before += s_before[q][tid];
            }
        }
        uint32_t total;
        base = block_exclusive_scan<kSortBlock>(all, wsum, total) + before;  // ends with a barrier
    } else {
        if (tid < 256)
            base = hist[(size_t)tid * nblk + me];
        __syncthreads();
    }
    digit_ranks<kSortItems>(key, valid, shift, wcnt[w], rank);
    __syncthreads();
    if (tid < 256)
        digit_bases<kSortWaves>(wcnt, base);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        if (valid[r]) {
            const uint32_t off = wcnt[w][(key[r] >> shift) & 255u] + rank[r];
            kout[off] = key[r];
            vout[off] = val[r];
        }
    }
}

// ---------------------------------------------------------------------------
// Exclusive prefix sum of uint32 (in place allowed), three kernels.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_scan_blocks(const uint32_t *in, uint32_t *out, int n,
                                                        uint32_t *__restrict__ partials)
{
    __shared__ uint32_t wsum[kWavesPerBlock];
    const size_t base = (size_t)blockIdx.x * kScanChunk + (size_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        size_t i = base + q;
        v[q] = i < (size_t)n ? in[i] : 0u;
        s += v[q];
    }
    uint32_t total;
    uint32_t run = block_exclusive_scan(s, wsum, total);
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        size_t i = base + q;
        if (i < (size_t)n)
            out[i] = run;
        run += v[q];
    }
    if (threadIdx.x == 0)
        partials[blockIdx.x] = total;
}

// One workgroup scans the per-block totals (nb <= kBlock * 64).
__global__ __launch_bounds__(kBlock) void k_scan_partials(uint32_t *partials, int nb)
{
    __shared__ uint32_t wsum[kWavesPerBlock];
    const int per = (nb + kBlock - 1) / kBlock;
    const int b0 = threadIdx.x * per;
    uint32_t s = 0;
    for (int q = 0; q < per; ++q)
        if (b0 + q < nb)
            s += partials[b0 + q];
    uint32_t total;
    uint32_t run = block_exclusive_scan(s, wsum, total);
    for (int q = 0; q < per; ++q) {
        if (b0 + q < nb) {
            uint32_t v = partials[b0 + q];
            partials[b0 + q] = run;
            run += v;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_scan_add(uint32_t *out, int n, const uint32_t *__restrict__ partials)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        out[i] += partials[i / kScanChunk];
}

// ---------------------------------------------------------------------------
// Gather to structure of arrays, inverse permutation, tiles.
// ---------------------------------------------------------------------------

// First position of the voxel that sorted position p lies in, by all lanes of
// a wavefront, 64 probes a step.  (Unsorted keys, after a failed build, give
// some position in [0, p].)
__device__ uint32_t voxel_start(const uint32_t *__restrict__ skey, uint32_t p, int lane)
{
    const uint32_t key = skey[p];
    uint32_t lo = 0, hi = p;
    while (lo < hi) {
        const uint32_t step = (hi - lo + kWave - 1) / kWave;
        const uint32_t q = lo + lane * step;
        const uint32_t c = (uint32_t)__popcll(__ballot(q < hi && skey[q < hi ? q : p] < key));
        const uint32_t nlo = c ? lo + (c - 1) * step + 1 : lo;
        hi = min(lo + c * step, hi);
        lo = nlo;
    }
    return lo;
}

// Heads among BLOCK consecutive sorted positions from p0: whether this
// thread's position starts a voxel and whether it starts a tile, a voxel's
// positions being cut into tiles of T.  `open` is the first position of the
// voxel that p0 - 1 lies in (anything if p0 starts one) and becomes that of
// the last position.  s: [BLOCK / kWave].
template <int BLOCK>
__device__ __forceinline__ void block_heads(const uint32_t *__restrict__ skey, int n, int T, uint32_t p0,
                                            uint32_t &open, uint32_t *s, bool &voxel, bool &tile)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const uint32_t p = p0 + tid;
    const bool in = p < (uint32_t)n;
    voxel = in && (p == 0 || skey[p] != skey[p - 1]);
    const unsigned long long m = __ballot(voxel);
    __syncthreads();  // s is free
    if (lane == 0)
        s[w] = m ? p + (63 - __builtin_clzll(m)) : 0xffffffffu;
    __syncthreads();
    uint32_t mine = open;
#pragma unroll
    for (int q = 0; q < BLOCK / kWave; ++q) {
        if (q < w && s[q] != 0xffffffffu)
            mine = s[q];
        if (s[q] != 0xffffffffu)
            open = s[q];
    }
    const unsigned long long upto = m & (~0ull >> (63 - lane));
    if (upto)
        mine = p0 + w * kWave + (63 - __builtin_clzll(upto));
    tile = in && (p - mine) % (uint32_t)T == 0;
}

// Positions a workgroup of the next two kernels takes, so that there are at
// most kTileParts of them (every workgroup sums the tiles of those before it).
constexpr int kTileParts = 2048;
__host__ __device__ inline int tile_steps(int n) { return (n - 1) / (kBlock * kTileParts) + 1; }

__global__ __launch_bounds__(kBlock) void k_gather(const float *__restrict__ xyz, const uint32_t *__restrict__ orig,
                                                   const uint32_t *__restrict__ skey, int n, int T,
                                                   float *__restrict__ xs, float *__restrict__ ys,
                                                   float *__restrict__ zs, uint32_t *__restrict__ inv,
                                                   uint32_t *__restrict__ part_tiles,
                                                   uint32_t *__restrict__ part_voxels)
{
    __shared__ uint32_t s_head[kWavesPerBlock], s_open, s_tiles, s_voxels;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int steps = tile_steps(n);
    const uint32_t first = blockIdx.x * (uint32_t)(kBlock * steps);
    if (tid < kWave) {
        const uint32_t o = voxel_start(skey, first, lane);
        if (tid == 0) {
            s_open = o;
            s_tiles = s_voxels = 0u;
        }
    }
    __syncthreads();
    uint32_t open = s_open;
    for (int r = 0; r < steps; ++r) {
        const uint32_t p = first + r * kBlock + tid;
        if (p < (uint32_t)n) {
            const uint32_t o = orig[p];
            xs[p] = xyz[3 * (size_t)o];
            ys[p] = xyz[3 * (size_t)o + 1];
            zs[p] = xyz[3 * (size_t)o + 2];
            inv[o] = p;
        }
        bool voxel, tile;
        block_heads<kBlock>(skey, n, T, first + r * kBlock, open, s_head, voxel, tile);
        const unsigned long long mt = __ballot(tile), mv = __ballot(voxel);
        if (lane == 0) {
            atomicAdd(&s_tiles, (uint32_t)__popcll(mt));
            atomicAdd(&s_voxels, (uint32_t)__popcll(mv));
        }
    }
    __syncthreads();
    if (tid == 0) {
        part_tiles[blockIdx.x] = s_tiles;
        part_voxels[blockIdx.x] = s_voxels;
    }
}

struct TileArrays {
    uint32_t *start, *cnt;
    float *cx, *cy, *cz, *rad;
};

// Tiles.  A wavefront takes those that start in 64 consecutive sorted
// positions, as many at a time as lie whole in a window of 64 (the next window
// starts where the last of them ended, so there are two at most), and reduces
// them together: lane by lane towards the tile's first position, as far as
// the longest tile of the window goes.  Most tiles of a sparse cloud hold a
// few points (125,000 points in 64 clouds: 10 us; 37 with a wavefront's
// reductions for every tile).
//
// The sphere centre is the FP32-rounded centre of the tile's bounding box; the
// radius is the largest member distance to that centre, in FP64, enlarged by
// 2^-40 relative and rounded up to FP32, so it is never below the true largest
// distance.  Any sphere that encloses the members keeps the pruning test
// conservative.
//
// seg, starts: the 64 positions and those that start a tile; t0: number of the
// first of these tiles.
__device__ void wave_tiles(const uint32_t *skey, int n, int T, uint32_t seg, unsigned long long starts, uint32_t t0,
                           const float *xs, const float *ys, const float *zs, const TileArrays &out)
{
    const int lane = threadIdx.x & (kWave - 1);
    uint32_t todo = (uint32_t)__popcll(starts);
    uint32_t start = seg + (starts ? __builtin_ctzll(starts) : 0);
    while (todo) {
        const uint32_t i = start + lane, ic = i < (uint32_t)n ? i : start;
        const uint32_t k = skey[ic];
        const uint32_t kn = i + 1 < (uint32_t)n ? skey[i + 1] : ~k;
        const uint32_t kp = (uint32_t)__shfl_up((int)k, 1, kWave);
        const unsigned long long change = __ballot(lane == 0 || k != kp);
        // position in the voxel, from its first position in the window or
        // (the window starts with a tile) from the window's
        const uint32_t off = lane - (63 - __builtin_clzll(change & (~0ull >> (63 - lane))));
        const bool in = i < (uint32_t)n;
        const unsigned long long ends = __ballot(in && (kn != k || (off + 1) % (uint32_t)T == 0));
        const unsigned long long heads = __ballot(in && off % (uint32_t)T == 0);
        // whole tiles of the window that are this wavefront's (at least
        // one: a tile has at most 64 positions)
        const uint32_t have = min(todo, (uint32_t)__popcll(ends));
        const unsigned long long after = ends >> lane;
        const int left = after ? __builtin_ctzll(after) : 0;  // positions of the lane's tile after it
        const uint32_t rank = (uint32_t)__popcll(heads & ((1ull << lane) - 1ull));
        const bool mine = after != 0ull && rank - (((heads >> lane) & 1ull) ? 0u : 1u) < have;
        const bool head = ((heads >> lane) & 1ull) && mine;
        const int longest = (int)wave_max_u32(head ? (uint32_t)left : 0u);
        float p[3], lo[3], hi[3], c[3];
        p[0] = xs[ic];
        p[1] = ys[ic];
        p[2] = zs[ic];
#pragma unroll
        for (int a = 0; a < 3; ++a)
            lo[a] = hi[a] = p[a];
        // after the step with offset o a lane covers 2 o positions of its tile
        for (int o = 1; o <= longest; o <<= 1) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float l = __shfl_down(lo[a], o, kWave), h = __shfl_down(hi[a], o, kWave);
                lo[a] = o <= left ? fminf(lo[a], l) : lo[a];
                hi[a] = o <= left ? fmaxf(hi[a], h) : hi[a];
            }
        }
        const int hl = 63 - __builtin_clzll((heads | 1ull) & (~0ull >> (63 - lane)));
        double r2 = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            c[a] = __shfl((float)(0.5 * ((double)lo[a] + (double)hi[a])), hl, kWave);
            const double d = (double)p[a] - (double)c[a];
            r2 = a ? r2 + d * d : d * d;
        }
        for (int o = 1; o <= longest; o <<= 1) {
            const double v = __shfl_down(r2, o, kWave);
            r2 = o <= left ? fmax(r2, v) : r2;
        }
        if (head) {
            double rr = sqrt(r2) * (1.0 + 0x1p-40) + 0x1p-120;
            float r32 = (float)rr;
            if ((double)r32 < rr)
                r32 = nextafterf(r32, INFINITY);
            const uint32_t t = t0 + rank;
            out.start[t] = i;
            out.cnt[t] = (uint32_t)left + 1u;
            out.cx[t] = c[0];
            out.cy[t] = c[1];
            out.cz[t] = c[2];
            out.rad[t] = r32;
        }
        // (unsorted keys, after a failed build, could end no tile here)
        if (!have)
            break;
        t0 += have;
        todo -= have;
        unsigned long long e = ends;
        for (uint32_t q = 1; q < have && todo; ++q)
            e &= e - 1;
        start += todo ? __builtin_ctzll(e) + 1 : 0;
    }
}

__global__ __launch_bounds__(kBlock) void k_tiles(const uint32_t *__restrict__ skey, int n, int T,
                                                  const uint32_t *__restrict__ part_tiles,
                                                  const uint32_t *__restrict__ part_voxels, IndexHeader *hdr,
                                                  const float *__restrict__ xs, const float *__restrict__ ys,
                                                  const float *__restrict__ zs, TileArrays out)
{
    __shared__ uint32_t s_head[kWavesPerBlock], s_open, wsum[kWavesPerBlock];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int steps = tile_steps(n), nb = gridDim.x, me = blockIdx.x;
    const uint32_t first = me * (uint32_t)(kBlock * steps);
    uint32_t sum = 0, voxels = 0, base, total;
    for (int q = tid; q < me; q += kBlock)
        sum += part_tiles[q];
    if (me == nb - 1)
        for (int q = tid; q < nb; q += kBlock)
            voxels += part_voxels[q];
    if (tid < kWave) {
        const uint32_t o = voxel_start(skey, first, lane);
        if (tid == 0)
            s_open = o;
    }
    block_exclusive_scan(sum, wsum, base);
    block_exclusive_scan(voxels, wsum, total);
    if (me == nb - 1 && tid == 0) {
        hdr->n_voxels = total;
        hdr->n_tiles = base + part_tiles[me];
    }
    uint32_t open = s_open;
    for (int r = 0; r < steps; ++r) {
        bool voxel, tile;
        block_heads<kBlock>(skey, n, T, first + r * kBlock, open, s_head, voxel, tile);
        uint32_t nt;
        uint32_t t0 = base + block_exclusive_scan(tile ? 1u : 0u, wsum, nt);  // lane 0's: of the wavefront's first
        t0 = (uint32_t)__shfl((int)t0, 0, kWave);
        wave_tiles(skey, n, T, first + r * kBlock + w * kWave, __ballot(tile), t0, xs, ys, zs, out);
        base += nt;
    }
}

// The build of a small cloud up to its tiles in one workgroup: the same steps
// as the kernels above, with barriers for launches and the sort in LDS.  The launches
// are what a small build costs, so this takes over while one workgroup's work
// is below theirs (1,024 points 38 us against 46 by the kernels, 4,096 points
// 49 against 51; with the tiles in it too, 4,096 points took 66).
constexpr int kSmallItems = 4;
constexpr int kSmallPoints = kSmallItems * kSortBlock;
constexpr int kSmallParts = kSmallPoints / kBlock;
static_assert(kSmallPoints <= kBlock * kTileParts, "one step per block of k_tiles");
__global__ __launch_bounds__(kSortBlock) void k_build_small(const float *__restrict__ xyz, int n, IndexHeader *hdr,
                                                            int n_vox, double shell_inv, uint32_t shell_cap,
                                                            int passes, int T, uint32_t *skey, uint32_t *orig,
                                                            uint32_t *inv, float *xs, float *ys, float *zs,
                                                            uint32_t *part_tiles, uint32_t *part_voxels)
{
    __shared__ float s_box[kSortWaves][8];
    __shared__ uint32_t s_key[kSmallPoints], s_val[kSmallPoints];
    __shared__ uint32_t wcnt[kSortWaves][256];
    __shared__ uint32_t wsum[kSortWaves], s_head[kSortWaves], s_part[2][kSmallParts];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    // a wavefront takes consecutive points
    const int items = (n + kSortBlock - 1) / kSortBlock;
    const int first = w * (items * kWave) + lane;
    float p[kSmallItems][3];
    bool valid[kSmallItems];
    Box b = {{INFINITY, INFINITY, INFINITY}, {-INFINITY, -INFINITY, -INFINITY}, false};
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
        const int i = first + r * kWave;
        valid[r] = r < items && i < n;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            p[r][a] = valid[r] ? xyz[3 * (size_t)i + a] : 0.0f;
            if (valid[r]) {
                b.bad |= !isfinite(p[r][a]);
                b.mn[a] = fminf(b.mn[a], p[r][a]);
                b.mx[a] = fmaxf(b.mx[a], p[r][a]);
            }
        }
    }
    b = block_box<kSortBlock>(b, s_box);
    const Grid g = grid_of(b.mn, b.mx, b.bad, (uint32_t)n_vox);
    begin_header(hdr, b, g, shell_inv, shell_cap);
    uint32_t key[kSmallItems], val[kSmallItems], rank[kSmallItems];
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
        key[r] = valid[r] ? voxel_key(p[r][0], p[r][1], p[r][2], g.pmin, g.L, (uint32_t)n_vox, g.origin, shell_inv,
                                      shell_cap)
                          : 0u;
        val[r] = (uint32_t)(first + r * kWave);
    }
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = 8 * pass;
        for (int q = tid; q < kSortWaves * 256; q += kSortBlock)
            wcnt[0][q] = 0;
        if (pass) {
#pragma unroll
            for (int r = 0; r < kSmallItems; ++r) {
                key[r] = valid[r] ? s_key[first + r * kWave] : 0u;
                val[r] = valid[r] ? s_val[first + r * kWave] : 0u;
            }
        }
        __syncthreads();
        digit_ranks<kSmallItems>(key, valid, shift, wcnt[w], rank);
        __syncthreads();
        uint32_t all = 0, total;
        if (tid < 256)
#pragma unroll
            for (int q = 0; q < kSortWaves; ++q)
                all += wcnt[q][tid];
        const uint32_t base = block_exclusive_scan<kSortBlock>(all, wsum, total);
        if (tid < 256)
            digit_bases<kSortWaves>(wcnt, base);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSmallItems; ++r) {
            if (valid[r]) {
                const uint32_t off = wcnt[w][(key[r] >> shift) & 255u] + rank[r];
                s_key[off] = key[r];
                s_val[off] = val[r];
            }
        }
        __syncthreads();
    }
    if (tid < 2 * kSmallParts)
        s_part[0][tid] = 0u;
    for (int q = tid; q < n; q += kSortBlock) {
        const uint32_t o = s_val[q];
        skey[q] = s_key[q];
        orig[q] = o;
        inv[o] = (uint32_t)q;
        xs[q] = xyz[3 * (size_t)o];
        ys[q] = xyz[3 * (size_t)o + 1];
        zs[q] = xyz[3 * (size_t)o + 2];
    }
    // tiles and voxels of every block of k_tiles
    uint32_t open = 0;
    for (int p0 = 0; p0 < n; p0 += kSortBlock) {
        bool voxel, tile;
        block_heads<kSortBlock>(s_key, n, T, (uint32_t)p0, open, s_head, voxel, tile);
        const unsigned long long mt = __ballot(tile), mv = __ballot(voxel);
        if (lane == 0) {
            atomicAdd(&s_part[0][(p0 + w * kWave) / kBlock], (uint32_t)__popcll(mt));
            atomicAdd(&s_part[1][(p0 + w * kWave) / kBlock], (uint32_t)__popcll(mv));
        }
    }
    __syncthreads();
    if (tid < (n + kBlock - 1) / kBlock) {
        part_tiles[tid] = s_part[0][tid];
        part_voxels[tid] = s_part[1][tid];
    }
}

// Coordinates of the picks in pick order: the input of the next stage of a
// multi-stage down-sampling.  An index outside [0, n) gives NaN coordinates,
// which the next index build reports as non-finite input.
__global__ __launch_bounds__(kBlock) void k_gather_xyz(const float *__restrict__ xyz, int n,
                                                       const int32_t *__restrict__ idx, int m,
                                                       float *__restrict__ out)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= m)
        return;
    const int32_t i = idx[j];
    const bool ok = i >= 0 && i < n;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        out[3 * (size_t)j + a] = ok ? xyz[3 * (size_t)i + a] : NAN;
}

// Euclidean mode: the sampler keeps squared class tops; the reported
// distance is their correctly rounded root (the same root for every value of
// a class).
__global__ __launch_bounds__(kBlock) void k_sqrt_out(float *__restrict__ d, int m)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < m)
        d[j] = sqrt_rn(d[j]);
}

}  // namespace rfps

namespace rfps {

static inline int blocks_for(long long n, int per_block) { return (int)((n + per_block - 1) / per_block); }

hipError_t launch_gather_xyz(const float *xyz, int n, const int32_t *idx, int m, float *out, hipStream_t s)
{
    k_gather_xyz<<<blocks_for(m, kBlock), kBlock, 0, s>>>(xyz, n, idx, m, out);
    return hipGetLastError();
}

hipError_t launch_sqrt_out(float *d, int m, hipStream_t s)
{
    k_sqrt_out<<<blocks_for(m, kBlock), kBlock, 0, s>>>(d, m);
    return hipGetLastError();
}

static hipError_t launch_scan(const uint32_t *in, uint32_t *out, int n, uint32_t *partials, hipStream_t s)
{
    const int nb = blocks_for(n, kScanChunk);
    if (nb > kBlock * 64)
        return hipErrorInvalidValue;
    k_scan_blocks<<<nb, kBlock, 0, s>>>(in, out, n, partials);
    k_scan_partials<<<1, kBlock, 0, s>>>(partials, nb);
    k_scan_add<<<blocks_for(n, kBlock), kBlock, 0, s>>>(out, n, partials);
    return hipGetLastError();
}

static TileArrays tile_arrays(const IndexView &v) { return {v.tstart, v.tcnt, v.tcx, v.tcy, v.tcz, v.trad}; }

// Sorts the keys in A (whose first histogram is there) and builds the tiles.
static hipError_t launch_sort_and_tiles(const IndexView &v, const float *xyz, const uint32_t *range, hipStream_t s)
{
    const int n = v.n, nblk = blocks_for(n, kRadixTile);
    const bool rows = nblk <= kDirectBlocks;
    uint32_t *kin = v.keyA, *vin = v.valA, *kout = v.keyB, *vout = v.valB;
    for (int pass = 0; pass < v.radix_passes; ++pass) {
        const int shift = 8 * pass;
        // (two passes at a time, so that the result stays in its buffer)
        const bool skip = range && v.radix_passes == 4 && pass >= 2;
        if (pass)
            k_radix_hist<<<nblk, kSortBlock, 0, s>>>(kin, n, shift, v.hist, nblk, rows, range, skip);
        if (!rows) {
            const hipError_t e = launch_scan(v.hist, v.hist, 256 * nblk, v.partials, s);
            if (e != hipSuccess)
                return e;
        }
        k_radix_scatter<<<nblk, kSortBlock, 0, s>>>(kin, vin, kout, vout, n, shift, v.hist, nblk, rows, range, skip);
        std::swap(kin, kout);
        std::swap(vin, vout);
    }
    // v.skey / v.orig alias the buffers that hold the final pass
    const int nb = blocks_for(n, kBlock * tile_steps(n));
    k_gather<<<nb, kBlock, 0, s>>>(xyz, v.orig, v.skey, n, v.tile, v.xs, v.ys, v.zs, v.inv, v.tcount, v.tbase);
    k_tiles<<<nb, kBlock, 0, s>>>(v.skey, n, v.tile, v.tcount, v.tbase, v.hdr, v.xs, v.ys, v.zs, tile_arrays(v));
    return hipGetLastError();
}

hipError_t launch_build_index(const IndexView &v, const float *xyz, hipStream_t s)
{
    const int n = v.n, nblk = blocks_for(n, kRadixTile);
    if (n <= kSmallPoints) {
        k_build_small<<<1, kSortBlock, 0, s>>>(xyz, n, v.hdr, v.n_vox, v.shell_inv, v.shell_cap, v.radix_passes,
                                               v.tile, v.skey, v.orig, v.inv, v.xs, v.ys, v.zs, v.tcount, v.tbase);
        k_tiles<<<blocks_for(n, kBlock), kBlock, 0, s>>>(v.skey, n, v.tile, v.tcount, v.tbase, v.hdr, v.xs, v.ys, v.zs,
                                                         tile_arrays(v));
        return hipGetLastError();
    }
    const int parts = std::min(blocks_for(n, kBlock * 4), kBoxParts);
    float *box = reinterpret_cast<float *>(v.flags);  // 8 words per 1,024 points, and 64 words at least
    k_bbox<<<parts, kBlock, 0, s>>>(xyz, n, box);
    k_voxel_key<<<nblk, kSortBlock, 0, s>>>(xyz, n, box, parts, v.hdr, v.n_vox, v.shell_inv, v.shell_cap, v.keyA, v.valA,
                                        v.hist, nblk, nblk <= kDirectBlocks);
    return launch_sort_and_tiles(v, xyz, nullptr, s);
}

}  // namespace rfps

// ---------------------------------------------------------------------------
// Batched index: the clouds of a batch share one sorted index.  A point of
// cloud c gets the key base_c + V_id (V_id on the cloud's own grid), so
// voxels and tiles never mix clouds and the tiles of every cloud are one
// contiguous range.
// ---------------------------------------------------------------------------
namespace rfps {

// Cloud of global point i: the largest c in [lo, hi] with offsets[c] <= i (lo
// if there is none).
__device__ __forceinline__ int cloud_of(const int32_t *off, int lo, int hi, int i)
{
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= i)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// The same for one point by all lanes of a wavefront, 64 probes a step (a
// chain of single loads took most of the kernels that start with it).
__device__ __forceinline__ int wave_cloud_of(const int32_t *off, int B, int i)
{
    const int lane = threadIdx.x & (kWave - 1);
    int lo = 0, hi = B - 1;
    while (lo < hi) {
        const int step = (hi - lo + kWave - 1) / kWave, q = lo + (lane + 1) * step;
        // clouds lo + step, lo + 2 step, .. that start at or before i
        const int c = __popcll(__ballot(q <= hi && off[q <= hi ? q : lo] <= i));
        lo += c * step;
        hi = min(lo + step - 1, hi);
    }
    return lo;
}

// Clears the per-cloud boxes and the exchange board (epochs restart at 1 in
// every call) and, in the first workgroup, resets the header and the batch
// state, checks the batch description (offsets from 0 to n with every cloud
// non-empty, 1 <= m_c <= N_c, start indices inside their clouds, sum of m
// equal to the output length) and computes the output offsets, the bins per
// axis and the first key of every cloud.
__global__ __launch_bounds__(kBlock) void k_batch_begin(IndexHeader *hdr, BatchCtl bc, int n, uint32_t *cl_bb,
                                                        uint32_t *cl_nvox, uint32_t *cl_base, BatchState *st,
                                                        unsigned long long *board)
{
    __shared__ uint32_t s_bad, wsum[kWavesPerBlock];
    const int tid = threadIdx.x;
    if (blockIdx.x) {
        const int t = (blockIdx.x - 1) * kBlock + tid, nth = (gridDim.x - 1) * kBlock;
        for (int c = t; c < bc.batch; c += nth) {
            for (int a = 0; a < 3; ++a) {
                cl_bb[6 * c + a] = 0xffffffffu;
                cl_bb[6 * c + 3 + a] = 0u;
            }
        }
        for (int w = t; w < kBoardWords; w += nth)
            board[w] = 0ull;
        return;
    }
    if (tid == 0) {
        hdr->build_status = 0;
        hdr->sample_status = 0;
        hdr->n_voxels = 0;
        hdr->n_tiles = 0;
        hdr->last_m = (uint32_t)bc.m_total;
        hdr->trace_n = 0;
        for (int t = 0; t < kTeleFields; ++t)
            hdr->tele[t] = 0;
        st->joined = 0;
        for (int x = 0; x < kMaxXcds; ++x)
            st->next[x] = st->xcd_count[x] = 0;
        s_bad = (bc.offsets[0] != 0 || bc.offsets[bc.batch] != n) ? 1u : 0u;
    }
    __syncthreads();
    // kBlock clouds at a time; keys of a valid batch are below 2^32, and a
    // larger range is caught by its high part
    unsigned long long base = 0, out = 0;
    for (int c0 = 0; c0 < bc.batch; c0 += kBlock) {
        const int c = c0 + tid;
        uint32_t cells_lo = 0, cells_hi = 0, m = 0;
        if (c < bc.batch) {
            const int nc = bc.offsets[c + 1] - bc.offsets[c];
            const int mc = bc.m[c];
            const int sc = bc.starts ? bc.starts[c] : 0;
            if (nc < 1 || mc < 1 || mc > nc || sc < 0 || sc >= nc)
                atomicOr(&s_bad, 1u);
            const uint32_t nv = (uint32_t)(bc.fixed_n_vox ? bc.fixed_n_vox : default_n_vox_rule(nc > 0 ? nc : 1));
            cl_nvox[c] = nv;
            const unsigned long long cells =
                (unsigned long long)nv * nv * nv * shell_cap_for(nv, bc.shell_inv > 0.0);
            cells_lo = (uint32_t)(cells & 0xffffffu);  // sums of 256 of either part stay below 2^32
            cells_hi = (uint32_t)(cells >> 24);
            m = mc > 0 ? (uint32_t)mc : 0u;
        }
        uint32_t tl, th, tm;
        const uint32_t lo = block_exclusive_scan(cells_lo, wsum, tl);
        const uint32_t hi = block_exclusive_scan(cells_hi, wsum, th);
        // (m <= N_c in a valid batch; of an invalid one only the flag counts)
        const uint32_t mo = block_exclusive_scan(m, wsum, tm);
        if (c < bc.batch) {
            cl_base[c] = (uint32_t)(base + lo + ((unsigned long long)hi << 24));
            bc.out_offsets[c] = (uint32_t)out + mo;
        }
        base += tl + ((unsigned long long)th << 24);
        out += tm;
    }
    __syncthreads();
    if (tid == 0) {
        cl_base[bc.batch] = (uint32_t)base;
        bc.out_offsets[bc.batch] = (uint32_t)out;
        if (s_bad || out != (unsigned long long)bc.m_total)
            set_status(&hdr->build_status, RFPS_ERR_INVALID_ARG);
        else if (base > 0xffffffffull)
            set_status(&hdr->build_status, RFPS_ERR_UNSUPPORTED);
    }
}

// Bounding box of every cloud.  A wavefront takes a run of
// consecutive points and keeps the running box of the cloud it is in,
// flushing it with one atomic per bound when the run moves into the next
// cloud (clouds are contiguous ranges of the input) and at its end.  A run is
// long enough that the atomics are few, and short enough that there are
// wavefronts for the device.
__host__ __device__ inline int bbox_run(int n) { return n < (1 << 20) ? 256 : 2048; }

__global__ __launch_bounds__(kBlock) void k_bbox_batch(const float *__restrict__ xyz, int n, BatchCtl bc,
                                                       uint32_t *cl_bb, IndexHeader *hdr)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int gw = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int nw = gridDim.x * blockDim.x / kWave;
    const int run = bbox_run(n);
    bool bad = false;
    for (int b = gw * run; b < n; b += nw * run) {
        const int e = min(b + run, n);
        // (the last cloud runs to n whatever the offsets say, so that
        // inconsistent offsets, reported by the setup kernel, stay in bounds)
        int c = wave_cloud_of(bc.offsets, bc.batch, b);
        int cend = c + 1 < bc.batch ? bc.offsets[c + 1] : n;
        float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
        auto flush = [&]() {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float lo = wave_min_f32(mn[a]);
                const float hi = wave_max_f32(mx[a]);
                if (lane == 0 && lo <= hi) {
                    atomicMin(&cl_bb[6 * c + a], f2ord(lo));
                    atomicMax(&cl_bb[6 * c + 3 + a], f2ord(hi));
                }
                mn[a] = INFINITY;
                mx[a] = -INFINITY;
            }
        };
        for (int i0 = b; i0 < e; i0 += kWave) {
            const int i = i0 + lane;
            const bool valid = i < e;
            float p[3] = {0.0f, 0.0f, 0.0f};
            if (valid) {
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    p[a] = xyz[3 * (size_t)i + a];
                    bad |= !isfinite(p[a]);
                }
            }
            // the lanes of one step may belong to several clouds
            bool todo = valid;
            while (__any(todo)) {
                const bool mine = todo && i < cend;
                if (mine) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        mn[a] = fminf(mn[a], p[a]);
                        mx[a] = fmaxf(mx[a], p[a]);
                    }
                }
                todo = todo && !mine;
                if (__any(todo)) {
                    flush();
                    ++c;
                    cend = c + 1 < bc.batch ? bc.offsets[c + 1] : n;
                }
            }
        }
        flush();
    }
    if (__any(bad) && lane == 0)
        set_status(&hdr->build_status, RFPS_ERR_NONFINITE);
}

// Voxel key of every point on its own cloud's grid (eq. voxel_size; formed
// from the cloud's box, a few operations beside the key's), the identity
// payload and the histogram of the first digit.
__global__ __launch_bounds__(kSortBlock) void k_voxel_key_batch(const float *__restrict__ xyz, int n, BatchCtl bc,
                                                            const IndexHeader *__restrict__ hdr,
                                                            const uint32_t *__restrict__ cl_nvox,
                                                            const uint32_t *__restrict__ cl_base,
                                                            const uint32_t *__restrict__ cl_bb, uint32_t *key,
                                                            uint32_t *val, uint32_t *__restrict__ hist, int nblk,
                                                            bool rows)
{
    __shared__ uint32_t h[256];
    const int tid = threadIdx.x;
    if (tid < 256)
        h[tid] = 0;
    __syncthreads();
    const bool failed = hdr->build_status != 0;
    const int base = blockIdx.x * kRadixTile;
    // the clouds of the workgroup's points: usually one or two
    const int c0 = wave_cloud_of(bc.offsets, bc.batch, base);
    const int c1 = wave_cloud_of(bc.offsets, bc.batch, min(base + kRadixTile, n) - 1);
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int i = base + r * kSortBlock + tid;
        if (i < n) {
            const int c = cloud_of(bc.offsets, c0, c1, i);
            const uint32_t nv = cl_nvox[c];
            float lo[3], hi[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                lo[a] = ord2f(cl_bb[6 * c + a]);
                hi[a] = ord2f(cl_bb[6 * c + 3 + a]);
            }
            const Grid g = grid_of(lo, hi, failed, nv);
            const uint32_t k = cl_base[c] + voxel_key(xyz[3 * (size_t)i], xyz[3 * (size_t)i + 1],
                                                      xyz[3 * (size_t)i + 2], g.pmin, g.L, nv, g.origin, bc.shell_inv,
                                                      shell_cap_for(nv, bc.shell_inv > 0.0));
            key[i] = k;
            val[i] = (uint32_t)i;
            atomicAdd(&h[k & 255u], 1u);
        }
    }
    __syncthreads();
    if (tid < 256)
        hist[hist_at(tid, blockIdx.x, nblk, rows)] = h[tid];
}

hipError_t launch_build_batch(const IndexView &v, const float *xyz, hipStream_t s)
{
    const int n = v.n, nblk = blocks_for(n, kRadixTile);
    k_batch_begin<<<33, kBlock, 0, s>>>(v.hdr, v.bc, n, v.cl_bb, v.cl_nvox, v.cl_base, v.bstate, v.board);
    k_bbox_batch<<<std::min(blocks_for(n, bbox_run(n) * kWavesPerBlock), 1024), kBlock, 0, s>>>(xyz, n, v.bc, v.cl_bb,
                                                                                          v.hdr);
    k_voxel_key_batch<<<nblk, kSortBlock, 0, s>>>(xyz, n, v.bc, v.hdr, v.cl_nvox, v.cl_base, v.cl_bb, v.keyA, v.valA,
                                              v.hist, nblk, nblk <= kDirectBlocks);
    return launch_sort_and_tiles(v, xyz, v.cl_base + v.bc.batch, s);
}

}  // namespace rfps
