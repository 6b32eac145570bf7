// Farthest point sampling of a small cloud by one workgroup, all of it in
// registers: no pruning, no exchange between workgroups, one barrier per
// selection.
//
// Thread t keeps the points t, t + BLOCK, .. of the cloud in original order.
// A selection is: update every distance, the largest of the lane and of the
// wavefront, and an LDS maximum over the wavefronts' keys (distance, then
// lowest index); the winner's coordinates are read back from LDS.  The keys
// lie in a ring, one word per selection, so that nothing is cleared or stored
// on the way: every 64 selections one wavefront writes them out and clears
// them.
//
// What bounds it is that chain (two LDS reads, an LDS maximum, a barrier, six
// cross-lane steps): 0.20 us a selection with two points a thread of eight
// wavefronts, 0.28 with four; from there on the arithmetic over all points.
// The team sampler's rounds cost 6 to 7 us whatever the cloud and settle eight
// picks of a cloud of 1,024 points: 1,024 -> 256 from call to completion 213
// -> 73 us, 2,048 -> 512 263 -> 167.  (Sixteen wavefronts: 98 and 197; keys in
// a slot per wavefront, certified several at a time by one of them: 145 and
// 296.)
#pragma once

#include "rfps_internal.h"
#include "round_layout.h"

namespace rfps {

struct SoloJob {
    const float *xs, *ys, *zs;  // sorted points of the index
    const uint32_t *inv;        // sorted positions of the cloud's points, by original index
    int32_t n, m, start;
    int32_t *out_idx;
    float *out_d2;
};

constexpr int kSoloRing = 2 * kWave;
static_assert(kSoloRing * 8 == kSoloRingBytes, "the ring's part of solo_lds");

// LDS maximum of the 64-bit value hi : lo.  As an instruction of its own: the
// compiler would reduce over the active lanes first, and there is one, or a
// few that tie.  (The wait before the barrier is the caller's.)
__device__ __forceinline__ void lds_max_u64(unsigned long long *p, uint32_t hi, uint32_t lo)
{
    typedef __attribute__((address_space(3))) unsigned long long lds_u64;
    const uint32_t at = (uint32_t)reinterpret_cast<uintptr_t>((lds_u64 *)p);
    const unsigned long long v = ((unsigned long long)hi << 32) | lo;
    asm volatile("ds_max_u64 %0, %1" ::"v"(at), "v"(v) : "memory");
}

// All threads of a workgroup of WAVES wavefronts, P points a thread
// (job.n <= P * WAVES * 64); smem: solo_lds(n) bytes.  Writes the selections
// after the start, whose output is the caller's.
template <int WAVES, int P, bool E>
__device__ void solo_cloud(const SoloJob &job, unsigned char *smem)
{
    constexpr int BLOCK = WAVES * kWave;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    unsigned long long *const ring = reinterpret_cast<unsigned long long *>(smem);
    unsigned char *const place = smem + kSoloRingBytes;
    float4 *const pts = reinterpret_cast<float4 *>(place);
    float x[P], y[P], z[P], d[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int i = p * BLOCK + tid;
        const bool in = i < job.n;
        x[p] = y[p] = z[p] = 0.0f;
        d[p] = in ? INFINITY : 0.0f;  // a slot without a point follows all points (by its index)
        if (in) {
            const uint32_t q = job.inv[i];
            x[p] = job.xs[q];
            y[p] = job.ys[q];
            z[p] = job.zs[q];
            pts[i] = make_float4(x[p], y[p], z[p], 0.0f);
        }
    }
    if (tid < kSoloRing)
        ring[tid] = 0ull;
    __syncthreads();
    // low half of a point's key: minus (16 times its index + 1), so that the
    // lowest index is the largest, and the complement its place in LDS
    const uint32_t low0 = ~(uint32_t)(16 * tid), low_step = (uint32_t)(-16 * BLOCK);
    const bool some = wave * kWave < job.n;   // the wavefront has points
    uint32_t at = 16u * (uint32_t)job.start;  // the last selection
    // selections first .. last - 1 of one half of the ring, by one wavefront
    auto flush = [&](int first, int last) {
        const int j = first + lane;
        const unsigned long long key = ring[j & (kSoloRing - 1)];
        ring[j & (kSoloRing - 1)] = 0ull;
        if (j >= 1 && j < last) {
            job.out_idx[j] = (int32_t)(~(uint32_t)key / 16u);
            if (job.out_d2)
                job.out_d2[j] = __uint_as_float((uint32_t)(key >> 32));
        }
    };
    for (int j = 1; j < job.m; ++j) {
        const float4 s = *reinterpret_cast<const float4 *>(place + at);
        uint32_t top = 0, low = low0;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const float t = sqdist(x[p], y[p], z[p], s.x, s.y, s.z);
            d[p] = min_dist(d[p], t, E);
            // distances are not negative, so their bits order like them
            const uint32_t db = __float_as_uint(d[p]);
            low = p && db > top ? low0 + (uint32_t)p * low_step : low;
            top = p ? max(top, db) : db;
        }
        const uint32_t mh = wave_max_u32(top);
        // (lanes that tie all raise the maximum: the lowest index wins it)
        unsigned long long *const word = &ring[j & (kSoloRing - 1)];
        if (top == mh && some)
            lds_max_u64(word, top, low);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        at = ~(uint32_t)*word;
        // a half of the ring is full: nobody reads it any more, and it is
        // written again 64 selections on (but its last word is read just now)
        if ((j & (kWave - 1)) == 0 && wave == (j / kWave) % WAVES && j >= kWave)
            flush(j - kWave, j);
    }
    __syncthreads();
    const int left = (job.m - 1) / kWave * kWave;
    if (wave == 0)
        flush(left, job.m);
    __syncthreads();  // LDS is reused by the next cloud
}

// The same for the smallest P that holds the cloud (kSoloPoints at most).
constexpr int kSoloWaves = 8;
template <bool E>
__device__ __forceinline__ void solo_any(const SoloJob &job, unsigned char *smem)
{
    constexpr int B = kSoloWaves * kWave;
    if (job.n <= B)
        solo_cloud<kSoloWaves, 1, E>(job, smem);
    else if (job.n <= 2 * B)
        solo_cloud<kSoloWaves, 2, E>(job, smem);
    else if (job.n <= 4 * B)
        solo_cloud<kSoloWaves, 4, E>(job, smem);
    else if (job.n <= 6 * B)
        solo_cloud<kSoloWaves, 6, E>(job, smem);
    else if (job.n <= 8 * B)
        solo_cloud<kSoloWaves, 8, E>(job, smem);
    else
        solo_cloud<kSoloWaves, 16, E>(job, smem);
}
static_assert(kSoloPoints <= 16 * kSoloWaves * kWave, "points of a lane");

}  // namespace rfps
