// Voxel-parameter network: cloud features, forward pass, gradient and Adam
// training step (C ABI in include/rfps_mlp.h).
//
// The network maps 516 features of a cloud (log N, the bounding-box extents
// and the 8^3 occupancy histogram) through two hidden layers of 64 ReLU
// units to 72 outputs: a predicted relative log run time and a pruning rate
// for each of 36 candidate (n_vox, shell spacing) pairs.  Weight matrices are used in
// bfloat16 (round to nearest even of an FP32 master copy); biases,
// activations, accumulation and the optimiser state are FP32.  Whatever the
// network picks, the sampled sequence is the same (every partition is
// output-neutral); it only changes the speed.
//
// The products run on the matrix cores (v_mfma_f32_16x16x4f32).  A gradient is
// two launches: k_rows takes 16 rows of the batch through the forward pass,
// the loss and the backward pass with everything in LDS, and k_wgrad forms the
// weight gradients, one 16 x 16 tile per workgroup.  The arithmetic is 0.3
// GFLOP for 2,000 rows; what bounds both is their chains of loads and matrix
// instructions, so every chain is cut as short as the device and the order of
// the sums allow (a product over the rows is split over eight wavefronts, and
// no step of the backward pass waits for a launch).  2,000 rows: 1,532 -> 34
// us; as 14 launches, the three one-workgroup column sums and the loss alone
// took over a millisecond.
#include <math.h>

#include <algorithm>

#include "../../include/rfps_mlp.h"
#include "rfps_internal.h"

namespace rfps {
namespace mlp {

constexpr int kIn = RFPS_MLP_INPUTS, kH = 64, kOut = RFPS_MLP_OUTPUTS;
constexpr int kP = RFPS_MLP_PARAMS;
// packed parameter order: W1 [64][516], b1 [64], W2 [64][64], b2 [64], W3 [72][64], b3 [72]
constexpr int oW1 = 0, ob1 = oW1 + kH * kIn, oW2 = ob1 + kH, ob2 = oW2 + kH * kH, oW3 = ob2 + kH,
              ob3 = oW3 + kOut * kH, oEnd = ob3 + kOut;
static_assert(oEnd == kP, "parameter count");

constexpr float kBeta1 = 0.9f, kBeta2 = 0.999f, kEps = 1e-8f;
constexpr int kMaxRows = 1 << 16;  // rows of one forward or training call

// Candidate table: n_vox major, shell spacing minor (0 = one shell).
constexpr int kNVox[9] = {12, 16, 24, 32, 48, 64, 96, 128, 192};
constexpr float kShell[4] = {0.0f, 5.0f, 10.0f, 20.0f};

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Round to nearest even (finite inputs).
__device__ __forceinline__ uint16_t f32_to_bf16(float x)
{
    uint32_t u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Model state in the caller's memory (rfps_mlp_state_size bytes).
struct State {
    float *master, *m, *v;
    uint16_t *wbf;   // bf16 copy of master (packed like it; only the weight blocks are read)
    uint32_t *step;  // Adam steps taken
};

__device__ __forceinline__ floatx4 mma(float a, float b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Matrix instructions take A element (i, k) in lane i + 16k and B element
// (k, j) in lane j + 16k; result element (i, j) is in lane j + 16 (i / 4),
// component i % 4.  A row's products are added in the order of k, four to an
// instruction: the signs of the hidden layers' inputs decide which units pass
// a gradient, and another order, or a wider sum, turns a sign now and then,
// which changes the gradient by far more than rounding does.

// What the backward pass leaves for the weight gradients.
struct RowArrays {
    float *a1, *a2, *dy, *dz2, *dz1;
    double *loss;  // one term per workgroup of k_rows
};

// 16 rows of the batch: Y = X -> 64 ReLU -> 64 ReLU -> 72 outputs, and with
// GRAD the loss sum w (Y - T)^2 / B, dY = 2 w (Y - T) / B and the gradients of
// both hidden layers' inputs.  One 16 x 16 output tile per wavefront; a first
// layer's tile is one chain of 129 matrix instructions (32 clocks each), which
// is what bounds the kernel.  The first layer's weights and the inputs are
// staged in LDS by all eight wavefronts with wide loads, and the other layers'
// weights are loaded before the first barrier, so the later layers wait for
// LDS only.  LDS row strides are 4 mod 64 words (12 for dY; 2 for the weights,
// whose words hold two values), which spreads the 16 rows of an operand over
// all banks.
constexpr int kRows = 16, kRowsBlock = 512;
constexpr int kSteps1 = kIn / 4, kSteps2 = kH / 4, kSteps3 = kOut / 4;  // matrix instructions over 516, 64 and 72
static_assert(kIn % 4 == 0 && kH % 4 == 0 && kOut % 4 == 0, "whole instructions");
template <bool GRAD>
__global__ __launch_bounds__(kRowsBlock) void k_rows(const float *__restrict__ master,
                                                     const uint16_t *__restrict__ wbf, const float *__restrict__ x,
                                                     const float *__restrict__ t, const float *__restrict__ wt, int B,
                                                     float *__restrict__ yout, RowArrays out)
{
    constexpr int sX = kIn, sH = kH + 4, sY = kOut + 4;
    constexpr int kW1Bytes = kH * kIn * 2;
    static_assert(oW1 == 0 && kW1Bytes % 16 == 0, "copied in pieces of 16 bytes");
    __shared__ __align__(16) uint16_t W1[kH * kIn];
    __shared__ __align__(16) float X[kRows * sX];
    __shared__ __align__(16) float A1[kRows * sH], A2[kRows * sH], DY[kRows * sY], DZ[kRows * sH];
    __shared__ double s_loss[kRowsBlock / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const int m0 = blockIdx.x * kRows;
    const int rows = min(kRows, B - m0);
    const int n0 = (wave & 3) * 16;

    for (int e = tid; e < kW1Bytes / 16; e += kRowsBlock)
        reinterpret_cast<uint4 *>(W1)[e] = reinterpret_cast<const uint4 *>(wbf + oW1)[e];
    for (int e = tid; e < kRows * kIn; e += kRowsBlock)
        X[e] = e < rows * kIn ? x[(size_t)m0 * kIn + e] : 0.0f;
    float w2[kSteps2], w3[kSteps2], b3w[kSteps3], b2w[kSteps2];
    const int o3 = wave * 16 + li;  // output column of the third layer
    if (wave < 4) {
#pragma unroll
        for (int q = 0; q < kSteps2; ++q)
            w2[q] = bf16_to_f32(wbf[oW2 + (size_t)(n0 + li) * kH + 4 * q + lk]);
        if constexpr (GRAD) {
#pragma unroll
            for (int q = 0; q < kSteps3; ++q)
                b3w[q] = bf16_to_f32(wbf[oW3 + (size_t)(4 * q + lk) * kH + n0 + li]);
#pragma unroll
            for (int q = 0; q < kSteps2; ++q)
                b2w[q] = bf16_to_f32(wbf[oW2 + (size_t)(4 * q + lk) * kH + n0 + li]);
        }
    }
    if (wave < 5) {
#pragma unroll
        for (int q = 0; q < kSteps2; ++q)
            w3[q] = bf16_to_f32(wbf[oW3 + (size_t)min(o3, kOut - 1) * kH + 4 * q + lk]);
    }
    __syncthreads();

    // ---- layer 1 ----
    if (wave < 4) {
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        const float *xa = &X[li * sX + lk];
        const uint16_t *wb = &W1[(n0 + li) * kIn + lk];
#pragma unroll 16
        for (int q = 0; q < kSteps1; ++q)
            acc = mma(xa[4 * q], bf16_to_f32(wb[4 * q]), acc);
        const float bias = master[ob1 + n0 + li];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 4 * lk + r;
            const float z = acc[r] + bias;
            const float v = z > 0.0f ? z : 0.0f;
            A1[m * sH + n0 + li] = v;
            if (GRAD && m < rows)
                out.a1[(size_t)(m0 + m) * kH + n0 + li] = v;
        }
    }
    __syncthreads();
    // ---- layer 2 ----
    if (wave < 4) {
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int q = 0; q < kSteps2; ++q)
            acc = mma(A1[li * sH + 4 * q + lk], w2[q], acc);
        const float bias = master[ob2 + n0 + li];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 4 * lk + r;
            const float z = acc[r] + bias;
            const float v = z > 0.0f ? z : 0.0f;
            A2[m * sH + n0 + li] = v;
            if (GRAD && m < rows)
                out.a2[(size_t)(m0 + m) * kH + n0 + li] = v;
        }
    }
    __syncthreads();
    // ---- layer 3, loss ----
    double part = 0.0;
    if (wave < 5) {
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int q = 0; q < kSteps2; ++q)
            acc = mma(A2[li * sH + 4 * q + lk], w3[q], acc);
        if (o3 < kOut) {
            const float bias = master[ob3 + o3], sc = 2.0f / (float)B;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = 4 * lk + r;
                const float y = acc[r] + bias;
                const size_t o = (size_t)(m0 + m) * kOut + o3;
                if constexpr (GRAD) {
                    float g = 0.0f;
                    if (m < rows) {
                        const float w = wt ? wt[o] : 1.0f;
                        const float d = y - t[o];
                        g = sc * w * d;
                        part += (double)w * (double)d * (double)d;
                        out.dy[o] = g;
                    }
                    DY[m * sY + o3] = g;
                } else if (m < rows) {
                    yout[o] = y;
                }
            }
        }
    }
    if constexpr (!GRAD)
        return;
#pragma unroll
    for (int h = 32; h > 0; h >>= 1)
        part += __shfl_xor(part, h, 64);
    if (lane == 0)
        s_loss[wave] = part;
    __syncthreads();
    if (tid == 0) {
        double v = 0.0;
        for (int q = 0; q < kRowsBlock / 64; ++q)
            v += s_loss[q];
        out.loss[blockIdx.x] = v;
    }
    // ---- dZ2 = (dY W3) where A2 > 0 ----
    if (wave < 4) {
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int q = 0; q < kSteps3; ++q)
            acc = mma(DY[li * sY + 4 * q + lk], b3w[q], acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 4 * lk + r;
            const float v = A2[m * sH + n0 + li] > 0.0f ? acc[r] : 0.0f;
            DZ[m * sH + n0 + li] = v;
            if (m < rows)
                out.dz2[(size_t)(m0 + m) * kH + n0 + li] = v;
        }
    }
    __syncthreads();
    // ---- dZ1 = (dZ2 W2) where A1 > 0 ----
    if (wave < 4) {
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int q = 0; q < kSteps2; ++q)
            acc = mma(DZ[li * sH + 4 * q + lk], b2w[q], acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 4 * lk + r;
            if (m < rows)
                out.dz1[(size_t)(m0 + m) * kH + n0 + li] = A1[m * sH + n0 + li] > 0.0f ? acc[r] : 0.0f;
        }
    }
}

// Weight and bias gradients of the three layers, dW = dZ^T A and db = the
// column sums of dZ (dZ^T times a column of ones), one 16 x 16 tile of one dW
// per workgroup: 33 x 4 tiles of dW1, 4 x 4 of dW2, 4 x 5 of dW3.  The eight
// wavefronts take every eighth group of four rows, and their sums meet in LDS
// in a fixed order.  The first workgroup adds up the loss.
constexpr int kTiles1 = ((kIn + 15) / 16) * (kH / 16), kTiles2 = (kH / 16) * (kH / 16),
              kTiles3 = (kH / 16) * ((kOut + 15) / 16);
constexpr int kGradWaves = 8;
__global__ __launch_bounds__(kGradWaves * 64) void k_wgrad(RowArrays in, const float *__restrict__ x, int B,
                                                           float *__restrict__ grad, float *__restrict__ loss)
{
    __shared__ float s_w[kGradWaves][256], s_b[kGradWaves][16];
    __shared__ double s_loss[kGradWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const float *dz, *act;
    int tile = blockIdx.x, M, N, ow, ob;
    if (tile < kTiles1) {
        dz = in.dz1;
        act = x;
        M = kH;
        N = kIn;
        ow = oW1;
        ob = ob1;
    } else if (tile < kTiles1 + kTiles2) {
        tile -= kTiles1;
        dz = in.dz2;
        act = in.a1;
        M = kH;
        N = kH;
        ow = oW2;
        ob = ob2;
    } else {
        tile -= kTiles1 + kTiles2;
        dz = in.dy;
        act = in.a2;
        M = kOut;
        N = kH;
        ow = oW3;
        ob = ob3;
    }
    const int nt = (N + 15) / 16;
    const int m0 = tile / nt * 16, n0 = tile % nt * 16;
    const bool bias = n0 == 0;
    const int am = min(m0 + li, M - 1), bn = min(n0 + li, N - 1);  // (past the edge: not stored)
    floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f}, sum = {0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int U = 8;  // groups in flight
    for (int k0 = wave * 4; k0 < B; k0 += U * kGradWaves * 4) {
        float a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u * kGradWaves * 4 + lk;
            a[u] = k < B ? dz[(size_t)k * M + am] : 0.0f;
            b[u] = k < B ? act[(size_t)k * N + bn] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            acc = mma(a[u], b[u], acc);
        if (bias)
#pragma unroll
            for (int u = 0; u < U; ++u)
                sum = mma(a[u], 1.0f, sum);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        s_w[wave][(4 * lk + r) * 16 + li] = acc[r];
        if (li == 0)
            s_b[wave][4 * lk + r] = sum[r];
    }
    double l = 0.0;
    if (blockIdx.x == 0) {
        const int parts = (B + kRows - 1) / kRows;
        for (int q = tid; q < parts; q += kGradWaves * 64)
            l += in.loss[q];
#pragma unroll
        for (int h = 32; h > 0; h >>= 1)
            l += __shfl_xor(l, h, 64);
        if (lane == 0)
            s_loss[wave] = l;
    }
    __syncthreads();
    if (tid < 256) {
        const int m = m0 + tid / 16, n = n0 + tid % 16;
        float v = 0.0f;
#pragma unroll
        for (int q = 0; q < kGradWaves; ++q)
            v += s_w[q][tid];
        if (m < M && n < N)
            grad[ow + (size_t)m * N + n] = v;
    } else if (bias && tid < 256 + 16) {
        const int m = m0 + tid - 256;
        float v = 0.0f;
#pragma unroll
        for (int q = 0; q < kGradWaves; ++q)
            v += s_b[q][tid - 256];
        if (m < M)
            grad[ob + m] = v;
    }
    if (blockIdx.x == 0 && tid == 0) {
        double v = 0.0;
        for (int q = 0; q < kGradWaves; ++q)
            v += s_loss[q];
        *loss = (float)(v / (double)B);
    }
}

__global__ void k_step_inc(uint32_t *step)
{
    if (threadIdx.x == 0 && blockIdx.x == 0)
        *step += 1u;
}

__global__ __launch_bounds__(256) void k_adam(float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                                              uint16_t *__restrict__ wbf, const float *__restrict__ g,
                                              const uint32_t *__restrict__ step, float lr)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kP)
        return;
    const float t = (float)*step;
    const float gi = g[i];
    const float mi = kBeta1 * m[i] + (1.0f - kBeta1) * gi;
    const float vi = kBeta2 * v[i] + (1.0f - kBeta2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / (1.0f - powf(kBeta1, t));
    const float vh = vi / (1.0f - powf(kBeta2, t));
    const float wi = w[i] - lr * mh / (sqrtf(vh) + kEps);
    w[i] = wi;
    wbf[i] = f32_to_bf16(wi);
}

// Load: master from the caller, moments and step cleared, bf16 copy made.
__global__ __launch_bounds__(256) void k_load(float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                                              uint16_t *__restrict__ wbf, uint32_t *__restrict__ step)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0)
        *step = 0u;
    if (i >= kP)
        return;
    m[i] = 0.0f;
    v[i] = 0.0f;
    wbf[i] = f32_to_bf16(w[i]);
}

// ---------------------------------------------------------------------------
// Features: bounding box, 8^3 occupancy histogram over a cubic grid of edge
// (1 + 1e-4) max(E) / 8 from the box minimum (FP64, clamped), then
// f0 = (ln N - 11) / 2, f1..3 = ln(1 + E_a) / 2, f(4 + cell) =
// ln(1 + 64 count / N) (the logarithm tames the dense near-sensor cells of
// a spinning scan).
// ---------------------------------------------------------------------------
struct FeatScratch {
    uint32_t status;
    uint32_t bb[6];
    uint32_t pad;
    uint32_t counts[512];
};

__global__ void k_feat_reset(FeatScratch *fs)
{
    const int t = threadIdx.x;
    if (t == 0)
        fs->status = 0;
    if (t < 3) {
        fs->bb[t] = 0xffffffffu;
        fs->bb[3 + t] = 0u;
    }
    for (int c = t; c < 512; c += blockDim.x)
        fs->counts[c] = 0;
}

__global__ __launch_bounds__(kBlock) void k_feat_bbox(const float *__restrict__ xyz, int n, FeatScratch *fs)
{
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    bool bad = false;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float v = xyz[3 * (size_t)i + a];
            bad |= !isfinite(v);
            mn[a] = fminf(mn[a], v);
            mx[a] = fmaxf(mx[a], v);
        }
    }
    __shared__ float s_mn[3][kWavesPerBlock], s_mx[3][kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float lo = wave_min_f32(mn[a]), hi = wave_max_f32(mx[a]);
        if (lane == 0) {
            s_mn[a][w] = lo;
            s_mx[a][w] = hi;
        }
    }
    if (__any(bad) && lane == 0)
        atomicOr(&fs->status, 1u);
    __syncthreads();
    if (threadIdx.x < 3) {
        const int a = threadIdx.x;
        float lo = s_mn[a][0], hi = s_mx[a][0];
        for (int q = 1; q < kWavesPerBlock; ++q) {
            lo = fminf(lo, s_mn[a][q]);
            hi = fmaxf(hi, s_mx[a][q]);
        }
        if (lo <= hi) {
            atomicMin(&fs->bb[a], f2ord(lo));
            atomicMax(&fs->bb[3 + a], f2ord(hi));
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_feat_hist(const float *__restrict__ xyz, int n, FeatScratch *fs)
{
    __shared__ uint32_t h[512];
    for (int c = threadIdx.x; c < 512; c += blockDim.x)
        h[c] = 0;
    double lo[3], emax = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = (double)ord2f(fs->bb[a]);
        const double e = (double)ord2f(fs->bb[3 + a]) - lo[a];
        emax = e > emax ? e : emax;
    }
    const double edge = (emax > 0.0 && emax < INFINITY) ? (1.0 + 1e-4) * emax / 8.0 : 1.0;
    __syncthreads();
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        int b[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double q = floor(((double)xyz[3 * (size_t)i + a] - lo[a]) / edge);
            q = q > 0.0 ? q : 0.0;
            q = q < 7.0 ? q : 7.0;
            b[a] = (int)q;
        }
        atomicAdd(&h[(b[2] * 8 + b[1]) * 8 + b[0]], 1u);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < 512; c += blockDim.x)
        if (h[c])
            atomicAdd(&fs->counts[c], h[c]);
}

__global__ void k_feat_final(int n, const FeatScratch *__restrict__ fs, float *__restrict__ f)
{
    for (int t = threadIdx.x; t < kIn; t += blockDim.x) {
        double v;
        if (t == 0) {
            v = (log((double)n) - 11.0) / 2.0;
        } else if (t < 4) {
            const int a = t - 1;
            v = log1p((double)ord2f(fs->bb[3 + a]) - (double)ord2f(fs->bb[a])) / 2.0;
        } else {
            v = log1p(64.0 * (double)fs->counts[t - 4] / (double)n);
        }
        f[t] = fs->status ? __uint_as_float(0x7fc00000u) : (float)v;
    }
}

// Pick: the candidate with the lowest predicted log time, unless it does
// not beat the default candidate's prediction by `margin`.
__global__ void k_choose(const float *__restrict__ y, int default_cand, float margin, int32_t *__restrict__ choice)
{
    if (threadIdx.x != 0)
        return;
    int best = default_cand;
    float bv = y[default_cand];
    for (int k = 0; k < RFPS_MLP_CANDIDATES; ++k)
        if (y[k] < bv) {
            bv = y[k];
            best = k;
        }
    const float yd = y[default_cand];
    *choice = (isfinite(bv) && bv < yd - margin) ? best : default_cand;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
constexpr size_t kAlign = 256;
inline size_t up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

struct StateLayout {
    size_t master, m, v, wbf, step, total;
};
StateLayout state_layout()
{
    StateLayout L;
    L.master = 0;
    L.m = up(L.master + 4 * (size_t)kP);
    L.v = up(L.m + 4 * (size_t)kP);
    L.wbf = up(L.v + 4 * (size_t)kP);
    L.step = up(L.wbf + 2 * (size_t)kP);
    L.total = up(L.step + 4);
    return L;
}

State state_view(void *p)
{
    const StateLayout L = state_layout();
    unsigned char *b = static_cast<unsigned char *>(p);
    State s;
    s.master = reinterpret_cast<float *>(b + L.master);
    s.m = reinterpret_cast<float *>(b + L.m);
    s.v = reinterpret_cast<float *>(b + L.v);
    s.wbf = reinterpret_cast<uint16_t *>(b + L.wbf);
    s.step = reinterpret_cast<uint32_t *>(b + L.step);
    return s;
}

struct WsLayout {
    size_t feat, loss_parts, a1, a2, y, dy, dz2, dz1, grad, loss, total;
};
WsLayout ws_layout(int B)
{
    WsLayout L;
    size_t cur = 0;
    auto take = [&](size_t bytes) {
        const size_t o = up(cur);
        cur = o + bytes;
        return o;
    };
    const size_t b = (size_t)B;
    L.feat = take(sizeof(FeatScratch));
    L.loss_parts = take(4 * b * kH);  // a double per 16 rows; workspace sizes stay as they are
    L.a1 = take(4 * b * kH);
    take(4 * b * kH);  // not used
    L.a2 = take(4 * b * kH);
    L.y = take(4 * b * kOut);
    L.dy = take(4 * b * kOut);
    L.dz2 = take(4 * b * kH);
    L.dz1 = take(4 * b * kH);
    L.grad = take(4 * (size_t)kP);
    L.loss = take(4);
    L.total = up(cur);
    return L;
}

template <typename T>
T *at(void *ws, size_t off)
{
    return reinterpret_cast<T *>(static_cast<unsigned char *>(ws) + off);
}

// Forward pass of B rows.
void forward(const State &st, const float *x, int B, float *y, hipStream_t s)
{
    k_rows<false><<<(B + kRows - 1) / kRows, kRowsBlock, 0, s>>>(st.master, st.wbf, x, nullptr, nullptr, B, y,
                                                                 RowArrays{});
}

// Gradient of the loss with respect to the packed parameters into `grad`.
void backward(const State &st, const float *x, const float *t, const float *wt, int B, void *ws, const WsLayout &L,
              float *grad, float *loss, hipStream_t s)
{
    const RowArrays r = {at<float>(ws, L.a1),  at<float>(ws, L.a2),  at<float>(ws, L.dy),
                         at<float>(ws, L.dz2), at<float>(ws, L.dz1), at<double>(ws, L.loss_parts)};
    k_rows<true><<<(B + kRows - 1) / kRows, kRowsBlock, 0, s>>>(st.master, st.wbf, x, t, wt, B, nullptr, r);
    k_wgrad<<<kTiles1 + kTiles2 + kTiles3, kGradWaves * 64, 0, s>>>(r, x, B, grad, loss);
}

bool aligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) % kAlign) == 0; }

}  // namespace mlp
}  // namespace rfps

using namespace rfps::mlp;

extern "C" {

int32_t rfps_mlp_candidate(int32_t k, int32_t *n_vox, float *shell_spacing)
{
    if (k < 0 || k >= RFPS_MLP_CANDIDATES)
        return 1;
    if (n_vox)
        *n_vox = kNVox[k / 4];
    if (shell_spacing)
        *shell_spacing = kShell[k % 4];
    return 0;
}

size_t rfps_mlp_state_size(void) { return state_layout().total; }

size_t rfps_mlp_workspace_size(int32_t batch)
{
    if (batch < 1 || batch > kMaxRows)
        return 0;
    return ws_layout(batch).total;
}

static rfps_status check_state(const void *state, size_t bytes)
{
    if (!state || !aligned(state) || bytes < state_layout().total)
        return RFPS_ERR_WORKSPACE;
    return RFPS_OK;
}

static rfps_status check_ws(const void *ws, size_t bytes, int batch)
{
    if (batch < 1 || batch > kMaxRows)
        return RFPS_ERR_INVALID_ARG;
    if (!ws || !aligned(ws) || bytes < ws_layout(batch).total)
        return RFPS_ERR_WORKSPACE;
    return RFPS_OK;
}

static rfps_status launched(hipStream_t s)
{
    (void)s;
    return hipGetLastError() == hipSuccess ? RFPS_OK : RFPS_ERR_DEVICE;
}

rfps_status rfps_mlp_load(void *state, size_t state_bytes, const float *params, void *stream)
{
    rfps_status r = check_state(state, state_bytes);
    if (r != RFPS_OK)
        return r;
    if (!params)
        return RFPS_ERR_INVALID_ARG;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    State st = state_view(state);
    if (hipMemcpyAsync(st.master, params, 4 * (size_t)kP, hipMemcpyHostToDevice, s) != hipSuccess)
        return RFPS_ERR_DEVICE;
    k_load<<<(kP + 255) / 256, 256, 0, s>>>(st.master, st.m, st.v, st.wbf, st.step);
    if (launched(s) != RFPS_OK || hipStreamSynchronize(s) != hipSuccess)
        return RFPS_ERR_DEVICE;
    return RFPS_OK;
}

rfps_status rfps_mlp_save(const void *state, size_t state_bytes, float *params, void *stream)
{
    rfps_status r = check_state(state, state_bytes);
    if (r != RFPS_OK)
        return r;
    if (!params)
        return RFPS_ERR_INVALID_ARG;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    if (hipStreamSynchronize(s) != hipSuccess)
        return RFPS_ERR_DEVICE;
    State st = state_view(const_cast<void *>(state));
    if (hipMemcpy(params, st.master, 4 * (size_t)kP, hipMemcpyDeviceToHost) != hipSuccess)
        return RFPS_ERR_DEVICE;
    return RFPS_OK;
}

rfps_status rfps_mlp_features(const float *xyz, int32_t n, void *ws, size_t ws_bytes, float *feat, void *stream)
{
    if (!xyz || !feat || n < 1 || n > rfps::kMaxPoints)
        return RFPS_ERR_INVALID_ARG;
    rfps_status r = check_ws(ws, ws_bytes, 1);
    if (r != RFPS_OK)
        return r;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    FeatScratch *fs = at<FeatScratch>(ws, ws_layout(1).feat);
    const int blocks = std::min((n + 1023) / 1024, 512);
    k_feat_reset<<<1, 256, 0, s>>>(fs);
    k_feat_bbox<<<blocks, rfps::kBlock, 0, s>>>(xyz, n, fs);
    k_feat_hist<<<blocks, rfps::kBlock, 0, s>>>(xyz, n, fs);
    k_feat_final<<<1, 256, 0, s>>>(n, fs, feat);
    return launched(s);
}

rfps_status rfps_mlp_forward(const void *state, size_t state_bytes, const float *x, int32_t batch, void *ws,
                             size_t ws_bytes, float *y, void *stream)
{
    rfps_status r = check_state(state, state_bytes);
    if (r == RFPS_OK)
        r = check_ws(ws, ws_bytes, batch);
    if (r != RFPS_OK)
        return r;
    if (!x || !y)
        return RFPS_ERR_INVALID_ARG;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    forward(state_view(const_cast<void *>(state)), x, batch, y, s);
    return launched(s);
}

rfps_status rfps_mlp_gradient(const void *state, size_t state_bytes, const float *x, const float *t,
                              const float *w, int32_t batch, void *ws, size_t ws_bytes, float *grad, float *loss,
                              void *stream)
{
    rfps_status r = check_state(state, state_bytes);
    if (r == RFPS_OK)
        r = check_ws(ws, ws_bytes, batch);
    if (r != RFPS_OK)
        return r;
    if (!x || !t || !grad)
        return RFPS_ERR_INVALID_ARG;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const WsLayout L = ws_layout(batch);
    backward(state_view(const_cast<void *>(state)), x, t, w, batch, ws, L, grad, loss ? loss : at<float>(ws, L.loss),
             s);
    return launched(s);
}

rfps_status rfps_mlp_train_step(void *state, size_t state_bytes, const float *x, const float *t, const float *w,
                                int32_t batch, float lr, void *ws, size_t ws_bytes, float *loss, void *stream)
{
    rfps_status r = check_state(state, state_bytes);
    if (r == RFPS_OK)
        r = check_ws(ws, ws_bytes, batch);
    if (r != RFPS_OK)
        return r;
    if (!x || !t || !(lr > 0.0f) || !isfinite(lr))
        return RFPS_ERR_INVALID_ARG;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const WsLayout L = ws_layout(batch);
    const State st = state_view(state);
    float *grad = at<float>(ws, L.grad);
    backward(st, x, t, w, batch, ws, L, grad, loss ? loss : at<float>(ws, L.loss), s);
    k_step_inc<<<1, 64, 0, s>>>(st.step);
    k_adam<<<(kP + 255) / 256, 256, 0, s>>>(st.master, st.m, st.v, st.wbf, grad, st.step, lr);
    return launched(s);
}

rfps_status rfps_mlp_choose(const void *state, size_t state_bytes, const float *feat, int32_t default_cand,
                            float margin, void *ws, size_t ws_bytes, int32_t *choice, float *y, void *stream)
{
    rfps_status r = check_state(state, state_bytes);
    if (r == RFPS_OK)
        r = check_ws(ws, ws_bytes, 1);
    if (r != RFPS_OK)
        return r;
    if (!feat || !choice || default_cand < 0 || default_cand >= RFPS_MLP_CANDIDATES || !(margin >= 0.0f))
        return RFPS_ERR_INVALID_ARG;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const WsLayout L = ws_layout(1);
    float *out = y ? y : at<float>(ws, L.y);
    forward(state_view(const_cast<void *>(state)), feat, 1, out, s);
    k_choose<<<1, 64, 0, s>>>(out, default_cand, margin, choice);
    return launched(s);
}

}  // extern "C"
