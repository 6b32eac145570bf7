// The FP-safe form of the spherical pruning bound (Sec. 3.4.2, eq.
// radius_pruning_condition and eq. radius_pruning_correctness), shared by
// the GPU samplers and the CPU sampler of librfps: one definition, compiled
// for the device by hipcc and for the host by any C++ compiler.
//
// A tile with enclosing radius R (rounded up) and tile distance dv (the
// largest Dist_p of its members) is skipped for sample s when the FP32 value
// q = fl32(||s - c||^2), computed with the point-distance formula
// ((dx*dx + dy*dy) + dz*dz), satisfies q >= thr(R, dv).  Why that is safe
// (u = 2^-24, the unit roundoff of FP32):
//   - the formula rounds five times along any path (a subtraction that
//     enters squared, one product, two sums), so q lies within a factor
//     (1 +- u)^5 of the exact squared distance, barring underflow;
//   - thr >= (R + sqrt(dv / (1 - 2^-20)))^2 (1 + 2^-20) (shown below), and
//     (1 + 2^-20) >= (1 + u)^5, so q >= thr gives
//     ||s - c|| >= R + sqrt(dv / (1 - 2^-20));
//   - by the triangle inequality (eq. triangle_inequality_bound) every
//     member p then has ||p - s||^2 >= dv / (1 - 2^-20);
//   - its FP32 squared distance is at least (1 - u)^5 ||p - s||^2 >= dv,
//     since (1 - u)^5 >= 1 - 2^-20, so it is >= dv >= Dist_p[p] and the
//     strict update cannot fire.
// The threshold is evaluated in FP32, each step rounded to nearest:
//   a = fl(dv * k1), k1 = 1 + 2^-20 + 2^-22: a >= dv k1 (1 - u) >= dv / (1 - 2^-20);
//   b = sqrt(a), within one unit in the last place: b >= sqrt(a) (1 - 2u);
//   t = fl(R + b) >= (R + sqrt(a)) (1 - 2u) (1 - u);
//   thr = fl(fl(t * t) * k2) >= (R + sqrt(a))^2 (1 - 2u)^2 (1 - u)^4 k2, and
//   k2 = 1 + 2^-19 >= (1 + 2^-20) / ((1 - 2u)^2 (1 - u)^4).
// dv == 0 means no member can decrease (thr = 0 always skips); dv below
// 2^-100 or above 2^100, or a square beyond the FP32 range, gives NaN, which
// never skips and keeps the bound clear of subnormals and overflow.
#pragma once

#include <math.h>
#include <stdint.h>
#include <string.h>

#if defined(__HIP__)
#define RFPS_HOST_DEVICE __host__ __device__
#else
#define RFPS_HOST_DEVICE
#endif

namespace rfps {

// Margins of the production bound: the factor on dv before the root and the
// factor on the square (both exact in FP32).
constexpr float kPruneInner = 1.0f + 0x1p-20f + 0x1p-22f;
constexpr float kPruneOuter = 1.0f + 0x1p-19f;

RFPS_HOST_DEVICE inline float prune_nan()
{
    const uint32_t u = 0x7fc00000u;
    float f;
    memcpy(&f, &u, 4);
    return f;
}

// The bound with explicit margins (the production ones are the defaults of
// prune_threshold below); a margin of exactly 1 removes that safeguard.
RFPS_HOST_DEVICE inline float prune_threshold_with(float R, float dv, float inner, float outer)
{
    if (dv == 0.0f)
        return 0.0f;
    if (!(dv >= 0x1p-100f) || !(dv <= 0x1p100f))
        return prune_nan();
    const float a = dv * inner;
    const float t = R + sqrtf(a);
    const float t2 = t * t;
    if (!(t2 <= 3.0e38f))
        return prune_nan();
    return t2 * outer;
}

RFPS_HOST_DEVICE inline float prune_threshold(float R, float dv)
{
    return prune_threshold_with(R, dv, kPruneInner, kPruneOuter);
}

// Distance filter on the matrix cores.  The samplers test many points s
// against many points p with one matrix product: with both shifted by a
// common origin, fl(x - o),
//   D = col(|s|^2) - 2 p.s - row(limit, |p|^2)
// (a 4-long dot product and its addend, FP32), and the pair is kept for the
// exact FP32 work iff !(D >= 0).  A kept pair costs work; a dropped one must
// be one whose formula distance ((dx*dx + dy*dy) + dz*dz) is not below
// `limit`.  Why that is so (u = 2^-24, a = |p|, b = |s| of the shifted
// points, r the true distance):
//   - the shift moves each point by at most u a and u b, so the squared
//     distance of the shifted points is at most r^2 + 2.01 u (a + b)^2, and
//     the formula distance is at least r^2 (1 - 5.1 u);
//   - |s|^2 and col() round four times (4 u b^2), row() errs by at most
//     6 u a^2 + 3 u limit, and the product's nine operations err by at most
//     2 u each, truncation included, of partial sums below
//     b^2 + 2 a b + a^2 + limit (18 u times that);
//   - with (a + b)^2 <= 2 (a^2 + b^2) and 2 a b <= a^2 + b^2 these add up to
//     less than 63 u (a^2 + b^2) + 27 u limit, and the two sides give
//     2^-17 (a^2 + b^2) = 128 u (a^2 + b^2) and 2^-19 limit = 32 u limit away.
// A limit or square beyond 1e36 (overflow, or NaN: "never skip") keeps every
// pair; 1e-36 keeps the comparison clear of subnormals.
constexpr float kFilterNorm = 1.0f - 0x1p-17f;
constexpr float kFilterLimit = 1.0f + 0x1p-19f;

RFPS_HOST_DEVICE inline float filter_col(float n2)
{
    return n2 <= 1e36f ? n2 * kFilterNorm : -INFINITY;
}

RFPS_HOST_DEVICE inline float filter_row(float limit, float n2)
{
    if (!(limit <= 1e36f) || !(n2 <= 1e36f))
        return INFINITY;
    const float a = limit * kFilterLimit;
    const float b = n2 * kFilterNorm;
    const float t = a - b;
    return t + 1e-36f;
}

// Whether the filter's margin around a candidate at squared distance n2 from
// the origin spans a good part of what j selections at squared distances near
// d cover, so that pairs of listed candidates (100 or so, spread over the
// cloud) are kept without being near: the margin is 2^-16 n2, on a surface j
// selections cover an area of about j d, and a list of 128 then keeps one
// false pair a row from 2^-9 n2 = j d on.  (Unlikely clouds: one that fills
// its box has n2 below j d.  NaN and overflow count as too far.)
RFPS_HOST_DEVICE inline bool filter_blurred(float n2, float d, int j)
{
    return !(n2 * 0x1p-9f <= (float)j * d);
}

}  // namespace rfps
