// Host build of the multi-pick sampler's distance filter (prune_bound.h) and
// of its capacity and layout rules (round_layout.h) for the CPU tests.
#include <cfenv>

#include "../../paper_2606_06255_amd/csrc/round_layout.h"

namespace {

float sqdist(const float *a, const float *b)
{
    volatile float x = a[0] - b[0], y = a[1] - b[1], z = a[2] - b[2];
    volatile float xx = x * x, yy = y * y, zz = z * z;
    volatile float s = xx + yy;
    return s + zz;
}

float norm2(const volatile float *a)
{
    volatile float xx = a[0] * a[0], yy = a[1] * a[1], zz = a[2] * a[2];
    volatile float s = xx + yy;
    return s + zz;
}

}  // namespace

// keep[i]: the filter keeps pair (s_i, p_i) with limit[i], the product formed
// in the given way (0: nearest, 1: every operation towards zero, 2: nearest,
// in the opposite order, 3: exact up to the last rounding); d[i]: the FP32
// formula distance.
extern "C" void shim_filter(int n, const float *s, const float *p, const float *o, const float *limit, int way,
                            unsigned char *keep, float *d)
{
    for (int i = 0; i < n; ++i) {
        d[i] = sqdist(s + 3 * i, p + 3 * i);
        volatile float a[3], b[3];
        for (int c = 0; c < 3; ++c) {
            b[c] = s[3 * i + c] - o[c];
            a[c] = p[3 * i + c] - o[c];
        }
        const volatile float col = rfps::filter_col(norm2(b));
        const volatile float row = -rfps::filter_row(limit[i], norm2(a));
        volatile float acc = row;
        if (way == 3) {
            double e = (double)row + (double)col;
            for (int c = 0; c < 3; ++c)
                e += -2.0 * (double)a[c] * (double)b[c];
            acc = (float)e;
        } else {
            std::fesetround(way == 1 ? FE_TOWARDZERO : FE_TONEAREST);
            const float term[4] = {1.0f, 1.0f, 1.0f, 1.0f};
            for (int k = 0; k < 4; ++k) {
                const int c = way == 2 ? 3 - k : k;
                volatile float t;
                if (c == 3) {
                    t = term[c] * col;
                } else {
                    volatile float m = -2.0f * a[c];
                    t = m * b[c];
                }
                acc = acc + t;
            }
            std::fesetround(FE_TONEAREST);
        }
        keep[i] = !(acc >= 0.0f);
    }
}

extern "C" unsigned shim_budget(unsigned max_lds) { return rfps::rounds_budget(max_lds); }
extern "C" unsigned shim_dynamic(unsigned max_lds) { return rfps::rounds_dynamic(max_lds); }
extern "C" int shim_granted(unsigned tiles, unsigned pts, unsigned G, unsigned R, unsigned budget)
{
    return rfps::share_granted(tiles, pts, G, R, budget);
}
extern "C" unsigned shim_need(unsigned tiles, unsigned pts) { return rfps::rounds_lds_need(tiles, pts); }
