// Small clouds: the whole sampling call in one workgroup (solo_cloud.h).
#include "solo_cloud.h"

namespace rfps {

template <bool E>
__global__ __launch_bounds__(kSoloWaves *kWave) void k_rfps_solo(IndexHeader *hdr, SoloJob job)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const bool failed = hdr->build_status != 0;
    if (tid == 0) {
        hdr->sample_status = 0;
        hdr->last_m = (uint32_t)job.m;
        hdr->trace_n = 0;
    }
    if (tid < kTeleFields)
        hdr->tele[tid] = 0;
    if (failed) {
        for (int i = tid; i < job.m; i += kSoloWaves * kWave) {
            job.out_idx[i] = -1;
            if (job.out_d2)
                job.out_d2[i] = __uint_as_float(0x7fc00000u);
        }
        return;
    }
    if (tid == 0) {
        job.out_idx[0] = job.start;
        if (job.out_d2)
            job.out_d2[0] = INFINITY;
    }
    solo_any<E>(job, smem);
}

hipError_t launch_rfps_solo(const IndexView &v, int m, int start, bool euclid, int32_t *out_idx, float *out_d2,
                            hipStream_t s)
{
    SoloJob job = {v.xs, v.ys, v.zs, v.inv, v.n, m, start, out_idx, out_d2};
    const uint32_t lds = solo_lds((uint32_t)v.n);
    const void *fn = euclid ? reinterpret_cast<const void *>(k_rfps_solo<true>)
                            : reinterpret_cast<const void *>(k_rfps_solo<false>);
    IndexHeader *hdr = v.hdr;
    void *args[] = {&hdr, &job};
    return hipLaunchKernel(fn, dim3(1), dim3(kSoloWaves * kWave), args, lds, s);
}

}  // namespace rfps
