// The fused 1D kernels at order 2 (at_wave1d.h) and their launchers.
#include "at_wave1d.h"

namespace atk {

hipError_t launch_wave1d_o4(const Step1D &a, bool linear, bool fma, int ppt, int nw, int64_t nblocks,
                            size_t lds, hipStream_t st);
hipError_t launch_wave1d_batch_o4(const Step1D *descs, const int2 *tbl, int64_t nblocks,
                                  bool linear, bool fma, int ppt, int64_t n0, int flip,
                                  size_t lds, hipStream_t st);

// LDS of one wave: the stage part, the history of D + 1 levels (twice) of the
// 2 NT faces and a spare place, and the delays of s + 2 steps
size_t wave1d_lds_bytes(int order, int s, int NT, int D, int ppt, int nw)
{
    return 8 * ((size_t)wave_stage_doubles(ppt, nw) + (size_t)(D + 1) * (2 * NT + 1) * order) +
           ((size_t)(s + 2) * NT * 2 + 7) / 8 * 8;
}

hipError_t launch_wave1d(const Step1D &a, int order, bool linear, bool fma, int ppt, int nw,
                         int64_t nblocks, hipStream_t st)
{
    const size_t lds = wave1d_lds_bytes(order, a.s, a.NT, a.D, ppt, nw);
    if (order == 4) return launch_wave1d_o4(a, linear, fma, ppt, nw, nblocks, lds, st);
    return launch_wave1d_order<2>(a, linear, fma, ppt, nw, nblocks, lds, st);
}

hipError_t launch_wave1d_batch(const Step1D *descs, const int2 *tbl, int64_t nblocks, int order,
                               bool linear, bool fma, int ppt, int64_t n0, int flip, size_t lds,
                               hipStream_t st)
{
    if (order == 4)
        return launch_wave1d_batch_o4(descs, tbl, nblocks, linear, fma, ppt, n0, flip, lds, st);
    return launch_wave1d_batch_order<2>(descs, tbl, nblocks, linear, fma, ppt, n0, flip, lds, st);
}

}  // namespace atk
