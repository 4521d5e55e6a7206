// The fused 1D kernels at order 4 (at_wave1d.h).
#include "at_wave1d.h"

namespace atk {

hipError_t launch_wave1d_o4(const Step1D &a, bool linear, bool fma, int ppt, int nw, int64_t nblocks,
                            size_t lds, hipStream_t st)
{
    return launch_wave1d_order<4>(a, linear, fma, ppt, nw, nblocks, lds, st);
}

hipError_t launch_wave1d_batch_o4(const Step1D *descs, const int2 *tbl, int64_t nblocks,
                                  bool linear, bool fma, int ppt, int64_t n0, int flip,
                                  size_t lds, hipStream_t st)
{
    return launch_wave1d_batch_order<4>(descs, tbl, nblocks, linear, fma, ppt, n0, flip, lds, st);
}

}  // namespace atk
