// kernels_batch_grid.hip -- the batched two-step shape of 32 x 8 tiles.  It runs
// the arithmetic of the single-grid shape tile2x32x8, so an item agrees with a
// run of its own to the bit after any even number of steps.
#include "batch2.h"

namespace sclbm {

template <typename T>
hipError_t launch_batch_grid(const BatchItem<T>* items, const int2* work, int nwork, int parity, const StepArgs<T>& common,
                             hipStream_t s)
{
    hipLaunchKernelGGL((k_d2q9_batch2<T, GridNode, 32, 8, 256>), dim3(nwork), dim3(256), 0, s, items, work, parity,
                       common);
    return hipGetLastError();
}
template hipError_t launch_batch_grid<float>(const BatchItem<float>*, const int2*, int, int, const StepArgs<float>&,
                                             hipStream_t);
template hipError_t launch_batch_grid<double>(const BatchItem<double>*, const int2*, int, int,
                                              const StepArgs<double>&, hipStream_t);

}  // namespace sclbm
