// Persistent batch contraction kernels of float64 data.
#include "cg_batch_mfma_launch.hpp"

namespace cg {

template hipError_t launch_batch_mfma_t<double>(const BatchJob*, const BatchItem*, const BatchQueues&, int*,
                                             const BatchRanges&, const void*, int, int, int, int,
                                             hipStream_t);
template int batch_max_blocks_per_cu_t<double>(int, int, int);

}  // namespace cg
