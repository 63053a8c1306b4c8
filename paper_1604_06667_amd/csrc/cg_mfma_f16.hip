// Matrix-core contraction kernels of float16 data.
#include "cg_mfma_launch.hpp"

namespace cg {

template hipError_t launch_gather_mfma_t<_Float16>(const TileView&, const KernelParams&, const void*, const void*,
                                              int64_t, int64_t, int, const OutView&, hipStream_t);

}  // namespace cg
