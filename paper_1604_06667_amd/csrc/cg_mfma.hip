// Matrix-core (MFMA) contraction for many-channel cubes.
//
// For one tile of 64 targets, Eq. (1) over a chunk of candidate samples
// is a dense product S[c][t] += sum_k R[k][c] w[t][k] (the paper's remark
// that all channels of a spectrum share one weight, Sect. 5, is what makes
// it a GEMM).  The weight block w[64][16 KS] of a chunk of KS 16-sample steps
// is computed once (FP64 support test and distance, FP32 kernel value, rounded
// to BF16/FP16) and shared by all channel blocks; each lane loads the data
// values of its own operand of v_mfma_f32_32x32x16_{bf16,f16} (channels as M,
// targets as N, samples as K) and converts them to BF16/FP16 in registers.
// Accumulation is FP32 in the matrix cores.  In BF16 mode data and weights are each split into a BF16 high part and a BF16 residual and the
// block is formed from three products (hi*hi + lo*hi + hi*lo); a single
// BF16 product would round data and weights to 2^-9, which is too coarse
// for the 2e-3 bound on noise-dominated channels.  Two weight sums are kept
// in FP64: W of the unrounded weights (the weight map) and W' of the weights
// as they entered the products, which normalises the cube so that a
// constant field stays exactly constant.
#include "cg_internal.hpp"

namespace cg {

bool mfma_available() { return true; }

template <typename T>
hipError_t launch_gather_mfma_t(const TileView& tv, const KernelParams& kp, const void* data,
                                const void* zrow, int64_t ld, int64_t nchan, int prec,
                                const OutView& ov, hipStream_t st);
extern template hipError_t launch_gather_mfma_t<double>(const TileView&, const KernelParams&, const void*,
                                                        const void*, int64_t, int64_t, int,
                                                        const OutView&, hipStream_t);
extern template hipError_t launch_gather_mfma_t<float>(const TileView&, const KernelParams&, const void*,
                                                       const void*, int64_t, int64_t, int,
                                                       const OutView&, hipStream_t);
extern template hipError_t launch_gather_mfma_t<_Float16>(const TileView&, const KernelParams&, const void*,
                                                          const void*, int64_t, int64_t, int,
                                                          const OutView&, hipStream_t);
extern template hipError_t launch_gather_mfma_t<uint16_t>(const TileView&, const KernelParams&, const void*,
                                                          const void*, int64_t, int64_t, int,
                                                          const OutView&, hipStream_t);

hipError_t launch_gather_mfma(const TileView& tv, const KernelParams& kp, const void* data,
                              const void* zrow, int dtype, int64_t ld, int64_t nchan, int prec,
                              const OutView& ov, hipStream_t st) {
  if (tv.ntiles <= 0) return hipSuccess;
  switch (dtype) {
    case 0: return launch_gather_mfma_t<double>(tv, kp, data, zrow, ld, nchan, prec, ov, st);
    case 1: return launch_gather_mfma_t<float>(tv, kp, data, zrow, ld, nchan, prec, ov, st);
    case 2: return launch_gather_mfma_t<_Float16>(tv, kp, data, zrow, ld, nchan, prec, ov, st);
    default: return launch_gather_mfma_t<uint16_t>(tv, kp, data, zrow, ld, nchan, prec, ov, st);
  }
}

}  // namespace cg
