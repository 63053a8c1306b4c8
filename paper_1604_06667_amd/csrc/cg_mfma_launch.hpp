// The per-grid matrix-core kernel and its launch for one data type; each type
// is instantiated in a source file of its own (cg_mfma_<type>.hip).
#pragma once
#include "cg_mfma_tile.hpp"

namespace cg {

// One block of accumulators per wavefront leaves room for four wavefronts on a
// SIMD: without the bound some data types took a few registers too many, and
// 11.8 ms became 15.7 on the sight lines in FP16.
template <int NW, int BPW, int KT, bool SHORT, int MODE, bool FULL, typename T, int KS>
__global__ void __launch_bounds__(NW * 64, BPW == 1 ? 4 : 1) k_gather_mfma(TileView tv, KernelParams kp,
                                                         const T* __restrict__ data,
                                                         const T* __restrict__ zrow, int64_t ld,
                                                         int64_t nchan, OutView ov) {
  constexpr int CP = NW * BPW * 32;
  int64_t tile, pass;
  work_of_block(blockIdx.x, tv.ntiles, (nchan + CP - 1) / CP, &tile, &pass);
  if (tv.ntx > 0) tile = strip_tile(tile, tv.ntiles, tv.ntx);
  const int64_t c0 = pass * CP;
  const int64_t cend = c0 + CP < nchan ? c0 + CP : nchan;
  mfma_tile<NW, BPW, KT, SHORT, MODE, FULL, T, KS>(tv, kp, data, zrow, ld, nchan, ov, tile, c0, cend);
}

template <int NW, int BPW, int MODE, typename T, int KS>
static void launch_cfg(const TileView& tv, const KernelParams& kp, const void* data,
                       const void* zrow, int64_t ld, int64_t nchan, const OutView& ov,
                       hipStream_t st) {
  constexpr int CP = NW * BPW * 32;
  const bool full = nchan % CP == 0;
  // Elliptical kernels of long supports, BF16 mode, more than 512 channels but
  // no multiple of 1024: four blocks of accumulators, the bounds of a ragged
  // range and the call for long chords leave 37 to 106 registers spilled in
  // the loop, two blocks none, which pays for the weights' being formed twice
  // (120,000 samples x 1000 channels onto 200 x 200: BF16 rows 1125 us with
  // four and 449 with two, FP16 620 and 477, FP32 712 and 502; 43,200 x 600:
  // 277 and 217, 222 and 225, 238 and 222).  Whole multiples of 1024 spill
  // 23 and are the faster so (BF16 rows 157 and 191 us, 30,000 samples).
  constexpr bool RAGGED2 = BPW == 4 && MODE == 0 && sizeof(T) <= 4;
  if constexpr (RAGGED2) {
    if (!full && kp.type == 1 && !short_support(kp))
      return launch_cfg<8, 2, MODE, T, 2>(tv, kp, data, zrow, ld, nchan, ov, st);
  }
  const int64_t npass = (nchan + CP - 1) / CP;
  const dim3 g((unsigned)(tv.ntiles * npass)), b(NW * 64);
  const T* d = (const T*)data;
  const T* z = (const T*)zrow;
  const bool sh = short_support(kp);
#define CG_MFMA_LAUNCH(KT_, SH_)                                                                \
  do {                                                                                          \
    if (full)                                                                                   \
      hipLaunchKernelGGL((k_gather_mfma<NW, BPW, KT_, SH_, MODE, true, T, KS>), g, b, 0, st, tv, kp, \
                         d, z, ld, nchan, ov);                                                  \
    else if constexpr (!(RAGGED2 && KT_ == 1 && !SH_))                                          \
      hipLaunchKernelGGL((k_gather_mfma<NW, BPW, KT_, SH_, MODE, false, T, KS>), g, b, 0, st, tv, kp, \
                         d, z, ld, nchan, ov);                                                  \
  } while (0)
  if (sinc_by_series(kp)) CG_MFMA_LAUNCH(4, true);
  else if (kp.type >= 2 && sh) CG_MFMA_LAUNCH(3, true);
  else if (kp.type >= 2) CG_MFMA_LAUNCH(3, false);
  else if (kp.type == 0 && sh) CG_MFMA_LAUNCH(0, true);
  else if (kp.type == 0) CG_MFMA_LAUNCH(0, false);
  else if (sh) CG_MFMA_LAUNCH(1, true);
  else CG_MFMA_LAUNCH(1, false);
#undef CG_MFMA_LAUNCH
}

template <int MODE, typename T>
static void launch_dt(const TileView& tv, const KernelParams& kp, const void* data,
                      const void* zrow, int64_t ld, int64_t nchan, const OutView& ov,
                      hipStream_t st) {
  // KS: 16-sample MFMA steps per pipeline stage.  Two per stage (32 candidates
  // a barrier, more loads in flight) pay off up to 512 channels per workgroup;
  // four blocks of accumulators leave no registers for it, and four steps
  // cost more occupancy than they save (100 / 200 channels of 400,000 samples
  // onto 350 x 300: 1 step 352 / 423 us, 2 steps 296 / 374, 4 steps 305 / 463).
  // Up to 64 channels a workgroup of four wavefronts still beats two, although
  // half of them have no channels: they share the weights (48 channels: 283
  // us against 331 with two wavefronts and one step, 344 with two steps).
  // FP64 rows take one step per stage up to 256 channels: within the 128
  // registers of four wavefronts on a SIMD two steps spill in every kernel
  // but the circular Gaussian of short supports (120,000 samples x 200
  // channels onto 200 x 200, elliptical: 227 us against 427; x 100, FP16: 167
  // against 222; the largest loss is 10 %, at 256 channels of BF16 mode).
  constexpr int KS = sizeof(T) == 8 ? 1 : 2;
  if (nchan <= 128) launch_cfg<4, 1, MODE, T, KS>(tv, kp, data, zrow, ld, nchan, ov, st);
  else if (nchan <= 256) launch_cfg<8, 1, MODE, T, KS>(tv, kp, data, zrow, ld, nchan, ov, st);
  else if (nchan <= 512) launch_cfg<8, 2, MODE, T, 2>(tv, kp, data, zrow, ld, nchan, ov, st);
  else launch_cfg<8, 4, MODE, T, 1>(tv, kp, data, zrow, ld, nchan, ov, st);
}

template <typename T>
hipError_t launch_gather_mfma_t(const TileView& tv, const KernelParams& kp, const void* data,
                                const void* zrow, int64_t ld, int64_t nchan, int prec,
                                const OutView& ov, hipStream_t st) {
  if (prec == 2) launch_dt<1, T>(tv, kp, data, zrow, ld, nchan, ov, st);
  else launch_dt<0, T>(tv, kp, data, zrow, ld, nchan, ov, st);
  return hipGetLastError();
}

}  // namespace cg
