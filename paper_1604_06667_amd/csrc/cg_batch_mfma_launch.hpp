// The persistent batch kernel and its launch for one data type; each type is
// instantiated in a source file of its own (cg_batch_mfma_<type>.hip).
#pragma once
#include "cg_mfma_tile.hpp"

namespace cg {

// Launch shapes of the persistent kernel (chosen by the autotuner):
// wavefronts per workgroup and 32-channel blocks per wavefront.
//   shape 0: 8 x 1 (256 channels per item)    shape 1: 8 x 2 (512)
//   shape 2: 4 x 1 (128)                      shape 3: 4 x 2 (256, two workgroups per CU)
// Two 16-sample steps per pipeline stage, as in the per-grid kernel (16 jobs:
// 3.2 ms with one step, 2.9 with two; shape 3), one for FP64 rows, whose
// second step spills (16 jobs 2.77 ms with two and 2.05 with one in shape 3,
// another 16 4.10 and 3.81).
// (4-wavefront workgroups are held to two wavefronts per SIMD, so that two
// of them share a compute unit and cover each other's barrier waits.  Shape 0
// with 16-bit rows is held to four: it spills 27 to 62 registers for it, at
// even times (five batches 1.05, 2.22, 0.91, 0.94 and 3.22 ms against 1.10,
// 2.05, 0.97, 0.83 and 3.25); FP32 rows take 2.74 ms with the bound and 2.11
// without, FP64 rows 4.08 and 2.61)
template <int NW, int BPW, int KT, bool SHORT, int MODE, typename T>
__global__ void __launch_bounds__(NW * 64, NW == 4 ? 2 : BPW == 1 && sizeof(T) == 2 ? 4 : 1) k_batch_mfma(
    const BatchJob* __restrict__ jobs, const BatchItem* __restrict__ items, BatchQueues q,
    int* counter, BatchRanges br, const T* __restrict__ zrow) {
  __shared__ int64_t s_item;
  const int home = (int)(blockIdx.x % kNumXcd);
  int visited = 0;   // queues found empty so far (thread 0): home, home + 1, ...
  for (;;) {
    __syncthreads();  // the previous item is done with LDS
    if (threadIdx.x == 0) {
      int64_t next = -1;
      while (visited < kNumXcd) {
        const int k = (home + visited) % kNumXcd;
        const int64_t i = atomicAdd(&counter[k], 1);
        if (i < q.off[k + 1] - q.off[k]) {
          next = q.off[k] + i;
          break;
        }
        ++visited;   // every counter only grows, so an exhausted queue stays so
      }
      s_item = next;
    }
    __syncthreads();
    const int64_t it = s_item;
    if (it < 0) break;
    const BatchItem item = items[it];
    const BatchJob& jb = jobs[item.job];   // global memory, not a kernel argument
    TileView tv;
    tv.txyz = jb.txyz;
    tv.tll = jb.tll;
    tv.rng = br.ranges + 2 * jb.rbase;
    tv.roff = jb.range_off;
    tv.nr = br.nranges + jb.toff;
    tv.ntot = br.ncand + jb.toff;
    tv.nslots = jb.nslots;
    tv.ntiles = jb.ntiles;
    tv.ntx = jb.ntx;   // same candidate order as the per-grid kernel
    tv.srec = br.srec;
    OutView ov;
    ov.S = nullptr;
    ov.W = nullptr;
    ov.Wn = nullptr;
    ov.cube = jb.cube;
    ov.wout = jb.wout;
    ov.slot_target = jb.slot_target;
    ov.ntarget = jb.ntarget;
    ov.cst = jb.cst;
    ov.tst = jb.tst;
    ov.mode = ACC_FINAL;
    constexpr int KS = sizeof(T) == 8 ? 1 : 2;
    mfma_tile<NW, BPW, KT, SHORT, MODE, false, T, KS, true>(tv, jb.kp, (const T*)jb.data, zrow,
                                                            jb.ld, jb.nchan, ov, item.tile,
                                                            item.c0, item.cend);
  }
}

template <int NW, int BPW, int KT, bool SHORT, int MODE, typename T>
static int occ_of() {
  int occ = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_batch_mfma<NW, BPW, KT, SHORT, MODE, T>, NW * 64,
                                                   0) != hipSuccess)
    return 0;
  return occ;
}

template <int NW, int BPW, int KT, bool SHORT, int MODE, typename T>
static hipError_t launch_bt(const BatchJob* jobs, const BatchItem* items, const BatchQueues& q,
                            int* counter, const BatchRanges& br, const void* zrow,
                            int blocks_per_cu, hipStream_t st) {
  const int64_t nitems = q.off[kNumXcd];
  int dev = 0, ncu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const int occ = occ_of<NW, BPW, KT, SHORT, MODE, T>();
  int per = blocks_per_cu > 0 && blocks_per_cu < occ ? blocks_per_cu : occ;
  if (per < 1) per = 1;
  int64_t grid = (int64_t)ncu * per;
  if (grid > nitems) grid = nitems;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL((k_batch_mfma<NW, BPW, KT, SHORT, MODE, T>), dim3((unsigned)grid), dim3(NW * 64), 0, st,
                     jobs, items, q, counter, br, (const T*)zrow);
  return hipGetLastError();
}

// One launch shape for the kernel forms of the batch's jobs (BatchForm).
#define CG_BATCH_FORMS(CALL, NW_, BPW_)                              \
  (form == BATCH_SHORT_CIRCULAR ? CALL<NW_, BPW_, 0, true, MODE, T>  \
   : form == BATCH_SHORT        ? CALL<NW_, BPW_, 2, true, MODE, T>  \
                                : CALL<NW_, BPW_, 2, false, MODE, T>)
template <int MODE, typename T>
static hipError_t launch_bs(int shape, int form, const BatchJob* jobs, const BatchItem* items,
                            const BatchQueues& q, int* counter, const BatchRanges& br,
                            const void* zrow, int blocks_per_cu, hipStream_t st) {
#define CG_BT(NW_, BPW_) \
  CG_BATCH_FORMS(launch_bt, NW_, BPW_)(jobs, items, q, counter, br, zrow, blocks_per_cu, st)
  switch (shape) {
    case 0: return CG_BT(8, 1);
    case 1: return CG_BT(8, 2);
    case 2: return CG_BT(4, 1);
    case 3: return CG_BT(4, 2);
    default: return hipErrorInvalidValue;
  }
#undef CG_BT
}

template <int MODE, typename T>
static int occ_s(int shape, int form) {
  switch (shape) {
    case 0: return CG_BATCH_FORMS(occ_of, 8, 1)();
    case 1: return CG_BATCH_FORMS(occ_of, 8, 2)();
    case 2: return CG_BATCH_FORMS(occ_of, 4, 1)();
    case 3: return CG_BATCH_FORMS(occ_of, 4, 2)();
    default: return 0;
  }
}
#undef CG_BATCH_FORMS

template <typename T>
hipError_t launch_batch_mfma_t(const BatchJob* jobs, const BatchItem* items, const BatchQueues& q,
                               int* counter, const BatchRanges& br, const void* zrow, int prec,
                               int shape, int form, int blocks_per_cu, hipStream_t st) {
  if (prec == 2)
    return launch_bs<1, T>(shape, form, jobs, items, q, counter, br, zrow, blocks_per_cu, st);
  return launch_bs<0, T>(shape, form, jobs, items, q, counter, br, zrow, blocks_per_cu, st);
}

template <typename T>
int batch_max_blocks_per_cu_t(int prec, int shape, int form) {
  return prec == 2 ? occ_s<1, T>(shape, form) : occ_s<0, T>(shape, form);
}

}  // namespace cg
