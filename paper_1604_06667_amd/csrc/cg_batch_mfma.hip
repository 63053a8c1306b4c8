// Persistent matrix-core contraction for a batch of gridding jobs.
//
// Every (job, tile, channel range) of the batch is one work item.  The
// items sit in one queue per XCD: each job's tiles are split into one run
// of neighbouring tiles per XCD, and every queue lists its runs of all jobs
// in order of estimated item cost, largest first (longest processing time
// first).  A grid sized to the resident capacity of the chip takes items
// one at a time from atomic counters: a workgroup drains the queue of its
// own XCD (block b runs on XCD b % 8), so tiles that share candidate rows
// and output lines meet in that XCD's L2, then takes what is left in the
// other queues in turn.  Jobs of very different sizes thus share one launch
// without a tail of idle compute units.
// Each item runs the same tile contraction as the per-grid kernel, with the
// kernel type (circular or elliptical) taken from the job at run time where
// the batch holds both, and writes the normalised cube and weights of its job
// directly.
#include "cg_internal.hpp"

namespace cg {

template <typename T>
hipError_t launch_batch_mfma_t(const BatchJob* jobs, const BatchItem* items, const BatchQueues& q,
                               int* counter, const BatchRanges& br, const void* zrow, int prec,
                               int shape, int form, int blocks_per_cu, hipStream_t st);
template <typename T>
int batch_max_blocks_per_cu_t(int prec, int shape, int form);
extern template hipError_t launch_batch_mfma_t<double>(const BatchJob*, const BatchItem*, const BatchQueues&,
                                                     int*, const BatchRanges&, const void*, int, int, int,
                                                     int, hipStream_t);
extern template int batch_max_blocks_per_cu_t<double>(int, int, int);
extern template hipError_t launch_batch_mfma_t<float>(const BatchJob*, const BatchItem*, const BatchQueues&,
                                                     int*, const BatchRanges&, const void*, int, int, int,
                                                     int, hipStream_t);
extern template int batch_max_blocks_per_cu_t<float>(int, int, int);
extern template hipError_t launch_batch_mfma_t<_Float16>(const BatchJob*, const BatchItem*, const BatchQueues&,
                                                     int*, const BatchRanges&, const void*, int, int, int,
                                                     int, hipStream_t);
extern template int batch_max_blocks_per_cu_t<_Float16>(int, int, int);
extern template hipError_t launch_batch_mfma_t<uint16_t>(const BatchJob*, const BatchItem*, const BatchQueues&,
                                                     int*, const BatchRanges&, const void*, int, int, int,
                                                     int, hipStream_t);
extern template int batch_max_blocks_per_cu_t<uint16_t>(int, int, int);

hipError_t launch_batch_mfma(const BatchJob* jobs, const BatchItem* items, const BatchQueues& q,
                             int* counter, const BatchRanges& br, const void* zrow, int dtype,
                             int prec, int shape, int form, int blocks_per_cu, hipStream_t st) {
  if (q.off[kNumXcd] <= 0) return hipSuccess;
#define CG_BT(T) launch_batch_mfma_t<T>(jobs, items, q, counter, br, zrow, prec, shape, form, blocks_per_cu, st)
  switch (dtype) {
    case 0: return CG_BT(double);
    case 1: return CG_BT(float);
    case 2: return CG_BT(_Float16);
    default: return CG_BT(uint16_t);
  }
#undef CG_BT
}

int batch_max_blocks_per_cu(int dtype, int prec, int shape, int form) {
  switch (dtype) {
    case 0: return batch_max_blocks_per_cu_t<double>(prec, shape, form);
    case 1: return batch_max_blocks_per_cu_t<float>(prec, shape, form);
    case 2: return batch_max_blocks_per_cu_t<_Float16>(prec, shape, form);
    default: return batch_max_blocks_per_cu_t<uint16_t>(prec, shape, form);
  }
}

int batch_shape_rows(int shape) {
  static const int rows[4] = {256, 512, 128, 256};
  return shape >= 0 && shape < 4 ? rows[shape] : 0;
}

}  // namespace cg
