// FP32 gather contraction of narrow data, neighbour statistics and
// normalisation (wide data: cg_gather_wide.hip).
//
// Eq. (1)-(2): for every target t of a tile, S_t[c] += R_n[c] w and
// W_t += w over the tile's candidate samples n with d <= r_s.  Each tile's
// outputs are owned by one workgroup, so no atomics are needed (the
// ownership argument of Sect. 2.2).  The support test is FP64 on unit
// vectors; weights are FP32; products and sums are FP64 (an FP32 weight
// times an FP32 value is exact in FP64), so the result does not depend on
// the order in which candidates arrive, even where the sums cancel.
#include "cg_internal.hpp"

namespace cg {

constexpr int kChunk = 64;   // candidates staged per step

// ---------------------------------------------------------------------------
// Narrow data (nchan <= CMAX <= 16): one lane per target.  A chunk of
// candidates and their (sorted, FP32) data rows is staged in LDS; each lane
// first marks, in a 64-bit mask, the candidates within the support of its
// target (FP64 test), then walks only its own marked candidates: weight and
// channel products for those pairs alone, with no lane idling on the pairs
// of other targets.  Sums per lane run in the tile's visit order (see the
// loop), the same on every call.

template <int CMAX, bool RADIAL>
__global__ void __launch_bounds__(64) k_gather_tl(TileView tv, KernelParams kp,
                                                  const float* __restrict__ sdata, int64_t nchan,
                                                  OutView ov) {
  const int64_t tile = tile_of_block(blockIdx.x, tv.ntiles);
  const int lane = threadIdx.x;
  const int64_t slot = tile * kTile + lane;
  __shared__ double s_x[kChunk], s_y[kChunk], s_z[kChunk];
  __shared__ double s_d[kChunk * CMAX];
  const int64_t ns = tv.nslots;
  const double tx = tv.txyz[slot], ty = tv.txyz[ns + slot], tz = tv.txyz[2 * ns + slot];
  double ax[3] = {0.0, 0.0, 0.0}, bx[3] = {0.0, 0.0, 0.0};
  if (kp.type == 1 && isfinite(tx)) target_axes(kp, tv.tll[slot], tv.tll[ns + slot], ax, bx);
  double acc[CMAX];
#pragma unroll
  for (int c = 0; c < CMAX; ++c) acc[c] = 0.0;
  double wacc = 0.0;
  const uint32_t total = (uint32_t)tv.ntot[tile];
  const uint32_t nr = tv.nr[tile];
  const uint32_t* rng = tv.rng + 2 * tv.roff[tile];   // per range: first sorted position, first candidate index
  const double thr = 1.0 - 0.5 * kp.cs2 - 2e-15;
  // Visit order.  The candidates are sorted ring by ring, and only the
  // lanes whose target lies near a ring have pairs in its stretch, so a
  // chunk of consecutive candidates would leave most lanes idle while a few
  // walk their marked pairs.  The tile is therefore visited interleaved:
  // chunk ci takes candidates ci, nch + ci, 2 nch + ci, ..., one from each
  // 64th of the list, so every lane finds about its average share of pairs
  // in every chunk.  Lane j loads the candidates of its 64th in order,
  // following the ranges with a cursor of its own: it finds the range of
  // its first candidate by a binary search and, ranges being non-empty,
  // steps to the next range at most once per chunk.
  const uint32_t nch = (total + kChunk - 1) / kChunk;
  const uint64_t q0 = (uint64_t)lane * nch;
  uint32_t rb = 0, rs = 0, re = 0, ri = 0;   // cursor: range ri = positions rb.. for candidates [rs, re)
  if (q0 < total) {
    uint32_t lo = 0, hi = nr - 1;   // last range whose first candidate index is <= q0
    while (lo < hi) {
      const uint32_t mid = (lo + hi + 1) >> 1;
      if (rng[2 * mid + 1] <= q0) lo = mid;
      else hi = mid - 1;
    }
    ri = lo;
    rb = rng[2 * ri];
    rs = rng[2 * ri + 1];
    re = ri + 1 < nr ? rng[2 * ri + 3] : total;
  }
  const double nan = __longlong_as_double(0x7ff8000000000000ll);
  for (uint32_t ci = 0; ci < nch; ++ci) {
    const uint64_t q = q0 + ci;
    if (q < total) {
      while (q >= re) {   // re < total here, so range ri + 1 exists
        ++ri;
        rb = rng[2 * ri];
        rs = re;
        re = ri + 1 < nr ? rng[2 * ri + 3] : total;
      }
      const int64_t pos = (int64_t)rb + (int64_t)(q - rs);
      const double4 r = tv.srec[pos];
      s_x[lane] = r.x;
      s_y[lane] = r.y;
      s_z[lane] = r.z;
      // every slot of the row is written (zeros past nchan), so the walk
      // reads and multiplies all CMAX slots without a branch per channel
#pragma unroll
      for (int c = 0; c < CMAX; ++c)
        s_d[lane * CMAX + c] = c < nchan ? (double)sdata[pos * nchan + c] : 0.0;
    } else {
      s_x[lane] = s_y[lane] = s_z[lane] = nan;   // no candidate: no test marks it
    }
    __syncthreads();
    // candidates of the chunk that may lie within the support of this lane's
    // target: p_n . p_t >= 1 - cs2/2 (the same cut, as |p_n - p_t|^2 =
    // 2 - 2 p_n . p_t for unit vectors) loosened by 2e-15, which covers the
    // few-ulp deviation of the rounded vectors from unit length and the
    // rounding of the dot product, so the marked set is a superset.  The
    // exact FP64 chord test below decides every marked pair.
    uint64_t inside = 0;
#pragma unroll
    for (int k = kChunk - 1; k >= 0; --k) {
      const double dot = fma(s_x[k], tx, fma(s_y[k], ty, s_z[k] * tz));
      inside = (inside << 1) | (uint64_t)(dot >= thr);
    }
    while (inside) {
      const int k = __builtin_ctzll(inside);
      inside &= inside - 1;
      const double dx = s_x[k] - tx, dy = s_y[k] - ty, dz = s_z[k] - tz;
      const double c2 = dx * dx + dy * dy + dz * dz;
      const double w = c2 <= kp.cs2 ? (double)pair_weight<RADIAL>(kp, c2, dx, dy, dz, ax[0], ax[1],
                                                                   ax[2], bx[0], bx[1], bx[2])
                                    : 0.0;
      wacc += w;
#pragma unroll
      for (int c = 0; c < CMAX; ++c) acc[c] = fma(w, s_d[k * CMAX + c], acc[c]);
    }
    __syncthreads();
  }
  if (ov.mode == ACC_FINAL) {
    const int32_t t = ov.slot_target[slot];
    if (t >= 0) {
      for (int c = 0; c < CMAX && c < nchan; ++c)
        ov.cube[(int64_t)c * ov.cst + (int64_t)t * ov.tst] =
            wacc > 0.0 ? (float)(acc[c] / wacc) : qnan_f();
      if (ov.wout) ov.wout[t] = (float)wacc;
    }
  } else {
    const bool add = ov.mode == ACC_ADD;
    for (int c = 0; c < CMAX && c < nchan; ++c) {
      double* s = ov.S + (int64_t)c * ns + slot;
      *s = add ? *s + acc[c] : acc[c];
    }
    ov.W[slot] = add ? ov.W[slot] + wacc : wacc;
    ov.Wn[slot] = add ? ov.Wn[slot] + wacc : wacc;
  }
}

hipError_t launch_gather_fp32(const TileView& tv, const KernelParams& kp, const void* data,
                              int dtype, int64_t ld, const float* sdata, int64_t nchan,
                              const OutView& ov, hipStream_t st) {
  if (tv.ntiles <= 0) return hipSuccess;
  if (nchan <= kSmallC) {
    const dim3 g((unsigned)tv.ntiles), b(64);
#define CG_TL(C)                                                                      \
  do {                                                                                \
    if (kp.type >= 2)                                                                 \
      hipLaunchKernelGGL((k_gather_tl<C, true>), g, b, 0, st, tv, kp, sdata, nchan, ov);  \
    else                                                                              \
      hipLaunchKernelGGL((k_gather_tl<C, false>), g, b, 0, st, tv, kp, sdata, nchan, ov); \
  } while (0)
    if (nchan <= 1) CG_TL(1);
    else if (nchan <= 2) CG_TL(2);
    else if (nchan <= 4) CG_TL(4);
    else if (nchan <= 8) CG_TL(8);
    else CG_TL(16);
#undef CG_TL
    return hipGetLastError();
  }
  return launch_gather_wide(tv, kp, data, dtype, ld, nchan, ov, st);
}

// ---------------------------------------------------------------------------
// Neighbour statistics: per target, count of samples with d <= r_s and
// sum mod 2^64 of splitmix64(input index).

__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__global__ void __launch_bounds__(64) k_stats(TileView tv, KernelParams kp,
                                              const int32_t* __restrict__ slot_target,
                                              int32_t* __restrict__ counts,
                                              uint64_t* __restrict__ hashes) {
  const int64_t tile = tile_of_block(blockIdx.x, tv.ntiles);
  const int lane = threadIdx.x;
  const int64_t slot = tile * kTile + lane;
  __shared__ double s_x[kChunk], s_y[kChunk], s_z[kChunk];
  __shared__ uint32_t s_n[kChunk];
  const int64_t ns = tv.nslots;
  const double tx = tv.txyz[slot], ty = tv.txyz[ns + slot], tz = tv.txyz[2 * ns + slot];
  int32_t cnt = 0;
  uint64_t h = 0;
  const uint32_t total = (uint32_t)tv.ntot[tile];
  RangeWindow<false> rw;
  rw.init(tv.rng + 2 * tv.roff[tile], tv.nr[tile], total, true);
  for (uint32_t base = 0; base < total; base += kChunk) {
    const int kmax = (int)(total - base < (uint32_t)kChunk ? total - base : (uint32_t)kChunk);
    rw.cover(base, base + kmax - 1, true);
    const int64_t pos = rw.pos(base + (lane < kmax ? lane : kmax - 1), base, base + kmax - 1);
    if (lane < kmax) {
      const double4 r = tv.srec[pos];
      s_x[lane] = r.x;
      s_y[lane] = r.y;
      s_z[lane] = r.z;
      s_n[lane] = (uint32_t)rec_row(r);
    }
    __syncthreads();
    for (int k = 0; k < kmax; ++k) {
      const double dx = s_x[k] - tx, dy = s_y[k] - ty, dz = s_z[k] - tz;
      if (dx * dx + dy * dy + dz * dz <= kp.cs2) {
        ++cnt;
        h += splitmix64((uint64_t)s_n[k]);
      }
    }
    __syncthreads();
  }
  const int32_t t = slot_target[slot];
  if (t >= 0) {
    counts[t] = cnt;
    if (hashes) hashes[t] = h;
  }
}

hipError_t launch_stats(const TileView& tv, const KernelParams& kp, const int32_t* slot_target,
                        int32_t* counts, uint64_t* hashes, hipStream_t st) {
  if (tv.ntiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_stats, dim3((unsigned)tv.ntiles), dim3(64), 0, st, tv, kp, slot_target,
                     counts, hashes);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Eq. (3): R = S / W (NaN where W = 0) into the caller's layout.

__global__ void __launch_bounds__(256) k_normalize(const double* __restrict__ S,
                                                   const double* __restrict__ W,
                                                   const double* __restrict__ Wn,
                                                   const int32_t* __restrict__ target_slot,
                                                   int64_t nslots, int64_t nchan, int64_t ntarget,
                                                   int64_t cst, int64_t tst,
                                                   float* __restrict__ cube, float* __restrict__ wout) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ntarget) return;
  const int64_t c = blockIdx.y;
  const int64_t s = target_slot[t];
  if (cube) {
    const double wn = Wn[s];
    cube[c * cst + t * tst] = wn > 0.0 ? (float)(S[c * nslots + s] / wn) : qnan_f();
  }
  if (wout && c == 0) wout[t] = (float)W[s];
}

hipError_t launch_normalize(const double* S, const double* W, const double* Wn,
                            const int32_t* target_slot, int64_t nslots, int64_t nchan,
                            int64_t ntarget, int64_t cst, int64_t tst, float* cube, float* wout,
                            hipStream_t st) {
  if (ntarget <= 0) return hipSuccess;
  const int64_t gy = cube ? nchan : 1;
  hipLaunchKernelGGL(k_normalize, dim3((unsigned)((ntarget + 255) / 256), (unsigned)gy), dim3(256),
                     0, st, S, W, Wn, target_slot, nslots, nchan, ntarget, cst, tst, cube, wout);
  return hipGetLastError();
}

__global__ void k_fill(float* __restrict__ p, int64_t n, float v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_fill(float* p, int64_t n, float v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

}  // namespace cg
