// FP32 gather contraction of narrow data, neighbour statistics and
// normalisation (wide data: cg_gather_wide.hip).
//
// Eq. (1)-(2): for every target t of a tile, S_t[c] += R_n[c] w and
// W_t += w over the tile's candidate samples n with d <= r_s.  Each tile's
// outputs are owned by one workgroup, so no atomics are needed (the
// ownership argument of Sect. 2.2).  The support test is FP64 on unit
// vectors; weights are FP32; products and sums are FP64 (an FP32 weight
// times an FP32 value is exact in FP64), so the order in which candidates
// arrive, and the number of wavefronts that share a tile, change a sum only
// by its rounding in FP64.
#include "cg_internal.hpp"

namespace cg {

constexpr int kChunk = 64;   // candidates staged per step

typedef float f32x16_t __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------------------
// Narrow data (nchan <= CMAX <= 16): one lane per target, KW wavefronts per
// tile, each with chunks of its own.  A chunk of candidates and their
// (sorted, FP32) data rows is staged in LDS; each lane gets, as a 64-bit
// mask, the candidates that may lie within the support of its target, then
// walks only its own marked candidates: exact FP64 support test, weight and
// channel products for those pairs alone, with no lane idling on the pairs of
// other targets.  Sums per lane run in the tile's visit order (see the loop),
// the same on every call.
//
// The marks come from the matrix cores.  With u, v the components of a unit
// vector along two axes perpendicular to one of the tile's targets, the
// distance (u - u', v - v') is at most the chord, so
//   u^2 + v^2 - 2 u u' - 2 v v' + (u'^2 + v'^2 - cs2) > 0
// rules a pair out.  That is a product over four terms, (u, v, u^2 + v^2, 1)
// of the candidate times (-2u', -2v', 1, ...) of the target: two
// v_mfma_f32_32x32x2 per 32 x 32 pairs, whose sign bits are shifted into the
// masks, one vector instruction per pair and lane.  The FP32 values are
// widened by 4e-6 of the squared extent of the tile and its support (64
// roundings), and the support by 2e-15 for the rounding of u and v in FP64
// (products of unit vectors: 3e-16 each, which counts for supports below
// 1e-12 rad), so the marks are a superset and the FP64 test alone decides.
// Marking with an FP64 dot product per pair and lane took half of the
// kernel's vector instructions (47.2 million samples x 2 onto nside 512: 3.74
// ms, 3.35 with these marks and the kernel type fixed at compile time, and
// 2.57 with the two channels read from the record instead of an array of
// their own; 12 million x 8 onto 4320 x 2160: 3.31 and 2.43 ms).
template <int CMAX, int KT, bool SHORT, int KW>
__global__ void __launch_bounds__(64 * KW, CMAX <= 4 && KT != 3 && SHORT ? 5 : 4) k_gather_tl(TileView tv, KernelParams kp,
                                                       const float* __restrict__ sdata,
                                                       int64_t nchan, OutView ov) {
  // per wavefront: unit vectors, data rows and (u, v, u^2 + v^2, 1) of a chunk
  // rows of 4 channels and more are padded by 16 bytes: at 64 or 128 bytes the
  // lanes' rows fell on 4 or 2 groups of LDS banks (the LDS was busy 85 % of
  // the kernel; 12 million samples x 8: the call 3.59 -> 3.43 ms, 2 million x 16
  // onto 1000 x 1000: 1.82 -> 1.14 ms; FP32 rows in LDS: 3.53 and 1.12 ms)
  constexpr int DS = CMAX >= 4 ? CMAX + 2 : CMAX;
  struct Chunk {
    double x[kChunk], y[kChunk], z[kChunk];
    double d[kChunk * DS];
    float4 q[kChunk];
  };
  __shared__ Chunk s_chunk[KW];
  static_assert(sizeof(Chunk) >= sizeof(double) * 64 * (CMAX + 1), "partial sums");
  const int64_t tile = tile_of_block(blockIdx.x, tv.ntiles);
  const int lane = threadIdx.x & 63, kw = threadIdx.x >> 6;
  Chunk& sc = s_chunk[kw];
  const int64_t slot = tile * kTile + lane;
  const int64_t ns = tv.nslots;
  const uint32_t total = (uint32_t)tv.ntot[tile];
  // nothing to add (the same on every thread of the workgroup)
  if (ov.mode == ACC_ADD && total == 0) return;
  const double tx = tv.txyz[slot], ty = tv.txyz[ns + slot], tz = tv.txyz[2 * ns + slot];
  double ax[3] = {0.0, 0.0, 0.0}, bx[3] = {0.0, 0.0, 0.0};
  if (KT == 1 && isfinite(tx)) target_axes(kp, tv.tll[slot], tv.tll[ns + slot], ax, bx);
  double acc[CMAX];
#pragma unroll
  for (int c = 0; c < CMAX; ++c) acc[c] = 0.0;
  double wacc = 0.0;
  const uint32_t nr = tv.nr[tile];
  const uint32_t* rng = tv.rng + 2 * tv.roff[tile];   // per range: first sorted position, first candidate index
  // axes e, f perpendicular to the first valid target of the tile, c (the
  // branch-free basis of Duff et al. 2017, "Building an Orthonormal Basis,
  // Revisited")
  const uint64_t valid = __ballot(isfinite(tx));
  const int first = valid ? __builtin_ctzll(valid) : 0;
  const double cx = __shfl(tx, first, 64), cy = __shfl(ty, first, 64), cz = __shfl(tz, first, 64);
  const double sg = copysign(1.0, cz), aa = -1.0 / (sg + cz), bb = cx * cy * aa;
  const double ex = 1.0 + sg * cx * cx * aa, ey = sg * bb, ez = -sg * cx;
  const double fx = bb, fy = sg + cy * cy * aa, fz = -cy;
  // this lane's target as the second factor of the products (B operand: lane
  // l holds terms l / 32 and 2 + l / 32 of targets l % 32 and 32 + l % 32)
  float tb[2][2];
  {
    const bool ok = isfinite(tx);
    const float u = ok ? (float)(tx * ex + ty * ey + tz * ez) : 0.0f;
    const float v = ok ? (float)(tx * fx + ty * fy + tz * fz) : 0.0f;
    const float s = u * u + v * v;
    float smax = s;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) smax = fmaxf(smax, __shfl_xor(smax, o, 64));
    const float reach = sqrtf((float)kp.cs2) + 2e-15f;
    const float ext = sqrtf(smax) + reach;
    const float lim = reach * reach * (1.0f + 1e-6f) + 4e-6f * ext * ext;
    const float c0 = -2.0f * u, c1 = -2.0f * v, c3 = ok ? s - lim : 1e30f;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int src = 32 * n + (lane & 31);
      const float g0 = __shfl(c0, src, 64), g1 = __shfl(c1, src, 64), g3 = __shfl(c3, src, 64);
      tb[n][0] = lane < 32 ? g0 : g1;
      tb[n][1] = lane < 32 ? 1.0f : g3;
    }
  }
  // chunk entry in row i of the first factor's block m: bit 16 m + r of the
  // sign mask of half h = (i >> 2) & 1 is the row 8 (r / 4) + 4 h + r % 4
  const int ai = lane & 31;
  const int arow = 32 * ((ai >> 2) & 1) + 4 * (ai >> 3) + (ai & 3);
  // Visit order.  The candidates are sorted ring by ring, and only the
  // lanes whose target lies near a ring have pairs in its stretch, so a
  // chunk of consecutive candidates would leave most lanes idle while a few
  // walk their marked pairs.  The tile is therefore visited interleaved:
  // chunk ci takes candidates ci, nch + ci, 2 nch + ci, ..., one from each
  // 64th of the list, so every lane finds about its average share of pairs
  // in every chunk.  Lane j loads the candidates of its 64th in order,
  // following the ranges with a cursor of its own: it finds the range of
  // its first candidate by a binary search and steps on from there (ranges
  // are non-empty).  Wavefront kw takes the chunks kw, kw + KW, ...
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
  // record and row of this lane's candidate of chunk ci (lr.x NaN: none),
  // loaded one chunk ahead
  double4 lr;
  float ld[CMAX];
  const double nan = __longlong_as_double(0x7ff8000000000000ll);
  auto fetch = [&](uint32_t ci) {
    const uint64_t q = q0 + ci;
    lr.x = nan;
    if (ci < nch && q < total) {
      while (q >= re) {   // re < total here, so range ri + 1 exists
        ++ri;
        rb = rng[2 * ri];
        rs = re;
        re = ri + 1 < nr ? rng[2 * ri + 3] : total;
      }
      const int64_t pos = (int64_t)rb + (int64_t)(q - rs);
      lr = tv.srec[pos];
      // every slot of the row is set (zeros past nchan), so the walk reads
      // and multiplies all CMAX slots without a branch per channel
      if constexpr (CMAX <= kRecC) {   // carried in the record
        const uint64_t d = (uint64_t)__double_as_longlong(lr.w);
        ld[0] = __uint_as_float((uint32_t)d);
        if (CMAX > 1) ld[CMAX - 1] = __uint_as_float((uint32_t)(d >> 32));
      } else {
#pragma unroll
        for (int c = 0; c < CMAX; ++c) ld[c] = c < nchan ? sdata[pos * nchan + c] : 0.0f;
      }
    }
  };
  fetch(kw);
  for (uint32_t ci = kw; ci < nch; ci += KW) {
    if (lr.x == lr.x) {
      sc.x[lane] = lr.x;
      sc.y[lane] = lr.y;
      sc.z[lane] = lr.z;
      const float u = (float)(lr.x * ex + lr.y * ey + lr.z * ez);
      const float v = (float)(lr.x * fx + lr.y * fy + lr.z * fz);
      sc.q[lane] = make_float4(u, v, u * u + v * v, 1.0f);
#pragma unroll
      for (int c = 0; c < CMAX; ++c) sc.d[lane * DS + c] = (double)ld[c];
    } else {
      sc.q[lane] = make_float4(0.0f, 0.0f, 1e30f, 1.0f);   // no candidate: never marked
    }
    fetch(ci + KW);
    wave_lds_order();
    uint32_t mk[2];   // targets l % 32 and 32 + l % 32, rows of this lane's half
    {
      const float* qf = reinterpret_cast<const float*>(sc.q) + (lane >> 5);
      float a[2][2];
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int p = 0; p < 2; ++p) a[m][p] = qf[4 * (arow + 16 * m) + 2 * p];
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        uint32_t bits = 0;
#pragma unroll
        for (int m = 1; m >= 0; --m) {
          f32x16_t d;
#pragma unroll
          for (int r = 0; r < 16; ++r) d[r] = 0.0f;
          d = __builtin_amdgcn_mfma_f32_32x32x2f32(a[m][0], tb[n][0], d, 0, 0, 0);
          d = __builtin_amdgcn_mfma_f32_32x32x2f32(a[m][1], tb[n][1], d, 0, 0, 0);
#pragma unroll
          for (int r = 15; r >= 0; --r)   // bits = bits << 1 | sign
            bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(d[r]), 31);
        }
        mk[n] = bits;
      }
    }
    // lanes below 32 give their half of the upper targets' masks for the
    // upper lanes' half of the lower targets'
    const auto sw = __builtin_amdgcn_permlane32_swap(mk[0], mk[1], false, false);
    uint64_t inside = (uint64_t)sw[0] | ((uint64_t)sw[1] << 32);
    while (inside) {
      const int k = __builtin_ctzll(inside);
      inside &= inside - 1;
      const double dx = sc.x[k] - tx, dy = sc.y[k] - ty, dz = sc.z[k] - tz;
      const double c2 = dx * dx + dy * dy + dz * dz;
      if (c2 <= kp.cs2) {
        const double w = (double)pair_weight<KT, SHORT>(kp, c2, dx, dy, dz, ax[0], ax[1], ax[2],
                                                        bx[0], bx[1], bx[2]);
        wacc += w;
#pragma unroll
        for (int c = 0; c < CMAX; ++c) acc[c] = fma(w, sc.d[k * DS + c], acc[c]);
      }
    }
    wave_lds_order();
  }
  if constexpr (KW > 1) {
    // partial sums of the wavefronts, added in order
    double* part = reinterpret_cast<double*>(&sc);
#pragma unroll
    for (int c = 0; c < CMAX; ++c) part[64 * c + lane] = acc[c];
    part[64 * CMAX + lane] = wacc;
    __syncthreads();
    if (kw != 0) return;
#pragma unroll
    for (int k = 1; k < KW; ++k) {
      const double* p = reinterpret_cast<const double*>(&s_chunk[k]);
#pragma unroll
      for (int c = 0; c < CMAX; ++c) acc[c] += p[64 * c + lane];
      wacc += p[64 * CMAX + lane];
    }
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
    // Wavefronts per tile: one tile is a chain of chunks, so a map of few
    // tiles is split eight ways (27 tiles of 650 candidates: 73 us with one
    // wavefront each, 15 with eight; 361 tiles of 690: 103 and 25 us); from
    // 1024 tiles on there is a wavefront per SIMD without it, and no partial
    // sums to add.
    const bool split = tv.ntiles < 1024, sh = short_support(kp),
               sinc = sinc_by_series(kp);
#define CG_TLL(C, KT, SH, K) \
  hipLaunchKernelGGL((k_gather_tl<C, KT, SH, K>), g, b, 0, st, tv, kp, sdata, nchan, ov)
#define CG_TLK(C, K)                                        \
  do {                                                      \
    const dim3 g((unsigned)tv.ntiles), b(64 * K);           \
    if (sinc) CG_TLL(C, 4, true, K);                        \
    else if (kp.type >= 2 && sh) CG_TLL(C, 3, true, K);     \
    else if (kp.type >= 2) CG_TLL(C, 3, false, K);          \
    else if (kp.type == 0 && sh) CG_TLL(C, 0, true, K);     \
    else if (kp.type == 0) CG_TLL(C, 0, false, K);          \
    else if (sh) CG_TLL(C, 1, true, K);                     \
    else CG_TLL(C, 1, false, K);                            \
  } while (0)
#define CG_TL(C)            \
  do {                      \
    if (split) CG_TLK(C, 8); \
    else CG_TLK(C, 1);      \
  } while (0)
    if (nchan <= 1) CG_TL(1);
    else if (nchan <= 2) CG_TL(2);
    else if (nchan <= 4) CG_TL(4);
    else if (nchan <= 8) CG_TL(8);
    else CG_TL(16);
#undef CG_TL
#undef CG_TLK
#undef CG_TLL
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
