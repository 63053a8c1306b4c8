// FP32 gather contraction of wide data (more than kSmallC channels) on the
// FP64 matrix cores.
//
// Eq. (1) for a tile of 64 targets is S[t][c] += sum_k w[t][k] R[k][c].  The
// weights are FP32 and the data enter as FP32, so every product is exact in
// FP64, and products and sums are FP64 (v_mfma_f64_16x16x4): targets as M,
// channels as N, candidate samples as K.
//
// What bounds it: the FP64 rate (matrix and vector FP64 share it; a large
// library product reaches 71 TFLOP/s, a loop of vector FMAs 57), so the
// products spent on pairs outside the support are what counts.  The tile's 64 targets are therefore taken as
// four groups of 16 (4 x 4 pixels of a WCS tile, else 16 consecutive slots)
// and each group's products run over a list of its own: the candidates
// within the support of the group's bounding cap, about half of the tile's
// (8 x 8 pixels of 1', 4.5' support: 53 % of the listed pairs are in the
// support, against 27 % of the tile's).  The weights are formed for listed
// pairs only, by one wavefront per group, and shared by all channels of the
// workgroup through LDS.  The cube of 1e6 samples x 1024 channels onto 600 x
// 600 pixels takes 8.7 ms (44 % of the SIMD cycles on the matrix cores, 26 %
// on vector instructions); one lane per channel with a readlane per pair, the
// vector form of the same sums, took 21.8 ms.
//
// A workgroup is CWV x KW wavefronts: wavefront (kw, cw) owns the channels
// [64 cw, 64 cw + 64) of the workgroup's range and the chunks of 32
// candidates kw, kw + KW, ...; the KW partial sums are added in order at the
// end.  Each wavefront stages its own 32 x 64 block of data in LDS, so only
// the lists and weights cross wavefronts (double buffered, one barrier per
// chunk).  Data of the next chunk are in flight in registers meanwhile, and
// candidate records run two chunks ahead.
//
// The matrix products would spread a non-finite value to targets outside its
// support (0 x inf), so such values enter them as zeros, and the chunks that
// hold any are gone through once more at the end, for the targets that the
// values reach: a 16-bit product per chunk, group and channel quarter.  Kept
// out of the loop it takes no registers there, which the radial kernels do not
// have.  120,000 samples x 1000 channels onto 200 x 200 pixels take 1.15 ms,
// 2.40 with every 17th channel blanked (NaN) in every sample, 1.25 with one
// value in 100,000; adding such values pair by pair inside the loop took 4.69
// and 1.50 ms.
#include "cg_internal.hpp"

namespace cg {

namespace {

typedef double f64x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));

constexpr int kWC = 32;                 // candidates per chunk
constexpr int kWSteps = kWC / 4;        // most MFMA steps of a group per chunk
constexpr float kFltMax = 3.402823466e38f;
constexpr int kWRow = 66;               // padded row of the output transpose (doubles)

template <typename T>
__device__ __forceinline__ float cvt_in(T v) { return (float)v; }
template <>
__device__ __forceinline__ float cvt_in<uint16_t>(uint16_t v) {
  return __uint_as_float((uint32_t)v << 16);
}

// 4 consecutive values of a row (zeros past nvalid)
template <typename T>
__device__ __forceinline__ void load_raw4(const T* __restrict__ p, int nvalid, bool vec_ok, T* o) {
  if (vec_ok && nvalid >= 4) {
    typedef T t4_t __attribute__((ext_vector_type(4)));
    const t4_t v = *reinterpret_cast<const t4_t*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = v[i];
    return;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = i < nvalid ? p[i] : (T)0;
}

template <int CWV, int KW, int KT, bool SHORT, typename T>
__global__ void __launch_bounds__(64 * CWV * KW, 2) k_gather_wide(
    TileView tv, KernelParams kp, const T* __restrict__ data, int64_t ld, int64_t nchan,
    int vec_ok_in, OutView ov) {
  constexpr int NW = CWV * KW;
  constexpr int NB = CWV > 1 ? 2 : 1;   // list/weight buffers (a lone wavefront reads what it wrote)
  constexpr int NR = CWV > 1 ? 3 : 1;   // record slots (ring)
  constexpr int GPW = 4 / CWV;          // groups whose weights a wavefront forms
  __shared__ double s_rec[NR][KW][kWC][4];                      // x, y, z, element offset of the row
  __shared__ float s_w[NB][KW][4][kWSteps][64];                 // weights in operand order
  __shared__ __attribute__((aligned(8))) uint8_t s_list[NB][KW][4][4][kWSteps];   // [k][step]: chunk row
  __shared__ int s_nst[NB][KW][4];                              // steps of each group
  __shared__ double s_t[64][9];                                 // target xyz, major axis, minor axis
  __shared__ double s_gc[4][4];                                 // group centre, squared chord of its reach
  __shared__ double s_wp[KW][64], s_wt[64];
  __shared__ uint64_t s_odd[NW];
  __shared__ __attribute__((aligned(16))) double s_buf[NW][16 * kWRow];   // data block / output transpose
  static_assert(sizeof(s_buf[0]) >= sizeof(float) * kWC * 64, "data block");

  int64_t tile, pass;
  work_of_block(blockIdx.x, tv.ntiles, (nchan + 64 * CWV - 1) / (64 * CWV), &tile, &pass);
  if (tv.ntx > 0) tile = strip_tile(tile, tv.ntiles, tv.ntx);
  const uint32_t total = (uint32_t)tv.ntot[tile];
  // nothing to add (the same on every thread of the workgroup)
  if (ov.mode == ACC_ADD && total == 0) return;

  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int kw = wv / CWV, cw = wv % CWV;
  const int li = lane & 15, lk = lane >> 4;   // operand row (target / channel quad), candidate of the step
  const int64_t ns = tv.nslots;
  const int64_t c0 = pass * 64 * CWV;
  const bool quad = tv.ntx > 0;   // tile slots are an 8 x 8 pixel block
  auto slot_of = [&](int g, int i) {
    return quad ? (4 * (g >> 1) + (i >> 2)) * 8 + 4 * (g & 1) + (i & 3) : 16 * g + i;
  };

  if (t < 64) {
    const int g = t >> 4;
    const int sl = slot_of(g, t & 15);
    const int64_t slot = tile * kTile + sl;
    const double x = tv.txyz[slot], y = tv.txyz[ns + slot], z = tv.txyz[2 * ns + slot];
    const bool ok = isfinite(x);
    double a[3] = {0.0, 0.0, 0.0}, b[3] = {0.0, 0.0, 0.0};
    if (KT == 1 && ok) target_axes(kp, tv.tll[slot], tv.tll[ns + slot], a, b);
    double* st = s_t[t];   // in group order
    st[0] = x; st[1] = y; st[2] = z;
    st[3] = a[0]; st[4] = a[1]; st[5] = a[2];
    st[6] = b[0]; st[7] = b[1]; st[8] = b[2];
    // the group's cap: every sample within the support of one of its targets
    // lies within rs + (cap radius) of its centre
    double sx = ok ? x : 0.0, sy = ok ? y : 0.0, sz = ok ? z : 0.0, cnt = ok ? 1.0 : 0.0;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      sx += __shfl_xor(sx, o, 64);
      sy += __shfl_xor(sy, o, 64);
      sz += __shfl_xor(sz, o, 64);
      cnt += __shfl_xor(cnt, o, 64);
    }
    const double nrm = sqrt(sx * sx + sy * sy + sz * sz);
    double reach = -1.0;   // no target: no candidate
    double cx = 0.0, cy = 0.0, cz = 1.0;
    if (cnt > 0.0) {
      reach = 8.0;         // more than any squared chord: all candidates
      if (nrm > 1e-6 * cnt) {
        cx = sx / nrm; cy = sy / nrm; cz = sz / nrm;
        double ang = 0.0;
        if (ok) {
          const double qx = cy * z - cz * y, qy = cz * x - cx * z, qz = cx * y - cy * x;
          ang = atan2(sqrt(qx * qx + qy * qy + qz * qz), cx * x + cy * y + cz * z);
        }
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) ang = fmax(ang, __shfl_xor(ang, o, 64));
        const double half = asin(fmin(1.0, 0.5 * sqrt(kp.cs2))) + 0.5 * ang;
        if (half < 0.5 * hpx::kPi) {
          // chord of the reach, widened by the rounding of the coordinates
          const double ch = 2.0 * sin(half) * (1.0 + 1e-12) + 1e-14;
          reach = ch * ch;
        }
      }
    }
    if ((t & 15) == 0) {
      s_gc[g][0] = cx; s_gc[g][1] = cy; s_gc[g][2] = cz; s_gc[g][3] = reach;
    }
  }

  const int64_t cl = c0 + 64 * cw + 4 * li;   // this lane's four channels
  const int nvc = (int)((nchan - cl) < 4 ? (nchan - cl) : 4);
  const bool vec_ok = vec_ok_in != 0;
  f64x4_t acc[4][4];
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[g][j] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  double wl[GPW];
#pragma unroll
  for (int q = 0; q < GPW; ++q) wl[q] = 0.0;

  const uint32_t nch = (total + kWC - 1) / kWC;      // chunks of the tile
  const uint32_t nloc = (nch + KW - 1) / KW;         // chunks of each wavefront (some may be empty)
  RangeWindow<false> rw;   // walked by wavefront cw = 0 of each kw
  if (cw == 0) rw.init(tv.rng + 2 * tv.roff[tile], tv.nr[tile], total, true);
  double4 rec;
  const double nan = __longlong_as_double(0x7ff8000000000000ll);
  // record of candidate `lane` of the wavefront's local chunk ch (lanes past
  // the chunk: no candidate, row offset -1)
  auto load_rec = [&](uint32_t ch) {
    rec = make_double4(nan, nan, nan, __longlong_as_double(-1ll));
    const uint64_t base64 = ((uint64_t)ch * KW + kw) * kWC;
    if (base64 >= total) return;
    const uint32_t base = (uint32_t)base64;
    const uint32_t cnt = total - base < (uint32_t)kWC ? total - base : (uint32_t)kWC;
    rw.cover(base, base + cnt - 1, true);
    const int64_t p = rw.pos(base + ((uint32_t)lane < cnt ? (uint32_t)lane : cnt - 1), base,
                             base + cnt - 1);
    if ((uint32_t)lane < cnt) {
      const double4 r = tv.srec[p];
      rec = make_double4(r.x, r.y, r.z, __longlong_as_double(rec_row(r) * ld));
    }
  };
  auto put_rec = [&](int slot) {
    if (lane < kWC) {
      double* q = s_rec[slot][kw][lane];
      q[0] = rec.x; q[1] = rec.y; q[2] = rec.z; q[3] = rec.w;
    }
  };
  T raw[kWSteps][4];   // row 4 i + lk, channels cl .. cl + 3 of the chunk being fetched
  auto fetch = [&](int slot) {
#pragma unroll
    for (int i = 0; i < kWSteps; ++i) {
      const int64_t off = __double_as_longlong(s_rec[slot][kw][4 * i + lk][3]);
      if (off >= 0 && nvc > 0) load_raw4<T>(data + off + cl, nvc, vec_ok, raw[i]);
      else {
#pragma unroll
        for (int j = 0; j < 4; ++j) raw[i][j] = (T)0;
      }
    }
  };
  // FP64 rows become FP32 once the products of the chunk before have covered
  // their loads: as they are they would not fit beside the weights
  constexpr bool WIDE_IN = sizeof(T) == 8;
  float cv[WIDE_IN ? kWSteps : 1][4];
  auto settle = [&]() {
    if constexpr (WIDE_IN) {
#pragma unroll
      for (int i = 0; i < kWSteps; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          cv[i][j] = cvt_in<T>(raw[i][j]);
          __asm__ volatile("" : "+v"(cv[i][j]));
        }
    }
  };
  auto val = [&](int i, int j) -> float {
    if constexpr (WIDE_IN) return cv[i][j];
    else return cvt_in<T>(raw[i][j]);
  };
  float* const sd = reinterpret_cast<float*>(s_buf[wv]);
  // fetched block -> LDS; true when it holds a non-finite value
  auto stage = [&]() -> bool {
    float nf = 0.0f;
#pragma unroll
    for (int i = 0; i < kWSteps; ++i) {
      float4 v;
      v.x = val(i, 0); v.y = val(i, 1);
      v.z = val(i, 2); v.w = val(i, 3);
      nf = fmaf(v.x, 0.0f, nf); nf = fmaf(v.y, 0.0f, nf);
      nf = fmaf(v.z, 0.0f, nf); nf = fmaf(v.w, 0.0f, nf);
      *reinterpret_cast<float4*>(sd + (4 * i + lk) * 64 + 4 * li) = v;
    }
    return __ballot(nf != 0.0f) != 0;
  };
  // non-finite values of the staged block (the cells that this lane staged) -> zero
  auto clean = [&]() {
    wave_lds_order();
    for (int i = 0; i < kWSteps; ++i)
      for (int j = 0; j < 4; ++j) {
        float* c = sd + (4 * i + lk) * 64 + 4 * li + j;
        if (!(fabsf(*c) <= kFltMax)) *c = 0.0f;
      }
  };
  // lists and weights of this wavefront's groups for the chunk in record slot
  auto form = [&](int slot, int buf) {
#pragma unroll
    for (int q = 0; q < GPW; ++q) {
      const int g = cw * GPW + q;
      const double (*rc)[4] = s_rec[slot][kw];
      bool in = false;
      if (lane < kWC) {
        const double dx = rc[lane][0] - s_gc[g][0], dy = rc[lane][1] - s_gc[g][1],
                     dz = rc[lane][2] - s_gc[g][2];
        in = dx * dx + dy * dy + dz * dz <= s_gc[g][3];   // (no candidate: NaN)
      }
      const uint64_t m = __ballot(in);
      const int hits = __popcll(m);
      const int nst = (hits + 3) >> 2;
      uint8_t* lst = &s_list[buf][kw][g][0][0];
      if (in) {
        const int h = __popcll(m & ((1ull << lane) - 1ull));
        lst[(h & 3) * kWSteps + (h >> 2)] = (uint8_t)lane;
      }
      // the last step is filled up with row 0 at weight zero
      if (hits + lane < 4 * nst) {
        const int h = hits + lane;
        lst[(h & 3) * kWSteps + (h >> 2)] = 0;
      }
      if (lane == 0) s_nst[buf][kw][g] = nst;
      wave_lds_order();
      const uint64_t rows = *reinterpret_cast<const uint64_t*>(&s_list[buf][kw][g][lk][0]);
      const double* tt = s_t[16 * g + li];
      const double tx = tt[0], ty = tt[1], tz = tt[2];
      for (int s = 0; s < nst; ++s) {
        const int k = (int)((rows >> (8 * s)) & 255u);
        const double dx = rc[k][0] - tx, dy = rc[k][1] - ty, dz = rc[k][2] - tz;
        const double c2 = dx * dx + dy * dy + dz * dz;
        float w = 0.0f;
        if (c2 <= kp.cs2 && 4 * s + lk < hits)
          w = pair_weight<KT, SHORT>(kp, c2, dx, dy, dz, tt[3], tt[4], tt[5], tt[6], tt[7], tt[8]);
        s_w[buf][kw][g][s][lane] = w;
        wl[q] += (double)w;
      }
    }
  };

  // Non-finite values of the staged block: which targets have one in their
  // support (accumulators: target 4 r + lk, channels 4 li + j) comes from a
  // product of 16-bit numbers per channel quarter and group, all steps of the
  // group as K.  Weights enter as 1 (those below zero in a product of their
  // own), data as 1, 64 and 4096 for +inf, -inf and NaN, so that the sums over
  // at most 32 candidates hold the three counts, exactly in FP32.
  auto spread_non_finite = [&](int buf) {
    auto mark = [](float x) -> uint32_t {   // as FP16 bits
      const uint32_t u = __float_as_uint(x), m = u & 0x7fffffffu;
      return m < 0x7f800000u ? 0u : m > 0x7f800000u ? 0x6c00u : u == m ? 0x3c00u : 0x5400u;
    };
    // rows of the product: row 4 q + r is target 4 r + q
    const int wl_row = 16 * lk + 4 * (li & 3) + (li >> 2);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int nst = __builtin_amdgcn_readfirstlane(s_nst[buf][kw][g]);
      if (nst == 0) continue;
      const uint64_t rows = *reinterpret_cast<const uint64_t*>(&s_list[buf][kw][g][lk][0]);
      u32x4_t up = {0, 0, 0, 0}, dn = {0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < kWSteps; ++s) {
        const float w = s < nst ? s_w[buf][kw][g][s][wl_row] : 0.0f;
        const uint32_t one = 0x3c00u << (16 * (s & 1));
        up[s >> 1] |= w > 0.0f ? one : 0u;
        if (KT >= 3) dn[s >> 1] |= w < 0.0f ? one : 0u;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        __builtin_amdgcn_sched_barrier(0);   // (a quarter at a time, for the registers)
        u32x4_t md = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < kWSteps; ++s)
          md[s >> 1] |= mark(sd[(int)((rows >> (8 * s)) & (kWC - 1)) * 64 + 4 * li + j]) << (16 * (s & 1));
        if (!__ballot((md[0] | md[1] | md[2] | md[3]) != 0)) continue;
        const f16x8_t m = __builtin_bit_cast(f16x8_t, md);
        const f32x4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
        f32x4_t pos = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, up), m, zero, 0, 0, 0);
        f32x4_t neg = zero;
        if (KT >= 3)
          neg = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, dn), m, zero, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const uint32_t a = (uint32_t)pos[r], b = (uint32_t)neg[r];
          const bool plus = ((a & 63u) | ((b >> 6) & 63u)) != 0, minus = (((a >> 6) & 63u) | (b & 63u)) != 0;
          const float inf = __uint_as_float(0x7f800000u);
          float x = plus ? inf : minus ? -inf : 0.0f;
          if ((a | b) >> 12 || (plus && minus)) x = qnan_f();
          acc[g][j][r] += (double)x;
        }
      }
    }
  };

  // prologue: records of the first NR - 1 local chunks in LDS (at least one),
  // of the next one in registers
  if (cw == 0) {
    load_rec(0);
    put_rec(0);
    load_rec(1);
    if (NR > 1) {
      put_rec(1);
      load_rec(2);
    }
  }
  __syncthreads();
  if (nloc > 0) {
    fetch(0);
    settle();
    form(0, 0);
  }
  // record slots of chunks ch + 1, ch + 2 (a lone wavefront is done with the
  // records of chunk ch before it writes those of ch + 1 over them)
  int r1 = NR > 1 ? 1 : 0, r2 = NR > 1 ? 2 : 0;
  // chunks with non-finite values (of a run of 2^bsh to a bit)
  uint64_t odd = 0;
  int bsh = 0;
  while (nloc >> bsh >= 64) ++bsh;
  for (uint32_t ch = 0; ch < nloc; ++ch) {
    const int buf = NB > 1 ? (int)(ch & 1) : 0;
    if (stage()) {
      odd |= 1ull << (ch >> bsh);
      clean();
    }
    if (CWV > 1) __syncthreads();
    else wave_lds_order();
    if (cw == 0) {
      put_rec(r2);
      load_rec(ch + (NR > 1 ? 3 : 2));
    }
    if (CWV == 1) wave_lds_order();
    // (FP64 rows: also past the last chunk, as rows of zeros and empty lists, so
    // that no register is kept for a chunk without them)
    if (WIDE_IN || ch + 1 < nloc) fetch(r1);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int nst = __builtin_amdgcn_readfirstlane(s_nst[buf][kw][g]);
      const uint64_t rows = *reinterpret_cast<const uint64_t*>(&s_list[buf][kw][g][lk][0]);
      const float* wp = &s_w[buf][kw][g][0][lane];
      // operands of step s + 1 are read while step s is on the matrix cores
      float wn = wp[0];
      float4 vn = *reinterpret_cast<const float4*>(sd + (int)(rows & (kWC - 1)) * 64 + 4 * li);
#pragma unroll 1
      for (int s = 0; s < nst; ++s) {
        const double a = (double)wn, v0 = (double)vn.x, v1 = (double)vn.y, v2 = (double)vn.z,
                     v3 = (double)vn.w;
        const int sn = s + 1 < kWSteps ? s + 1 : s;
        wn = wp[64 * sn];
        vn = *reinterpret_cast<const float4*>(
            sd + (int)((rows >> (8 * sn)) & (kWC - 1)) * 64 + 4 * li);
        __builtin_amdgcn_sched_barrier(0);
        acc[g][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, v0, acc[g][0], 0, 0, 0);
        acc[g][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, v1, acc[g][1], 0, 0, 0);
        acc[g][2] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, v2, acc[g][2], 0, 0, 0);
        acc[g][3] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, v3, acc[g][3], 0, 0, 0);
      }
    }
    settle();
    if (WIDE_IN || ch + 1 < nloc) form(r1, NB > 1 ? buf ^ 1 : 0);
    if (NR > 1) {
      r1 = r2;
      r2 = r2 == 2 ? 0 : r2 + 1;
    }
  }

  if (CWV > 1) {   // the workgroup's (they share lists)
    if (lane == 0) s_odd[wv] = odd;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NW; ++k) odd |= s_odd[k];
  }
  if (odd) {
    double keep[GPW];   // the weights are summed already
#pragma unroll
    for (int q = 0; q < GPW; ++q) keep[q] = wl[q];
    if (cw == 0) rw.init(tv.rng + 2 * tv.roff[tile], tv.nr[tile], total, true);
    for (uint32_t ch = 0; ch < nloc; ++ch) {
      if (!((odd >> (ch >> bsh)) & 1)) continue;
      if (CWV > 1) __syncthreads();   // the lists of the chunk before are done with
      if (cw == 0) {
        load_rec(ch);
        put_rec(0);
      }
      if (CWV > 1) __syncthreads();
      else wave_lds_order();
      form(0, 0);
      fetch(0);
      settle();
      const bool mine = stage();
      if (CWV > 1) __syncthreads();
      else wave_lds_order();
      if (mine) spread_non_finite(0);
      if (CWV == 1) wave_lds_order();
    }
#pragma unroll
    for (int q = 0; q < GPW; ++q) wl[q] = keep[q];
  }

  // weight sums: target li of a group, summed over the four candidates of
  // the steps and then over kw
#pragma unroll
  for (int q = 0; q < GPW; ++q) {
    double w = wl[q];
    w += __shfl_xor(w, 16, 64);
    w += __shfl_xor(w, 32, 64);
    if (lk == 0) s_wp[kw][slot_of(cw * GPW + q, li)] = w;
  }
  __syncthreads();
  if (t < 64) {
    double w = s_wp[0][t];
#pragma unroll
    for (int k = 1; k < KW; ++k) w += s_wp[k][t];
    s_wt[t] = w;
  }
  // outputs through LDS, a quarter of each wavefront's block at a time: the
  // channels 4 n + j of all targets (channel-major: consecutive threads write
  // consecutive targets), or all channels of one group (target-major cubes)
  const bool fin = ov.mode == ACC_FINAL;
  const bool tmaj = fin && ov.tst != 1;
  double* const so = s_buf[wv];
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    __syncthreads();   // the previous quarter (or the last chunk's data) is done with
    if (tmaj) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) so[(4 * r + lk) * kWRow + 4 * li + j] = acc[h][j][r];
    } else {
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) so[li * kWRow + slot_of(g, 4 * r + lk)] = acc[g][h][r];
    }
    __syncthreads();
    for (int idx = t; idx < 1024 * CWV; idx += 64 * NW) {
      int sl, c, cwv, row, col;   // tile slot, channel in the range; place in the buffer
      if (tmaj) {
        c = idx % (64 * CWV);
        row = idx / (64 * CWV);
        col = c & 63;
        cwv = c >> 6;
        sl = slot_of(h, row);
      } else {
        sl = col = idx & 63;
        row = (idx >> 6) & 15;
        cwv = idx >> 10;
        c = 64 * cwv + 4 * row + h;
      }
      if (c0 + c >= nchan) continue;
      double o = s_buf[cwv][row * kWRow + col];
#pragma unroll
      for (int k = 1; k < KW; ++k) o += s_buf[k * CWV + cwv][row * kWRow + col];
      const int64_t slot = tile * kTile + sl;
      if (fin) {
        const int32_t tg = ov.slot_target[slot];
        const double wt = s_wt[sl];
        if (tg >= 0)
          ov.cube[(c0 + c) * ov.cst + (int64_t)tg * ov.tst] = wt > 0.0 ? (float)(o / wt) : qnan_f();
      } else if (ov.mode == ACC_ADD) {
        ov.S[(c0 + c) * ns + slot] += o;
      } else {
        ov.S[(c0 + c) * ns + slot] = o;
      }
    }
  }
  if (pass == 0 && t < kTile) {
    const int64_t slot = tile * kTile + t;
    if (fin) {
      const int32_t tg = ov.slot_target[slot];
      if (tg >= 0 && ov.wout) ov.wout[tg] = (float)s_wt[t];
    } else {
      ov.W[slot] = ov.mode == ACC_ADD ? ov.W[slot] + s_wt[t] : s_wt[t];
      ov.Wn[slot] = ov.mode == ACC_ADD ? ov.Wn[slot] + s_wt[t] : s_wt[t];
    }
  }
}

template <int CWV, int KW, typename T>
void launch_kt(const TileView& tv, const KernelParams& kp, const void* data, int64_t ld,
               int64_t nchan, const OutView& ov, hipStream_t st) {
  const int64_t npass = (nchan + 64 * CWV - 1) / (64 * CWV);
  const dim3 g((unsigned)(tv.ntiles * npass)), b(64 * CWV * KW);
  // vector loads need every row start aligned to four elements
  const int vec_ok = (ld % 4 == 0) && ((uintptr_t)data % (4 * sizeof(T)) == 0) ? 1 : 0;
  const T* d = (const T*)data;
#define CG_WIDE(KT, SH) \
  hipLaunchKernelGGL((k_gather_wide<CWV, KW, KT, SH, T>), g, b, 0, st, tv, kp, d, ld, nchan, vec_ok, ov)
  const bool sh = short_support(kp);
  if (sinc_by_series(kp)) CG_WIDE(4, true);
  else if (kp.type >= 2 && sh) CG_WIDE(3, true);
  else if (kp.type >= 2) CG_WIDE(3, false);
  else if (kp.type == 0 && sh) CG_WIDE(0, true);
  else if (kp.type == 0) CG_WIDE(0, false);
  else if (sh) CG_WIDE(1, true);
  else CG_WIDE(1, false);
#undef CG_WIDE
}

template <typename T>
void launch_shape(const TileView& tv, const KernelParams& kp, const void* data, int64_t ld,
                  int64_t nchan, const OutView& ov, hipStream_t st) {
  // Channels share a tile's weights, so the widest workgroup that the
  // channels fill; but when that leaves the chip (256 CUs, two workgroups
  // each) without work, 64-channel workgroups whose four wavefronts split
  // the candidates (eight scans of 40,000 samples x 60 channels, elliptical
  // beam, onto 301 x 257 pixels: 4.3 ms against 9.2 ms in the vector form).
  // Where even those leave CUs empty, eight wavefronts split them (9 tiles x
  // 400 channels: the call 139 us with four, 111 with eight; with two
  // workgroups of four to a CU, four are the better: 250,000 pixels x 60
  // channels 0.83 ms against 0.90).
  const bool few = tv.ntiles * ((nchan + 255) / 256) < 512;
  if (tv.ntiles * ((nchan + 63) / 64) <= 256) launch_kt<1, 8, T>(tv, kp, data, ld, nchan, ov, st);
  else if (nchan <= 64 || few) launch_kt<1, 4, T>(tv, kp, data, ld, nchan, ov, st);
  else if (nchan <= 128) launch_kt<2, 2, T>(tv, kp, data, ld, nchan, ov, st);
  else launch_kt<4, 1, T>(tv, kp, data, ld, nchan, ov, st);
}

}  // namespace

hipError_t launch_gather_wide(const TileView& tv, const KernelParams& kp, const void* data,
                              int dtype, int64_t ld, int64_t nchan, const OutView& ov,
                              hipStream_t st) {
  if (tv.ntiles <= 0) return hipSuccess;
  switch (dtype) {
    case 0: launch_shape<double>(tv, kp, data, ld, nchan, ov, st); break;
    case 1: launch_shape<float>(tv, kp, data, ld, nchan, ov, st); break;
    case 2: launch_shape<_Float16>(tv, kp, data, ld, nchan, ov, st); break;
    default: launch_shape<uint16_t>(tv, kp, data, ld, nchan, ov, st); break;
  }
  return hipGetLastError();
}

}  // namespace cg
