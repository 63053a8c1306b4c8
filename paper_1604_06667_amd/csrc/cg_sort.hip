// Sample preparation, device radix sort and HEALPix ring offsets.
//
// Sect. 2.2 step 3a / Sect. 3.4 (1): every input sample gets its HEALPix
// index.  Sect. 3.4 inverts the sample -> target mapping into a target ->
// sample mapping; here the inversion is a stable sort of the samples by
// RING index, after which the samples of any pixel range of a ring form one
// contiguous run that two binary searches find.
#include "cg_internal.hpp"

namespace cg {

// ---------------------------------------------------------------------------
// prep: RING key per sample; invalid coordinates get the sentinel key Npix
// (sorted past every ring) and raise the sticky input flag.

template <typename T>
__device__ __forceinline__ float to_f32(const T* p, int64_t i);
template <>
__device__ __forceinline__ float to_f32<double>(const double* p, int64_t i) { return (float)p[i]; }
template <>
__device__ __forceinline__ float to_f32<float>(const float* p, int64_t i) { return p[i]; }
template <>
__device__ __forceinline__ float to_f32<uint16_t>(const uint16_t* p, int64_t i) {
  return __uint_as_float(((uint32_t)p[i]) << 16);   // bfloat16 -> float (exact)
}
template <>
__device__ __forceinline__ float to_f32<_Float16>(const _Float16* p, int64_t i) { return (float)p[i]; }

// HEALPix RING key of every sample (its value in the sort is its own index,
// which the first pass forms by itself), and its record in input order: the unit vector and, when the cube has at most
// two channels, the channels as FP32 in the fourth word.  The permutation
// after the sort then reads one 32-byte record per sample instead of the
// separate longitude, latitude and data rows.
template <typename T>
__global__ void __launch_bounds__(256) k_prep(const double* __restrict__ lon,
                                              const double* __restrict__ lat, int64_t n,
                                              int64_t nside, uint32_t* __restrict__ keys, int* flag,
                                              double4* __restrict__ rec,
                                              const T* __restrict__ data, int64_t ld, int npack) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double a = lon[i];
  const double d = lat[i];
  const double nan = __longlong_as_double(0x7ff8000000000000ll);
  uint32_t key;
  double4 r = make_double4(nan, nan, nan, 0.0);
  if (!(isfinite(a) && isfinite(d) && fabs(d) <= 90.0)) {
    key = (uint32_t)hpx::npix(nside);
    atomicOr(flag, 1);
  } else {
    double am = fmod(a, 360.0);
    if (am < 0.0) am += 360.0;
    const double phi = am * (hpx::kPi / 180.0);
    double sd, cd, sa, ca;
    sincos(d * (hpx::kPi / 180.0), &sd, &cd);
    sincos(phi, &sa, &ca);
    key = (uint32_t)hpx::ang2pix_ring(nside, sd, cd, phi);
    r.x = cd * ca;
    r.y = cd * sa;
    r.z = sd;
  }
  if (npack > 0) {
    const float d0 = to_f32<T>(data, i * ld);
    const float d1 = npack > 1 ? to_f32<T>(data, i * ld + 1) : 0.0f;
    r.w = __longlong_as_double((long long)(((uint64_t)__float_as_uint(d1) << 32) |
                                           (uint64_t)__float_as_uint(d0)));
  }
  keys[i] = key;
  rec[i] = r;
}

hipError_t launch_prep(const double* lon, const double* lat, int64_t n, int64_t nside,
                       uint32_t* keys, int* flag, double* rec, const void* data,
                       int dtype, int64_t ld, int npack, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const dim3 grid((unsigned)((n + 255) / 256)), blk(256);
  double4* r = reinterpret_cast<double4*>(rec);
  switch (dtype) {
    case 0:
      hipLaunchKernelGGL(k_prep<double>, grid, blk, 0, st, lon, lat, n, nside, keys, flag, r,
                         (const double*)data, ld, npack);
      break;
    case 1:
      hipLaunchKernelGGL(k_prep<float>, grid, blk, 0, st, lon, lat, n, nside, keys, flag, r,
                         (const float*)data, ld, npack);
      break;
    case 2:
      hipLaunchKernelGGL(k_prep<_Float16>, grid, blk, 0, st, lon, lat, n, nside, keys, flag,
                         r, (const _Float16*)data, ld, npack);
      break;
    default:
      hipLaunchKernelGGL(k_prep<uint16_t>, grid, blk, 0, st, lon, lat, n, nside, keys, flag,
                         r, (const uint16_t*)data, ld, npack);
      break;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Stable LSD radix sort of (key, value) uint32 pairs.
//
// Every pass ranks its pairs inside each wavefront: a wavefront takes 64
// consecutive pairs per round, ballots find the lanes with the same digit,
// and a counter per digit, private to the wavefront, adds up the rounds.  The
// wavefronts' counters are put together once per pass, so a pass needs a few
// barriers whatever its number of rounds (a prefix over the wavefronts in
// every round, four barriers each, made the scatter of a 4096-pair block take
// 14-15 us, and a sort of 20,000 pairs with 30 key bits 95 us instead of 41).
//
//   * up to kSmallSort pairs: all passes in one workgroup of 16 wavefronts,
//     the pairs in registers and exchanged through LDS (3000 pairs with 30
//     key bits: 80 us with three kernels per pass as it was, 21 us with one;
//     at 8192 pairs the one workgroup's 35 us meets the passes' 38);
//   * more: per pass block histograms (digit-major), one exclusive scan per
//     digit, and a scatter.
//
// Digits take up to kDigitBits bits, split evenly over the passes (three
// passes instead of four: 20,000 pairs 40 us against 44, 47 million 1439
// against 1492 with digits of at most 8 bits).

constexpr int kMaxJobs = 256;   // the job pass sorts by one 8-bit digit

// Lanes of the wavefront whose digit (nbits wide) equals this lane's, among
// the lanes with `valid` set.
template <int NBITS>
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid) {
  uint64_t peers = __ballot(valid);
#pragma unroll
  for (int b = 0; b < NBITS; ++b) {
    const bool bit = (d >> b) & 1u;
    const uint64_t m = __ballot(bit);
    peers &= bit ? m : ~m;
  }
  return peers;
}

// Rank of this lane's pair among the wavefront's pairs with its digit so far
// (stable: rounds, then lanes), with the wavefront's counters in cnt[].
template <int NBITS, typename C>
__device__ __forceinline__ uint32_t rank_round(C* cnt, uint32_t d, bool valid, int lane) {
  const uint64_t peers = match_digit<NBITS>(d, valid);
  const uint64_t below = peers & ((1ull << lane) - 1ull);
  uint32_t base = 0;
  if (valid) base = cnt[d];
  // (LDS accesses of one wavefront are performed in order)
  __asm__ volatile("" ::: "memory");
  if (valid && below == 0) cnt[d] = (C)(base + (uint32_t)__popcll(peers));
  __asm__ volatile("" ::: "memory");
  return base + (uint32_t)__popcll(below);
}

// inclusive sum over the wavefront's lanes
__device__ __forceinline__ uint32_t wave_incl(uint32_t v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)v, o, 64);
    if (lane >= o) v += y;
  }
  return v;
}

// Digit of element i: NBITS key bits at `shift`, or (JOB) the job holding the
// value, i.e. its position in the concatenated order (job offsets in LDS).
template <bool JOB, int NBITS>
__device__ __forceinline__ uint32_t sort_digit(uint32_t key, uint32_t val, int shift,
                                               const int64_t* s_off, int njobs) {
  if constexpr (JOB) return (uint32_t)job_of(s_off, njobs, (int64_t)val);
  else return (key >> shift) & ((1u << NBITS) - 1u);
}

template <bool JOB>
__device__ __forceinline__ void stage_job_offsets(int64_t* s_off, const int64_t* joff, int njobs) {
  if constexpr (JOB) {
    for (int k = threadIdx.x; k <= njobs; k += blockDim.x) s_off[k] = joff[k];
    __syncthreads();
  }
}

// All passes of a small sort in one workgroup.  Round r of wavefront w holds
// the pairs (w nr + r) 64 + lane.
constexpr int kSmallThreads = 1024;
constexpr int kSmallRounds = 8;
constexpr int64_t kSmallSort = kSmallThreads * kSmallRounds;
constexpr int kDigitBits = 10;

template <int NBITS>
__global__ void __launch_bounds__(kSmallThreads) k_sort_small(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, int n, int npass,
    uint32_t* __restrict__ kout, uint32_t* __restrict__ vout) {
  constexpr int NW = kSmallThreads / 64;
  constexpr int BINS = 1 << NBITS;
  static_assert(BINS <= kSmallThreads, "one digit per thread");
  __shared__ uint16_t s_cnt[NW][BINS];   // counts, then first position of each wavefront's digit run
  __shared__ uint32_t s_k[kSmallSort], s_v[kSmallSort];
  __shared__ uint32_t s_w[NW];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int nr = (n + kSmallThreads - 1) / kSmallThreads;   // rounds of each wavefront
  const int first = w * nr * 64 + lane;
  uint32_t key[kSmallRounds], val[kSmallRounds], rank[kSmallRounds];
#pragma unroll
  for (int r = 0; r < kSmallRounds; ++r) {
    const int i = first + 64 * r;
    const bool ok = r < nr && i < n;
    key[r] = ok ? kin[i] : 0u;
    val[r] = ok ? (vin ? vin[i] : (uint32_t)i) : 0u;
  }
  for (int p = 0; p < npass; ++p) {
    const int shift = p * NBITS;
    for (int q = t; q < NW * BINS / 2; q += kSmallThreads) reinterpret_cast<uint32_t*>(&s_cnt[0][0])[q] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallRounds; ++r)
      if (r < nr)
        rank[r] = rank_round<NBITS>(s_cnt[w], (key[r] >> shift) & (BINS - 1), first + 64 * r < n, lane);
    __syncthreads();
    // digit t: its counts over the wavefronts, then the digits' prefix
    uint32_t tot = 0;
    if (t < BINS) {
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        const uint32_t c = s_cnt[q][t];
        s_cnt[q][t] = (uint16_t)tot;
        tot += c;
      }
    }
    const uint32_t incl = wave_incl(tot, lane);
    if (lane == 63) s_w[w] = incl;
    __syncthreads();
    uint32_t base = incl - tot;
    for (int q = 0; q < w; ++q) base += s_w[q];
    if (t < BINS) {
#pragma unroll
      for (int q = 0; q < NW; ++q) s_cnt[q][t] = (uint16_t)(s_cnt[q][t] + base);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallRounds; ++r)
      if (r < nr && first + 64 * r < n) {
        const uint32_t pos = rank[r] + s_cnt[w][(key[r] >> shift) & (BINS - 1)];
        s_k[pos] = key[r];
        s_v[pos] = val[r];
      }
    __syncthreads();
    if (p + 1 < npass) {
#pragma unroll
      for (int r = 0; r < kSmallRounds; ++r) {
        const int i = first + 64 * r;
        if (r < nr && i < n) {
          key[r] = s_k[i];
          val[r] = s_v[i];
        }
      }
      // (the next pass writes s_k and s_v after three more barriers)
    }
  }
  for (int i = t; i < n; i += kSmallThreads) {
    kout[i] = s_k[i];
    vout[i] = s_v[i];
  }
}

template <bool JOB, int NBITS, int ITEMS>
__global__ void __launch_bounds__(kSortThreads) k_hist(const uint32_t* __restrict__ keys,
                                                       const uint32_t* __restrict__ vals, int64_t n,
                                                       int shift, uint32_t* __restrict__ hist,
                                                       int64_t nblocks, const int64_t* joff,
                                                       int njobs) {
  constexpr int BINS = 1 << NBITS;
  __shared__ uint32_t h[BINS];
  __shared__ int64_t s_off[JOB ? kMaxJobs + 1 : 1];
  const int t = threadIdx.x;
  for (int q = t; q < BINS; q += kSortThreads) h[q] = 0;
  stage_job_offsets<JOB>(s_off, joff, njobs);
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * (kSortThreads * ITEMS);
  // (all loads first: none of them waits for another pair's count)
  uint32_t in[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t i = base + (int64_t)r * kSortThreads + t;
    in[r] = i < n ? (JOB ? vals[i] : keys[i]) : 0u;
  }
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (base + (int64_t)r * kSortThreads + t < n)
      atomicAdd(&h[sort_digit<JOB, NBITS>(in[r], in[r], shift, s_off, njobs)], 1u);
  __syncthreads();
  for (int q = t; q < BINS; q += kSortThreads) hist[(int64_t)q * nblocks + blockIdx.x] = h[q];
}

// Exclusive scan of each digit's per-block counts (one workgroup per digit,
// coalesced), leaving the digit totals in totals[].  Each pass over 1024
// counts gives every thread four consecutive ones; the threads' sums are
// scanned by shuffles within each wavefront and the four wavefront sums
// are combined through LDS, one barrier per pass.
__global__ void __launch_bounds__(256) k_digit_scan(uint32_t* __restrict__ hist, int64_t nblocks,
                                                    uint32_t* __restrict__ totals) {
  __shared__ uint32_t s_w[2][4];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  uint32_t* h = hist + (int64_t)blockIdx.x * nblocks;
  uint32_t carry = 0;
  int buf = 0;
  for (int64_t b0 = 0; b0 < nblocks; b0 += 1024, buf ^= 1) {
    const int64_t i0 = b0 + 4 * (int64_t)t;
    uint32_t v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = i0 + q < nblocks ? h[i0 + q] : 0u;
    const uint32_t local = v[0] + v[1] + v[2] + v[3];
    const uint32_t incl = wave_incl(local, lane);   // inclusive scan of the threads' sums
    if (lane == 63) s_w[buf][w] = incl;
    __syncthreads();   // (double-buffered sums: the next pass writes the other half)
    uint32_t wbase = 0;
    for (int k = 0; k < w; ++k) wbase += s_w[buf][k];
    uint32_t run = carry + wbase + (incl - local);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (i0 + q < nblocks) h[i0 + q] = run;
      run += v[q];
    }
    carry += s_w[buf][0] + s_w[buf][1] + s_w[buf][2] + s_w[buf][3];
  }
  if (t == 0) totals[blockIdx.x] = carry;
}

// Scatter of one block of kSortThreads * ITEMS pairs.  The pairs are ranked
// stably by digit and placed in LDS in block-sorted order; the block then
// writes them out in that order, so that each digit's run of the block goes
// to consecutive global positions (whole segments instead of one scattered
// 4-byte store per pair).
template <bool JOB, int NBITS, int ITEMS>
__global__ void __launch_bounds__(kSortThreads) k_scatter(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, int64_t n, int shift,
    const uint32_t* __restrict__ hist, const uint32_t* __restrict__ totals, int64_t nblocks,
    uint32_t* __restrict__ kout, uint32_t* __restrict__ vout, const int64_t* joff, int njobs) {
  constexpr int NW = kSortThreads / 64;
  constexpr int BINS = 1 << NBITS;
  constexpr int PER = (BINS + kSortThreads - 1) / kSortThreads;   // consecutive digits per thread
  constexpr int TILE = kSortThreads * ITEMS;
  __shared__ uint16_t s_cnt[NW][BINS];   // counts, then first place in the block of a wavefront's run
  __shared__ uint32_t s_out[BINS];       // global position of a digit's run less its place in the block
  __shared__ uint32_t s_w[2][NW];
  __shared__ uint32_t sk[TILE], sv[TILE];
  __shared__ int64_t s_off[JOB ? kMaxJobs + 1 : 1];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t blk = (int64_t)blockIdx.x * TILE;
  const int64_t first = blk + w * (64 * ITEMS) + lane;
  uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t i = first + 64 * r;
    key[r] = i < n ? kin[i] : 0u;
    val[r] = i < n ? (vin ? vin[i] : (uint32_t)i) : 0u;
  }
  for (int q = t; q < NW * BINS / 2; q += kSortThreads) reinterpret_cast<uint32_t*>(&s_cnt[0][0])[q] = 0u;
  stage_job_offsets<JOB>(s_off, joff, njobs);
  // digit totals (the whole sort) of this thread's digits, and this block's offsets
  uint32_t gt[PER], gb[PER], gsum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int d = PER * t + q;
    gt[q] = d < BINS ? totals[d] : 0u;
    gb[q] = d < BINS ? hist[(int64_t)d * nblocks + blockIdx.x] : 0u;
    gsum += gt[q];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const bool ok = first + 64 * r < n;
    rank[r] = rank_round<NBITS>(s_cnt[w], sort_digit<JOB, NBITS>(key[r], val[r], shift, s_off, njobs), ok, lane);
  }
  __syncthreads();
  // prefix of the counts over the wavefronts, of the digits in the block and
  // of the digit totals
  uint32_t lt[PER], lsum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int d = PER * t + q;
    uint32_t run = 0;
    if (d < BINS) {
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const uint32_t c = s_cnt[k][d];
        s_cnt[k][d] = (uint16_t)run;
        run += c;
      }
    }
    lt[q] = run;
    lsum += run;
  }
  const uint32_t lincl = wave_incl(lsum, lane), gincl = wave_incl(gsum, lane);
  if (lane == 63) {
    s_w[0][w] = lincl;
    s_w[1][w] = gincl;
  }
  __syncthreads();
  uint32_t lrun = lincl - lsum, grun = gincl - gsum;
  for (int k = 0; k < w; ++k) {
    lrun += s_w[0][k];
    grun += s_w[1][k];
  }
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int d = PER * t + q;
    if (d < BINS) {
#pragma unroll
      for (int k = 0; k < NW; ++k) s_cnt[k][d] = (uint16_t)(s_cnt[k][d] + lrun);
      s_out[d] = grun + gb[q] - lrun;
    }
    lrun += lt[q];
    grun += gt[q];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (first + 64 * r < n) {
      const uint32_t p =
          s_cnt[w][sort_digit<JOB, NBITS>(key[r], val[r], shift, s_off, njobs)] + rank[r];
      sk[p] = key[r];
      sv[p] = val[r];
    }
  __syncthreads();
  const int nb = (int)((n - blk) < (int64_t)TILE ? (n - blk) : (int64_t)TILE);
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int j = r * kSortThreads + t;
    if (j < nb) {
      const uint32_t k = sk[j], v = sv[j];
      const uint32_t pos = s_out[sort_digit<JOB, NBITS>(k, v, shift, s_off, njobs)] + (uint32_t)j;
      kout[pos] = k;
      vout[pos] = v;
    }
  }
}

// Pairs per thread of a block: few while that leaves at most 256 blocks (one
// per CU), as a pass is then a chain of latencies (524288 pairs of 30 bits: 62
// us with 4 against 82 with 16; a million: 75 with 8, 85 with 16); many beyond,
// for long runs of a digit in the writes (47.2 million of 26 bits: 1196 us with
// 16 and 512 threads, 1439 with 256 threads, 3323 with 4).
constexpr int64_t kSortBlocks = 256;
static int sort_items(int64_t n) {
  return n <= kSortBlocks * 4 * kSortThreads ? 4 : n <= kSortBlocks * 8 * kSortThreads ? 8 : 16;
}

size_t radix_hist_elems_of(int64_t n) {
  const int64_t tile = (int64_t)kSortThreads * sort_items(n);
  const int64_t nb = (n + tile - 1) / tile;
  return ((size_t)(nb < 1 ? 1 : nb) + 1) << kDigitBits;
}

// A sort of fewer pairs may have more blocks, but with less than 16 pairs per
// thread never more than kSortBlocks, nor more than n pairs make with 4.
size_t radix_hist_elems(int64_t n) {
  const int64_t least = 4 * (int64_t)kSortThreads;
  int64_t nb = (n + least - 1) / least;
  if (nb > kSortBlocks) nb = kSortBlocks;
  const size_t own = radix_hist_elems_of(n), below = ((size_t)(nb < 1 ? 1 : nb) + 1) << kDigitBits;
  return own > below ? own : below;
}

template <bool JOB, int NBITS, int ITEMS>
static void sort_pass(const uint32_t* ki, const uint32_t* vi, uint32_t* ko, uint32_t* vo,
                      uint32_t* hist, int64_t n, int shift, const int64_t* joff, int njobs,
                      hipStream_t st) {
  const int64_t tile = (int64_t)kSortThreads * ITEMS;
  const int64_t nb = (n + tile - 1) / tile;
  uint32_t* totals = hist + (nb << NBITS);
  const dim3 g((unsigned)nb), b(kSortThreads);
  hipLaunchKernelGGL((k_hist<JOB, NBITS, ITEMS>), g, b, 0, st, ki, vi, n, shift, hist, nb, joff, njobs);
  hipLaunchKernelGGL(k_digit_scan, dim3(1u << NBITS), dim3(256), 0, st, hist, nb, totals);
  hipLaunchKernelGGL((k_scatter<JOB, NBITS, ITEMS>), g, b, 0, st, ki, vi, n, shift, hist, totals, nb, ko,
                     vo, joff, njobs);
}

template <bool JOB, int NBITS>
static void sort_pass_items(const uint32_t* ki, const uint32_t* vi, uint32_t* ko, uint32_t* vo,
                            uint32_t* hist, int64_t n, int shift, const int64_t* joff, int njobs,
                            hipStream_t st) {
  const int items = sort_items(n);
  if (items == 4) sort_pass<JOB, NBITS, 4>(ki, vi, ko, vo, hist, n, shift, joff, njobs, st);
  else if (items == 8) sort_pass<JOB, NBITS, 8>(ki, vi, ko, vo, hist, n, shift, joff, njobs, st);
  else sort_pass<JOB, NBITS, 16>(ki, vi, ko, vo, hist, n, shift, joff, njobs, st);
}

hipError_t radix_sort(uint32_t* keys, uint32_t* vals, uint32_t* keys_tmp, uint32_t* vals_tmp,
                      uint32_t* hist, int64_t n, int bits, bool iota, bool* result_in_tmp,
                      hipStream_t st) {
  return radix_sort_jobs(keys, vals, keys_tmp, vals_tmp, hist, n, bits, iota, nullptr, 0,
                         result_in_tmp, st);
}

hipError_t radix_sort_jobs(uint32_t* keys, uint32_t* vals, uint32_t* keys_tmp, uint32_t* vals_tmp,
                           uint32_t* hist, int64_t n, int bits, bool iota, const int64_t* noff,
                           int njobs, bool* result_in_tmp, hipStream_t st) {
  *result_in_tmp = false;
  if (n < 1 || (n == 1 && !iota)) return hipSuccess;
  if (njobs > kMaxJobs) return hipErrorInvalidValue;
  uint32_t *ki = keys, *vi = vals, *ko = keys_tmp, *vo = vals_tmp;
  bool in_tmp = false;
  auto flip = [&]() {
    uint32_t* tk = ki; ki = ko; ko = tk;
    uint32_t* tv = vi; vi = vo; vo = tv;
    in_tmp = !in_tmp;
  };
  const int npass = bits > 0 ? (bits + kDigitBits - 1) / kDigitBits : 0;
  const int db = npass > 0 ? (bits + npass - 1) / npass : 8;   // bits per digit
  if (npass > 0 && n <= kSmallSort) {
    const int np = n == 1 ? 1 : npass;
    if (db <= 8) hipLaunchKernelGGL(k_sort_small<8>, dim3(1), dim3(kSmallThreads), 0, st, ki,
                                     iota ? nullptr : vi, (int)n, np, ko, vo);
    else if (db == 9) hipLaunchKernelGGL(k_sort_small<9>, dim3(1), dim3(kSmallThreads), 0, st, ki,
                                     iota ? nullptr : vi, (int)n, np, ko, vo);
    else hipLaunchKernelGGL(k_sort_small<10>, dim3(1), dim3(kSmallThreads), 0, st, ki,
                                     iota ? nullptr : vi, (int)n, np, ko, vo);
    flip();
  } else {
    for (int p = 0; p < npass; ++p) {
      const uint32_t* in = iota && p == 0 ? nullptr : vi;
      if (db <= 8) sort_pass_items<false, 8>(ki, in, ko, vo, hist, n, 8 * p, noff, njobs, st);
      else if (db == 9) sort_pass_items<false, 9>(ki, in, ko, vo, hist, n, 9 * p, noff, njobs, st);
      else sort_pass_items<false, 10>(ki, in, ko, vo, hist, n, 10 * p, noff, njobs, st);
      flip();
    }
  }
  if (njobs > 1) {
    sort_pass_items<true, 8>(ki, vi, ko, vo, hist, n, 0, noff, njobs, st);
    flip();
  }
  *result_in_tmp = in_tmp;
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Batches: the samples of all jobs in one concatenated order (job j at
// [noff[j], noff[j + 1])), each keyed with its own job's nside.

__global__ void __launch_bounds__(256) k_batch_prep(const BatchJob* __restrict__ jobs,
                                                    const int64_t* __restrict__ noff, int njobs,
                                                    int64_t ntot, uint32_t* __restrict__ keys,
                                                    uint32_t* __restrict__ vals, int* flag) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= ntot) return;
  const int j = job_of(noff, njobs, g);
  const BatchJob& jb = jobs[j];
  const int64_t i = g - jb.noff;
  const double a = jb.lon[i];
  const double d = jb.lat[i];
  uint32_t key;
  if (!(isfinite(a) && isfinite(d) && fabs(d) <= 90.0)) {
    key = (uint32_t)hpx::npix(jb.nside);
    atomicOr(flag, 1);
  } else {
    double am = fmod(a, 360.0);
    if (am < 0.0) am += 360.0;
    double sd, cd;
    sincos(d * (hpx::kPi / 180.0), &sd, &cd);
    key = (uint32_t)hpx::ang2pix_ring(jb.nside, sd, cd, am * (hpx::kPi / 180.0));
  }
  keys[g] = key;
  vals[g] = (uint32_t)g;
}

hipError_t launch_batch_prep(const BatchJob* jobs, const int64_t* noff, int njobs, int64_t ntot,
                             uint32_t* keys, uint32_t* vals, int* flag, hipStream_t st) {
  if (ntot <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_batch_prep, dim3((unsigned)((ntot + 255) / 256)), dim3(256), 0, st, jobs,
                     noff, njobs, ntot, keys, vals, flag);
  return hipGetLastError();
}

// ring offsets of every job: entry e of job j (ring i = e - rooff[j]) is the
// first position of the job's sorted run whose key is >= ring_start(i); entry
// 4 nside is the end of its valid samples.
__global__ void __launch_bounds__(256) k_batch_ring_offsets(const BatchJob* __restrict__ jobs,
                                                            const int64_t* __restrict__ rooff,
                                                            int njobs,
                                                            const uint32_t* __restrict__ keys,
                                                            uint32_t* __restrict__ ring_off) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= rooff[njobs]) return;
  const int j = job_of(rooff, njobs, e);
  const BatchJob& jb = jobs[j];
  const int64_t i = e - rooff[j];
  int64_t lo = jb.noff, hi = jb.noff + jb.n;
  if (i > 0) {
    const uint64_t target = (uint64_t)hpx::ring_start(jb.nside, i);
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if ((uint64_t)keys[mid] < target) lo = mid + 1;
      else hi = mid;
    }
  }
  ring_off[e] = (uint32_t)lo;
}

hipError_t launch_batch_ring_offsets(const BatchJob* jobs, const int64_t* rooff, int njobs,
                                     int64_t nentries, const uint32_t* keys, uint32_t* ring_off,
                                     hipStream_t st) {
  if (nentries <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_batch_ring_offsets, dim3((unsigned)((nentries + 255) / 256)), dim3(256), 0,
                     st, jobs, rooff, njobs, keys, ring_off);
  return hipGetLastError();
}

// sorted unit vectors of every job's valid samples
__global__ void __launch_bounds__(256) k_batch_permute(const BatchJob* __restrict__ jobs,
                                                       const int64_t* __restrict__ noff, int njobs,
                                                       int64_t ntot,
                                                       const uint32_t* __restrict__ vals,
                                                       const uint32_t* __restrict__ ring_off,
                                                       double4* __restrict__ srec) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= ntot) return;
  const int j = job_of(noff, njobs, p);
  const BatchJob& jb = jobs[j];
  if (p >= (int64_t)ring_off[jb.ro_off + 4 * jb.nside]) return;   // invalid samples sort last
  const int64_t src = (int64_t)vals[p] - jb.noff;
  double am = fmod(jb.lon[src], 360.0);
  if (am < 0.0) am += 360.0;
  double sa, ca, sd, cd;
  sincos(am * (hpx::kPi / 180.0), &sa, &ca);
  sincos(jb.lat[src] * (hpx::kPi / 180.0), &sd, &cd);
  // the row is the job's own input index
  srec[p] = make_double4(cd * ca, cd * sa, sd, __longlong_as_double(src));
}

hipError_t launch_batch_permute(const BatchJob* jobs, const int64_t* noff, int njobs, int64_t ntot,
                                const uint32_t* vals, const uint32_t* ring_off, double* srec,
                                hipStream_t st) {
  if (ntot <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_batch_permute, dim3((unsigned)((ntot + 255) / 256)), dim3(256), 0, st,
                     jobs, noff, njobs, ntot, vals, ring_off, reinterpret_cast<double4*>(srec));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// ring_off[i] = first sorted position whose key is >= ring_start(i), for
// i = 1 .. 4 nside; ring_off[4 nside] is the number of valid samples.

__device__ __forceinline__ void ring_offset(const uint32_t* __restrict__ keys, int64_t n, int64_t nside,
                                            int64_t i, uint32_t* __restrict__ ring_off) {
  if (i > 4 * nside) return;
  const uint64_t target = (uint64_t)hpx::ring_start(nside, i);
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((uint64_t)keys[mid] < target) lo = mid + 1;
    else hi = mid;
  }
  ring_off[i] = (uint32_t)lo;
  if (i == 1) ring_off[0] = 0;
}

__global__ void __launch_bounds__(256) k_ring_offsets(const uint32_t* __restrict__ keys, int64_t n,
                                                      int64_t nside, uint32_t* __restrict__ ring_off) {
  ring_offset(keys, n, nside, (int64_t)blockIdx.x * blockDim.x + threadIdx.x + 1, ring_off);
}

hipError_t launch_ring_offsets(const uint32_t* keys, int64_t n, int64_t nside, uint32_t* ring_off,
                               hipStream_t st) {
  const int64_t cnt = 4 * nside;
  hipLaunchKernelGGL(k_ring_offsets, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st, keys, n,
                     nside, ring_off);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// permute: sorted records (unit vector and input row, or the one or two
// channels of a narrow FP32 grid) and, for narrow cubes of more channels, the
// data rows in sorted order converted to FP32 (so the gather streams
// contiguous rows).  Bound by the cache line per record that the random read
// takes: 1.5 ms for 47.2 million records (1.6 with non-temporal loads).  Rows
// stored behind their unit vectors, one stretch per sample, cost more here
// than the gather gained: 12 million x 8 channels 0.77 -> 0.91 ms.

//
// RINGS: the first nrb blocks find the ring offsets, and the permutation tells
// the valid samples by their keys, so that up to kRingMerge samples need one
// launch for both (a map of 20,000 samples: the call 64.1 -> 61.4 us); beyond, the keys'
// bytes cost more than the launch.
constexpr int64_t kRingMerge = 1 << 20;

template <typename T, bool VEC4, bool RINGS>
__global__ void __launch_bounds__(256) k_permute(const uint32_t* __restrict__ keys,
                                                 const uint32_t* __restrict__ vals, int64_t n,
                                                 int64_t nside, int nrb, uint32_t* ring_off,
                                                 const double4* __restrict__ rec,
                                                 const T* __restrict__ data, int64_t ld,
                                                 int64_t nchan, int with_data, int npack,
                                                 double4* __restrict__ srec,
                                                 float* __restrict__ sdata) {
  int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if constexpr (RINGS) {
    if ((int)blockIdx.x < nrb) {
      ring_offset(keys, n, nside, p + 1, ring_off);
      return;
    }
    p -= (int64_t)nrb * blockDim.x;
    if (p >= n || keys[p] >= (uint32_t)hpx::npix(nside)) return;
  } else {
    if (p >= (int64_t)ring_off[4 * nside]) return;
  }
  const int64_t src = vals[p];
  const double4 r = rec[src];
  if (with_data && npack > 0) {
    srec[p] = r;   // one or two channels stay in the record
    return;
  }
  srec[p] = make_double4(r.x, r.y, r.z, __longlong_as_double(src));
  if (with_data) {
    if constexpr (VEC4) {
      // FP32 rows with nchan and ld multiples of 4 and 16-byte aligned: whole
      // 16-byte pieces per load and store
      const float4* in = reinterpret_cast<const float4*>(data + src * ld);
      float4* out = reinterpret_cast<float4*>(sdata + p * nchan);
      for (int64_t c = 0; c < nchan / 4; ++c) out[c] = in[c];
    } else {
      for (int64_t c = 0; c < nchan; ++c) sdata[p * nchan + c] = to_f32<T>(data, src * ld + c);
    }
  }
}

hipError_t launch_permute(const uint32_t* keys, const uint32_t* vals, int64_t n, int64_t nside,
                          uint32_t* ring_off, const double* rec, const void* data, int dtype,
                          int64_t ld, int64_t nchan, bool with_data, int npack, double* srec,
                          float* sdata, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const bool rings = n <= kRingMerge;
  const int nrb = rings ? (int)((4 * nside + 255) / 256) : 0;
  if (!rings) {
    const hipError_t e = launch_ring_offsets(keys, n, nside, ring_off, st);
    if (e != hipSuccess) return e;
  }
  // the grid covers all n sorted entries; threads of invalid ones return
  const dim3 grid((unsigned)((n + 255) / 256 + nrb)), blk(256);
  const int wd = with_data ? 1 : 0;
  const double4* r = reinterpret_cast<const double4*>(rec);
  double4* sr = reinterpret_cast<double4*>(srec);
#define CG_PERMUTE(T, VEC4)                                                                        \
  do {                                                                                             \
    if (rings)                                                                                     \
      hipLaunchKernelGGL((k_permute<T, VEC4, true>), grid, blk, 0, st, keys, vals, n, nside, nrb,  \
                         ring_off, r, (const T*)data, ld, nchan, wd, npack, sr, sdata);            \
    else                                                                                           \
      hipLaunchKernelGGL((k_permute<T, VEC4, false>), grid, blk, 0, st, keys, vals, n, nside, nrb, \
                         ring_off, r, (const T*)data, ld, nchan, wd, npack, sr, sdata);            \
  } while (0)
  switch (dtype) {
    case 0: CG_PERMUTE(double, false); break;
    case 1:
      if (wd && nchan % 4 == 0 && ld % 4 == 0 && ((uintptr_t)data & 15) == 0) CG_PERMUTE(float, true);
      else CG_PERMUTE(float, false);
      break;
    case 2: CG_PERMUTE(_Float16, false); break;
    default: CG_PERMUTE(uint16_t, false); break;
  }
#undef CG_PERMUTE
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// exclusive scan of uint64 counts (tile candidate offsets); out has n + 1
// entries, out[n] = total.

__global__ void __launch_bounds__(1024) k_scan_u64(const uint64_t* __restrict__ in,
                                                   uint64_t* __restrict__ out, int64_t n) {
  // one workgroup walks the array in coalesced rounds of 1024 x 4 values,
  // each round a block scan on top of the running total
  __shared__ uint64_t part[1024];
  const int t = threadIdx.x;
  uint64_t carry = 0;
  for (int64_t r0 = 0; r0 < n; r0 += 4096) {
    uint64_t v[4];
    uint64_t s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t i = r0 + 4 * (int64_t)t + k;
      v[k] = i < n ? in[i] : 0ull;
      s += v[k];
    }
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      const uint64_t u = t >= off ? part[t - off] : 0ull;
      __syncthreads();
      part[t] += u;
      __syncthreads();
    }
    uint64_t run = carry + part[t] - s;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t i = r0 + 4 * (int64_t)t + k;
      if (i < n) out[i] = run;
      run += v[k];
    }
    carry += part[1023];
    __syncthreads();
  }
  if (t == 0) out[n] = carry;
}

hipError_t scan_u64(const uint64_t* in, uint64_t* out, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_scan_u64, dim3(1), dim3(1024), 0, st, in, out, n);
  return hipGetLastError();
}

// Device-wide exclusive scan for long arrays: blocks of kScanBlock values
// are summed, the block sums scanned by k_scan_u64, then every block scans
// its own values on top of its offset.
constexpr int kScanBlock = 4096;

__global__ void __launch_bounds__(1024) k_scan_partials(const uint64_t* __restrict__ in, int64_t n,
                                                        uint64_t* __restrict__ part) {
  __shared__ uint64_t red[1024];
  const int t = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * kScanBlock;
  uint64_t s = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t i = base + 4 * (int64_t)t + k;
    if (i < n) s += in[i];
  }
  red[t] = s;
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if (t < off) red[t] += red[t + off];
    __syncthreads();
  }
  if (t == 0) part[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(1024) k_scan_apply(const uint64_t* __restrict__ in,
                                                     uint64_t* __restrict__ out, int64_t n,
                                                     const uint64_t* __restrict__ poff,
                                                     int64_t nb) {
  __shared__ uint64_t part[1024];
  const int t = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * kScanBlock;
  uint64_t v[4];
  uint64_t s = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t i = base + 4 * (int64_t)t + k;
    v[k] = i < n ? in[i] : 0ull;
    s += v[k];
  }
  part[t] = s;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const uint64_t u = t >= off ? part[t - off] : 0ull;
    __syncthreads();
    part[t] += u;
    __syncthreads();
  }
  uint64_t run = poff[blockIdx.x] + part[t] - s;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t i = base + 4 * (int64_t)t + k;
    if (i < n) out[i] = run;
    run += v[k];
  }
  if (blockIdx.x == 0 && t == 0) out[n] = poff[nb];
}

size_t scan_u64_wide_scratch(int64_t n) {
  const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
  return (size_t)(2 * nb + 1);
}

hipError_t scan_u64_wide(const uint64_t* in, uint64_t* out, int64_t n, uint64_t* scratch,
                         hipStream_t st) {
  const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
  if (nb <= 1) return scan_u64(in, out, n, st);
  uint64_t* part = scratch;
  uint64_t* poff = scratch + nb;
  hipLaunchKernelGGL(k_scan_partials, dim3((unsigned)nb), dim3(1024), 0, st, in, n, part);
  hipLaunchKernelGGL(k_scan_u64, dim3(1), dim3(1024), 0, st, part, poff, nb);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(1024), 0, st, in, out, n, poff, nb);
  return hipGetLastError();
}

}  // namespace cg
