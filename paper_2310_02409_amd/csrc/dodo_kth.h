// The `rank`-th largest of the scores that one workgroup holds in its registers: shared by the TopK selection and the
// threshold calibration.  Comparisons alone decide (of order_key, or of the scores to the same effect), so the result is
// unique.
//
// Latency is all there is (a few thousand scores, microseconds), so the work is arranged for few barriers: one
// histogram over 2048 equal steps of the scores' own range [min, max] leaves a handful of scores in the bin that holds
// the rank (a radix digit of the bit pattern, mostly exponent, would leave hundreds, and takes four passes), and those
// are ranked directly.  The map score -> bin is monotone whatever its rounding, so the bin holds an interval of the
// order.  Scores that tie in masses, or whose range is no finite positive number, go on with 11-bit steps of the key
// range (at most three: every step divides the range by 2048 and equal ends stop it).
#pragma once
#include "dodo_common.h"

namespace dodo {

// Inclusive prefix sum over the wavefront (data-parallel-primitive adds: within rows of 16 lanes, then across rows).
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t x) {
#define DODO_DPP_SCAN(CTRL, ROWS) \
  x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, ROWS, 0xf, false))
  DODO_DPP_SCAN(0x111, 0xf);  // row_shr:1
  DODO_DPP_SCAN(0x112, 0xf);
  DODO_DPP_SCAN(0x114, 0xf);
  DODO_DPP_SCAN(0x118, 0xf);  // row_shr:8
  DODO_DPP_SCAN(0x142, 0xa);  // row_bcast:15 into rows 1 and 3
  DODO_DPP_SCAN(0x143, 0xc);  // row_bcast:31 into rows 2 and 3
#undef DODO_DPP_SCAN
  return x;
}

// Reduction of a wavefront with an idempotent operation (min, max), same result in every lane; lanes without a partner
// in a step combine with themselves.
template <typename F>
__device__ __forceinline__ uint32_t wave_reduce_idempotent(uint32_t x, F op) {
#define DODO_DPP_RED(CTRL, ROWS) \
  x = op(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(static_cast<int>(x), static_cast<int>(x), CTRL, ROWS, 0xf, false)))
  DODO_DPP_RED(0x111, 0xf);
  DODO_DPP_RED(0x112, 0xf);
  DODO_DPP_RED(0x114, 0xf);
  DODO_DPP_RED(0x118, 0xf);
  DODO_DPP_RED(0x142, 0xa);
  DODO_DPP_RED(0x143, 0xc);
#undef DODO_DPP_RED
  return __builtin_amdgcn_readlane(x, kWave - 1);
}
__device__ __forceinline__ float wave_min(float x) {
  return __uint_as_float(wave_reduce_idempotent(__float_as_uint(x), [](uint32_t a, uint32_t b) {
    return __float_as_uint(fminf(__uint_as_float(a), __uint_as_float(b)));
  }));
}
__device__ __forceinline__ float wave_max(float x) {
  return __uint_as_float(wave_reduce_idempotent(__float_as_uint(x), [](uint32_t a, uint32_t b) {
    return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
  }));
}

// Between phases that compare the same registers: keeps the compiler from carrying one phase's comparison masks (two
// scalar registers each) to the next instead of comparing again.
template <int KPT>
__device__ __forceinline__ void forget_comparisons(float (&v)[KPT], int& lim) {
#pragma unroll
  for (int j = 0; j < KPT; ++j) asm volatile("" : "+v"(v[j]));
  asm volatile("" : "+v"(lim));
}

constexpr int kKthBins = 2048;
constexpr int kKthMaxCand = 64;  // a bin with at most this many scores is ranked directly, one per lane
// the scan gives a lane 32 neighbouring bins: four words of padding after each run of 32 keep its reads off each other's banks
__device__ __forceinline__ uint32_t kth_slot(uint32_t bin) { return bin + ((bin >> 5) << 2); }

constexpr int kKthHistWords = kKthBins / 32 * 36;

// HIST_WORDS: more of them where the histogram's room serves as a list between its uses (kth_largest_lds).
template <int THREADS, int HIST_WORDS = kKthHistWords>
struct KthShared {
  static constexpr int kWaves = THREADS / kWave;
  __attribute__((aligned(16))) uint32_t hist[HIST_WORDS];
  __attribute__((aligned(16))) uint32_t lo[kWaves], hi[kWaves];
  uint32_t cand[kKthMaxCand];
  uint32_t n_cand, bin, rem, cnt;
};

// What the steps below share: v[j] is score 64 j + lane of the wavefront's share, NaN beyond the share's `lim` scores.
template <int THREADS, int KPT, class Shared = KthShared<THREADS>>
struct Kth {
  static constexpr int kWaves = THREADS / kWave;
  Shared& sh;
  float (&v)[KPT];
  int& lim;
  uint32_t T = 0, need = 0;  // the result (see kth_largest)

  __device__ __forceinline__ bool valid(int j) const { return j * kWave + lane_id() < lim; }
  __device__ __forceinline__ void clear_hist() {
    for (int i = threadIdx.x; i < kKthHistWords; i += THREADS) sh.hist[i] = 0;
  }
  // Called by the first wavefront: the bin that holds the rem-th largest of what was counted, what is left of rem inside
  // it, and how many it holds.
  __device__ __forceinline__ void find_bin(uint32_t rem, uint32_t& bin, uint32_t& left, uint32_t& cnt) {
    const int lane = lane_id();
    // lane l owns the l-th run of 32 bins from the top
    uint32_t own = 0;
    const uint4* p = reinterpret_cast<const uint4*>(sh.hist + 36 * (63 - lane));
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint4 w = p[i];
      own += (w.x + w.y) + (w.z + w.w);
    }
    const uint32_t upto = wave_prefix_sum(own);
    const uint64_t ge = __ballot(upto >= rem);  // empty only if rem exceeds what was counted
    const int L = ge != 0 ? __ffsll(static_cast<long long>(ge)) - 1 : kWave - 1;
    const uint32_t above = __builtin_amdgcn_readlane(upto - own, L);
    const uint32_t b = lane < 32 ? sh.hist[36 * (63 - L) + 31 - lane] : 0u;
    const uint32_t upto2 = above + wave_prefix_sum(b);
    const uint64_t ge2 = __ballot(upto2 >= rem);
    const int L2 = ge2 != 0 ? __ffsll(static_cast<long long>(ge2)) - 1 : 31;
    bin = 32u * (63 - L) + 31 - L2;
    left = rem - __builtin_amdgcn_readlane(upto2 - b, L2);
    cnt = __builtin_amdgcn_readlane(b, L2);
  }
  __device__ __forceinline__ void find_bin_for_all(uint32_t rem) {
    if (threadIdx.x < kWave) {
      uint32_t bin, left, cnt;
      find_bin(rem, bin, left, cnt);
      if (lane_id() == 0) {
        sh.bin = bin;
        sh.rem = left;
        sh.cnt = cnt;
      }
    }
    __syncthreads();
  }
  // Few members left: their keys go to a list, and every wavefront ranks the list for itself.
  template <typename F>
  __device__ __forceinline__ void rank_members(uint32_t rem, F member) {
    const int lane = lane_id();
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
      if (valid(j) && member(j)) {
        const uint32_t at = atomicAdd(&sh.n_cand, 1u);
        if (at < kKthMaxCand) sh.cand[at] = order_key(v[j]);  // (always)
      }
      if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    const int c = min(static_cast<int>(sh.n_cand), kKthMaxCand);
    const uint32_t mine = lane < c ? sh.cand[lane] : 0u;
    uint32_t n_gt = 0, n_eq = 0;
    for (int i = 0; i < c; ++i) {
      const uint32_t other = __builtin_amdgcn_readlane(mine, i);
      n_gt += other > mine ? 1u : 0u;
      n_eq += other == mine ? 1u : 0u;
    }
    const uint64_t hit = __ballot(lane < c && n_gt < rem && rem <= n_gt + n_eq);
    const int L = hit != 0 ? __ffsll(static_cast<long long>(hit)) - 1 : 0;
    T = __builtin_amdgcn_readlane(mine, L);
    need = rem - __builtin_amdgcn_readlane(n_gt, L);
  }
  // Smallest and largest finite score of the workgroup.
  __device__ __forceinline__ void finite_range(float& mn, float& mx) {
    const float kInf = __builtin_inff();
    mn = kInf;
    mx = -kInf;
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
      const float f = fabsf(v[j]) < kInf ? v[j] : __builtin_nanf("");  // (min and max pass over NaN)
      mn = fminf(mn, f);
      mx = fmaxf(mx, f);
    }
    mn = wave_min(mn);
    mx = wave_max(mx);
    const int wave = threadIdx.x / kWave;
    if (lane_id() == 0) {
      sh.lo[wave] = __float_as_uint(mn);
      sh.hi[wave] = __float_as_uint(mx);
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      mn = fminf(mn, __uint_as_float(sh.lo[w]));
      mx = fmaxf(mx, __uint_as_float(sh.hi[w]));
    }
  }
  // -inf and NaN count with the smallest finite score, +inf with the largest
  static __device__ __forceinline__ uint32_t value_bin(float x, float mn, float steps) {
    return static_cast<uint32_t>(fminf(fmaxf((x - mn) * steps, 0.f), static_cast<float>(kKthBins - 1)));
  }

  // 11-bit steps of the key range, from the members that `first` names; rem counts among them.
  template <typename F>
  __device__ __forceinline__ void by_keys(uint32_t rem, F first) {
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    uint32_t k_lo = 0u, k_hi = 0xffffffffu;
    bool begin = true;
    for (;;) {
      forget_comparisons(v, lim);
      uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
      for (int j = 0; j < KPT; ++j) {
        const uint32_t key = order_key(v[j]);
        const bool m = valid(j) && (begin ? first(j) : (key >= k_lo && key <= k_hi));
        kmin = min(kmin, m ? key : 0xffffffffu);
        kmax = max(kmax, m ? key : 0u);
        if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
      kmin = wave_reduce_idempotent(kmin, [](uint32_t a, uint32_t b) { return min(a, b); });
      kmax = wave_reduce_idempotent(kmax, [](uint32_t a, uint32_t b) { return max(a, b); });
      __syncthreads();  // the previous use of lo, hi and of the histogram is over
      if (lane == 0) {
        sh.lo[wave] = kmin;
        sh.hi[wave] = kmax;
      }
      clear_hist();
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        kmin = min(kmin, sh.lo[w]);
        kmax = max(kmax, sh.hi[w]);
      }
      if (kmin >= kmax) {  // all equal
        T = kmin;
        need = rem;
        return;
      }
      begin = false;
      forget_comparisons(v, lim);
      const int shift = max(0, 21 - __clz(static_cast<int>(kmax - kmin)));  // (kmax - kmin) >> shift < 2048
#pragma unroll
      for (int j = 0; j < KPT; ++j) {
        const uint32_t key = order_key(v[j]);
        if (valid(j) && key >= kmin && key <= kmax) atomicAdd(&sh.hist[kth_slot((key - kmin) >> shift)], 1u);
        if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
      find_bin_for_all(rem);
      rem = sh.rem;
      k_lo = kmin + (sh.bin << shift);
      k_hi = k_lo + ((1u << shift) - 1u);
      if (shift == 0) {
        T = k_lo;
        need = rem;
        return;
      }
      forget_comparisons(v, lim);
      if (sh.cnt <= kKthMaxCand) {
        rank_members(rem, [&](int j) {
          const uint32_t key = order_key(v[j]);
          return key >= k_lo && key <= k_hi;
        });
        return;
      }
    }
  }

  // The whole search.
  __device__ __forceinline__ void run(uint32_t rank) {
    clear_hist();
    if (threadIdx.x == 0) sh.n_cand = 0;
    float mn, mx;
    finite_range(mn, mx);
    const float range = mx - mn, steps = static_cast<float>(kKthBins - 1) / range;
    forget_comparisons(v, lim);
    if (!(range > 0.f && range < __builtin_inff() && steps < __builtin_inff())) {
      by_keys(rank, [](int) { return true; });
      return;
    }
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
      if (valid(j)) atomicAdd(&sh.hist[kth_slot(value_bin(v[j], mn, steps))], 1u);
      if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    find_bin_for_all(rank);
    const uint32_t rem = sh.rem, bin = sh.bin;
    forget_comparisons(v, lim);
    auto in_bin = [&](int j) { return value_bin(v[j], mn, steps) == bin; };
    if (sh.cnt <= kKthMaxCand) {
      rank_members(rem, in_bin);
    } else {
      by_keys(rem, in_bin);
    }
  }
};

// 1 <= rank <= number of scores.  Returns the key of the rank-th largest in T, and in `need` how many of the scores
// equal to it are among the rank largest.  Called by the whole workgroup; sh is not in use by others.
template <int THREADS, int KPT, class Shared>
__device__ __forceinline__ void kth_largest(Shared& sh, float (&v)[KPT], int& lim, uint32_t rank, uint32_t& T,
                                            uint32_t& need) {
  Kth<THREADS, KPT, Shared> s{sh, v, lim};
  s.run(rank);
  T = s.T;
  need = s.need;
}

// ---- more scores than a few per thread ----
// Here the scores sit in LDS and every step is a short loop over them: code that is unrolled over many registers is
// executed once and bound by fetching its instructions (32768 scores, 34 registers per thread: 42 KB of code, 25 us as
// against 16 us as loops).
// Wavefront w owns `rows` x 64 neighbouring scores from row w * rows on; `mine` of them exist (the last wavefronts' may be fewer).
struct LdsShare {
  const float* p;  // this wavefront's scores
  int mine;        // how many
};
// Every wavefront stages its own scores (so no barrier is needed before it reads them back), 16 loads in flight per lane.
__device__ __forceinline__ void stage_share(float* dst, const float* __restrict__ src, int mine) {
  constexpr int kBatch = 16;
  const int lane = lane_id();
#pragma unroll 1
  for (int i0 = 0; i0 < mine; i0 += kBatch * kWave) {
    float x[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) x[u] = src[min(i0 + u * kWave + lane, mine - 1)];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (i0 + u * kWave + lane < mine) dst[i0 + u * kWave + lane] = x[u];
  }
}
template <int UNROLL, typename F>
__device__ __forceinline__ void for_share(const LdsShare& sh, F f) {  // f(score, index in the share, exists), whole rows of 64
  const int lane = lane_id();
  int i0 = 0;
#pragma unroll 1
  for (; i0 + kWave * UNROLL <= sh.mine; i0 += kWave * UNROLL) {
    float x[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) x[u] = sh.p[i0 + u * kWave + lane];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) f(x[u], i0 + u * kWave + lane, true);
  }
#pragma unroll 1
  for (; i0 < sh.mine; i0 += kWave) f(sh.p[min(i0 + lane, sh.mine - 1)], i0 + lane, i0 + lane < sh.mine);
}

// The rem-th largest among the scores whose keys lie in [k_lo, k_hi], by 11-bit steps of the key range.
template <int THREADS, class Shared>
__device__ __forceinline__ void kth_by_keys(Shared& sh, const LdsShare& share, uint32_t rem, uint32_t k_lo,
                                            uint32_t k_hi, uint32_t& T, uint32_t& need) {
  constexpr int kWaves = THREADS / kWave;
  const int lane = lane_id(), wave = threadIdx.x / kWave;
  float none[1];
  int no_lim = 0;
  Kth<THREADS, 1, Shared> s{sh, none, no_lim};
  for (;;) {
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    for_share<4>(share, [&](float x, int, bool exists) {
      const uint32_t key = order_key(x);
      const bool m = exists && key >= k_lo && key <= k_hi;
      kmin = min(kmin, m ? key : 0xffffffffu);
      kmax = max(kmax, m ? key : 0u);
    });
    kmin = wave_reduce_idempotent(kmin, [](uint32_t a, uint32_t b) { return min(a, b); });
    kmax = wave_reduce_idempotent(kmax, [](uint32_t a, uint32_t b) { return max(a, b); });
    __syncthreads();  // the previous use of lo, hi and of the histogram is over
    if (lane == 0) {
      sh.lo[wave] = kmin;
      sh.hi[wave] = kmax;
    }
    s.clear_hist();
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      kmin = min(kmin, sh.lo[w]);
      kmax = max(kmax, sh.hi[w]);
    }
    if (kmin >= kmax) {  // all equal
      T = kmin;
      need = rem;
      return;
    }
    const int shift = max(0, 21 - __clz(static_cast<int>(kmax - kmin)));  // (kmax - kmin) >> shift < 2048
    for_share<4>(share, [&](float x, int, bool exists) {
      const uint32_t key = order_key(x);
      if (exists && key >= kmin && key <= kmax) atomicAdd(&sh.hist[kth_slot((key - kmin) >> shift)], 1u);
    });
    __syncthreads();
    s.find_bin_for_all(rem);
    rem = sh.rem;
    k_lo = kmin + (sh.bin << shift);
    k_hi = k_lo + ((1u << shift) - 1u);
    if (shift == 0) {
      T = k_lo;
      need = rem;
      return;
    }
  }
}

// As kth_largest, for n scores in LDS: a sample of four rows per wavefront gives two bounds between which the rank-th
// largest lies almost surely, one pass counts what lies above them and lists what lies between them (about a thousand
// of 32768), and only the list is searched.  Scores that tie in masses overflow the list; then there are one or two
// values between the bounds, which are counted, or those between are searched by key.  If the rank is not between the
// bounds after all, everything is searched.
// wave_gt and wave_eq: how many of the wavefront's scores are larger than and equal to the result.
constexpr int kWideThreads = 1024;
constexpr int kWideMaxKeys = 34 * 1024;  // next to 17 KiB of static LDS
constexpr int kKthListPerWave = 256;  // on average 75 of a wavefront's 2048 scores lie between the bounds
// The list takes the histogram's room: it is written after the sample's histogram has been read (a barrier between) and
// read before the next one is cleared (another).
using KthWideShared = KthShared<kWideThreads, kWideThreads / kWave * kKthListPerWave>;
template <int THREADS>
__device__ __forceinline__ void kth_largest_lds(KthWideShared& sh, const LdsShare& share, int n, uint32_t rank, uint32_t& T,
                                                uint32_t& need, int& wave_gt, int& wave_eq) {
  static_assert(THREADS == kWideThreads && kWideThreads / kWave * kKthListPerWave >= kKthHistWords, "");
  using Shared = KthWideShared;
  constexpr int kWaves = THREADS / kWave, kSamples = 4;
  const int lane = lane_id(), wave = threadIdx.x / kWave;
  const float kInf = __builtin_inff();
  bool counted = false;
  {
    float smp[kSamples];
    const int rows = (share.mine + kWave - 1) / kWave;
    int lim = 0;
#pragma unroll
    for (int u = 0; u < kSamples; ++u) {
      const int at = (u * rows / kSamples) * kWave + lane;
      smp[u] = at < share.mine ? share.p[at] : __builtin_nanf("");
    }
    Kth<THREADS, kSamples, Shared> s{sh, smp, lim};
    s.clear_hist();
    if (threadIdx.x == 0) sh.n_cand = 0;
    float mn, mx;
    s.finite_range(mn, mx);
    const float range = mx - mn, steps = static_cast<float>(kKthBins - 1) / range;
    if (range > 0.f && range < kInf && steps < kInf) {
#pragma unroll
      for (int u = 0; u < kSamples; ++u)
        if ((u * rows / kSamples) * kWave + lane < share.mine) atomicAdd(&sh.hist[kth_slot(s.value_bin(smp[u], mn, steps))], 1u);
      __syncthreads();
      if (wave == 0) {
        uint32_t m = 0;  // size of the sample
        const uint4* p = reinterpret_cast<const uint4*>(sh.hist + 36 * lane);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint4 w = p[i];
          m += (w.x + w.y) + (w.z + w.w);
        }
        m = __builtin_amdgcn_readlane(wave_prefix_sum(m), kWave - 1);
        // expected rank in the sample and four standard deviations of it
        const float part = static_cast<float>(rank) / static_cast<float>(n), at = part * static_cast<float>(m);
        const float margin = 4.f * sqrtf(at * (1.f - part)) + 4.f;
        const int r_hi = static_cast<int>(at - margin), r_lo = static_cast<int>(at + margin) + 1;
        uint32_t b_hi = kKthBins, b_lo = 0, left, cnt;
        if (r_hi >= 1) s.find_bin(static_cast<uint32_t>(r_hi), b_hi, left, cnt);
        if (r_lo <= static_cast<int>(m)) s.find_bin(static_cast<uint32_t>(r_lo), b_lo, left, cnt);
        if (lane == 0) {
          sh.bin = b_hi;
          sh.rem = b_lo;
        }
      }
      __syncthreads();
      // (any two bounds are good as long as the counts below put the rank between them)
      const uint32_t b_hi = sh.bin, b_lo = sh.rem;
      const float x_hi = b_hi < kKthBins ? mn + static_cast<float>(b_hi + 1) / steps : kInf;
      const float x_lo = b_lo > 0 ? mn + static_cast<float>(b_lo) / steps : -kInf;
      int n_gt = 0, n_in = 0;
      float* mine = reinterpret_cast<float*>(sh.hist) + wave * kKthListPerWave;
      for_share<4>(share, [&](float x, int, bool exists) {
        const bool above = exists && x > x_hi, in = exists && x >= x_lo && x <= x_hi;
        const uint64_t mask = __ballot(in);
        const int at = n_in + popc_below_lane(mask);
        if (in && at < kKthListPerWave) mine[at] = x;
        n_gt += __popcll(__ballot(above));
        n_in += __popcll(mask);
      });
      if (lane == 0) {
        sh.lo[wave] = n_gt;
        sh.hi[wave] = n_in;
      }
      __syncthreads();
      uint32_t all_gt = 0, all_in = 0, most = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        all_gt += sh.lo[w];
        all_in += sh.hi[w];
        most = max(most, sh.hi[w]);
      }
      const uint32_t rem = rank - all_gt;
      if (!(all_gt < rank && rank <= all_gt + all_in)) {
        kth_by_keys<THREADS>(sh, share, rank, 0u, 0xffffffffu, T, need);
      } else if (most <= kKthListPerWave) {
        constexpr int kPer = kKthListPerWave / kWave;
        float c[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) c[j] = j * kWave + lane < n_in ? mine[j * kWave + lane] : __builtin_nanf("");
        int lim2 = n_in;
        __syncthreads();  // the counts have been read
        kth_largest<THREADS, kPer>(sh, c, lim2, rem, T, need);
        const float t = __uint_as_float((T & 0x80000000u) ? T ^ 0x80000000u : ~T);  // (no NaN lies between the bounds)
        counted = true;
        wave_gt = n_gt;
        wave_eq = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
          wave_gt += __popcll(__ballot(c[j] > t));
          wave_eq += __popcll(__ballot(c[j] == t));
        }
      } else {  // ties in masses: one or two values, to be seen in the lists' beginnings
        float lo = kInf, hi = -kInf;
        const int listed = min(n_in, kKthListPerWave);
        for (int i = lane; i < listed; i += kWave) {
          lo = fminf(lo, mine[i]);
          hi = fmaxf(hi, mine[i]);
        }
        lo = wave_min(lo);
        hi = wave_max(hi);
        __syncthreads();  // the counts have been read
        if (lane == 0) {
          sh.lo[wave] = __float_as_uint(lo);
          sh.hi[wave] = __float_as_uint(hi);
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
          lo = fminf(lo, __uint_as_float(sh.lo[w]));
          hi = fmaxf(hi, __uint_as_float(sh.hi[w]));
        }
        int eq_lo = 0, eq_hi = 0;
        for_share<4>(share, [&](float x, int, bool exists) {
          eq_lo += __popcll(__ballot(exists && x == lo));
          eq_hi += __popcll(__ballot(exists && x == hi));
        });
        __syncthreads();
        if (lane == 0) {
          sh.lo[wave] = eq_lo;
          sh.hi[wave] = eq_hi;
        }
        __syncthreads();
        uint32_t all_lo = 0, all_hi = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
          all_lo += sh.lo[w];
          all_hi += sh.hi[w];
        }
        if (lo == hi ? all_hi == all_in : all_hi + all_lo == all_in) {
          const bool top = rem <= all_hi;
          T = order_key(top ? hi : lo);
          need = top ? rem : rem - all_hi;
          counted = true;
          wave_gt = top ? n_gt : n_gt + eq_hi;
          wave_eq = top ? eq_hi : eq_lo;
        } else {
          kth_by_keys<THREADS>(sh, share, rem, order_key(x_lo), order_key(x_hi), T, need);
        }
      }
    } else {
      kth_by_keys<THREADS>(sh, share, rank, 0u, 0xffffffffu, T, need);
    }
  }
  if (!counted) {
    wave_gt = wave_eq = 0;
    for_share<4>(share, [&](float x, int, bool exists) {
      const uint32_t key = order_key(x);
      wave_gt += __popcll(__ballot(exists && key > T));
      wave_eq += __popcll(__ballot(exists && key == T));
    });
  }
}

}  // namespace dodo
