// dodo_score: the Scorer as a linear head d -> 1 (Eq. 6 / Eq. 15 of the Dodo paper).
//
// HBM-bound GEMV: every hidden row is read once, 16 bytes per lane per load,
// one wavefront per row with several loads in flight and, for widths of whole
// wave-wide loads, the next batch of loads in flight while the current one is
// reduced, with the weight vector in registers (in LDS beyond 32 loads); other
// widths stage it once per workgroup in LDS as fp32.
// Summation order is fixed, so the scores are run-to-run deterministic.
#include "dodo_common.h"

namespace dodo {
namespace {

constexpr int kScoreThreads = 256;
constexpr int kRowsPerWave = 4;  // (launch_pipelined)
constexpr int kUnroll = 8;  // 16-byte loads in flight per lane

// Layer dimension of a launch (grid y): layer l reads hidden + l * hidden_ls and w + l * w_ls (elements), writes
// scores + l * scores_ls and adds biases[l] (or the one bias when biases is null).  A single layer: all zero.
struct LayerDim {
  int64_t hidden_ls, w_ls, scores_ls;
  const float* biases;
};

template <int DTYPE>
struct Elems;
template <>
struct Elems<DODO_DTYPE_BF16> {
  static constexpr int kPerLoad = 8;
  typedef uint16_t Raw;
  // w points at 8 consecutive fp32 weights, 16-byte aligned
  __device__ static __forceinline__ float dot(const uint4& v, const float* w) {
    const float4 w0 = *reinterpret_cast<const float4*>(w), w1 = *reinterpret_cast<const float4*>(w + 4);
    float a = bf16_lo(v.x) * w0.x;
    a = fmaf(bf16_hi(v.x), w0.y, a);
    a = fmaf(bf16_lo(v.y), w0.z, a);
    a = fmaf(bf16_hi(v.y), w0.w, a);
    a = fmaf(bf16_lo(v.z), w1.x, a);
    a = fmaf(bf16_hi(v.z), w1.y, a);
    a = fmaf(bf16_lo(v.w), w1.z, a);
    a = fmaf(bf16_hi(v.w), w1.w, a);
    return a;
  }
  // both sides as they are in memory: products of pairs are exact in fp32 and summed in fp32
  __device__ static __forceinline__ float dot(const uint4& v, const uint4& w) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    auto two = [](uint32_t a, uint32_t b, float c) {
      return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
    };
    return two(v.w, w.w, two(v.z, w.z, two(v.y, w.y, two(v.x, w.x, 0.f))));
  }
  __device__ static __forceinline__ float load_one(const void* p, int64_t i) {
    return __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t*>(p)[i]) << 16);
  }
};
template <>
struct Elems<DODO_DTYPE_F32> {
  static constexpr int kPerLoad = 4;
  typedef uint32_t Raw;
  // w points at 4 consecutive fp32 weights, 16-byte aligned
  __device__ static __forceinline__ float dot(const uint4& v, const float* w) {
    const float4 w0 = *reinterpret_cast<const float4*>(w);
    float a = __uint_as_float(v.x) * w0.x;
    a = fmaf(__uint_as_float(v.y), w0.y, a);
    a = fmaf(__uint_as_float(v.z), w0.z, a);
    a = fmaf(__uint_as_float(v.w), w0.w, a);
    return a;
  }
  __device__ static __forceinline__ float dot(const uint4& v, const uint4& w) {
    float a = __uint_as_float(v.x) * __uint_as_float(w.x);
    a = fmaf(__uint_as_float(v.y), __uint_as_float(w.y), a);
    a = fmaf(__uint_as_float(v.z), __uint_as_float(w.z), a);
    return fmaf(__uint_as_float(v.w), __uint_as_float(w.w), a);
  }
  __device__ static __forceinline__ float load_one(const void* p, int64_t i) {
    return static_cast<const float*>(p)[i];
  }
};

__device__ __forceinline__ float wave_sum(float v) { return wave_sum64(v); }

// The weight vector as fp32 in LDS, staged by the whole workgroup.  16-byte loads, all of a thread's loads issued
// before the first is used (the kernel's first loads: one round trip instead of one per element); a weight
// vector that is not 16-byte aligned is fetched element by element.
template <int DTYPE>
__device__ __forceinline__ void stage_weights(const void* __restrict__ w, int d, float* __restrict__ w_lds) {
  using E = Elems<DTYPE>;
  constexpr int kEPL = E::kPerLoad;
  constexpr int kVecPerThread = 4;
  if ((reinterpret_cast<uintptr_t>(w) & 15u) == 0) {
    const int nvec = d / kEPL;  // d is a multiple of 8
    for (int v0 = threadIdx.x; v0 < nvec; v0 += kScoreThreads * kVecPerThread) {
      uint4 wv[kVecPerThread];
#pragma unroll
      for (int u = 0; u < kVecPerThread; ++u)
        wv[u] = static_cast<const uint4*>(w)[min(v0 + u * kScoreThreads, nvec - 1)];
#pragma unroll
      for (int u = 0; u < kVecPerThread; ++u) {
        const int v = v0 + u * kScoreThreads;
        if (v < nvec) {
          float* dst = w_lds + static_cast<size_t>(v) * kEPL;
          if (DTYPE == DODO_DTYPE_F32) {
            *reinterpret_cast<uint4*>(dst) = wv[u];
          } else {
            *reinterpret_cast<float4*>(dst) = make_float4(bf16_lo(wv[u].x), bf16_hi(wv[u].x), bf16_lo(wv[u].y), bf16_hi(wv[u].y));
            *reinterpret_cast<float4*>(dst + 4) = make_float4(bf16_lo(wv[u].z), bf16_hi(wv[u].z), bf16_lo(wv[u].w), bf16_hi(wv[u].w));
          }
        }
      }
    }
  } else {
    for (int c = threadIdx.x; c < d; c += kScoreThreads) w_lds[c] = E::load_one(w, c);
  }
}

// The weight vector as it is in memory, element by element (it need not be aligned to more than an element), by the whole
// workgroup; d is a multiple of 64 loads, and as many as fit a batch are in flight per thread.
template <int DTYPE>
__device__ __forceinline__ void stage_raw_weights(const void* __restrict__ w, int d, uint4* __restrict__ w_raw) {
  typedef typename Elems<DTYPE>::Raw Raw;
  constexpr int kBatch = 8;
  const Raw* src = static_cast<const Raw*>(w);
  Raw* dst = reinterpret_cast<Raw*>(w_raw);
  for (int c0 = threadIdx.x; c0 < d; c0 += kScoreThreads * kBatch) {
    Raw x[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) x[u] = src[min(c0 + u * kScoreThreads, d - 1)];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (c0 + u * kScoreThreads < d) dst[c0 + u * kScoreThreads] = x[u];
  }
}

template <int DTYPE>
__global__ __launch_bounds__(kScoreThreads) void score_kernel(const void* __restrict__ hidden_all,
                                                              const void* __restrict__ w_all, float bias, int64_t N,
                                                              int d, int64_t row_stride,
                                                              float* __restrict__ scores_all, LayerDim ld) {
  using E = Elems<DTYPE>;
  // all arguments in one round of scalar loads (the compiler would fetch them a few at a time, before each first use)
  asm volatile("" ::"s"(hidden_all), "s"(w_all), "s"(bias), "s"(N), "s"(d), "s"(row_stride), "s"(scores_all),
               "s"(ld.hidden_ls), "s"(ld.w_ls), "s"(ld.scores_ls), "s"(ld.biases));
  const int64_t layer = blockIdx.y;
  const size_t esz_l = DTYPE == DODO_DTYPE_F32 ? 4 : 2;
  const void* hidden = static_cast<const char*>(hidden_all) + layer * ld.hidden_ls * esz_l;
  const void* w = static_cast<const char*>(w_all) + layer * ld.w_ls * esz_l;
  float* scores = scores_all + layer * ld.scores_ls;
  if (ld.biases != nullptr) bias = ld.biases[layer];
  constexpr int kEPL = E::kPerLoad;     // elements per 16-byte load
  constexpr int kChunk = kWave * kEPL;  // elements one wave-wide load covers
  extern __shared__ __attribute__((aligned(16))) float w_lds[];
  stage_weights<DTYPE>(w, d, w_lds);
  __syncthreads();

  const int lane = lane_id();
  const int64_t wave = static_cast<int64_t>(blockIdx.x) * (kScoreThreads / kWave) + threadIdx.x / kWave;
  const int64_t nwaves = static_cast<int64_t>(gridDim.x) * (kScoreThreads / kWave);
  const int full_groups = d / (kChunk * kUnroll);
  const size_t esz = DTYPE == DODO_DTYPE_F32 ? 4 : 2;

  for (int64_t row = wave; row < N; row += nwaves) {
    const char* rp = static_cast<const char*>(hidden) + static_cast<size_t>(row) * row_stride * esz;
    float acc[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) acc[u] = 0.f;
    int c0 = lane * kEPL;
    for (int g = 0; g < full_groups; ++g) {
      uint4 v[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u)
        v[u] = load16_stream(rp + static_cast<size_t>(c0 + u * kChunk) * esz);
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) acc[u] += E::dot(v[u], &w_lds[c0 + u * kChunk]);
      c0 += kChunk * kUnroll;
    }
    for (; c0 < d; c0 += kChunk) {  // d is a multiple of 8: a 16-byte load never straddles the row end
      const uint4 v = *reinterpret_cast<const uint4*>(rp + static_cast<size_t>(c0) * esz);
      acc[0] += E::dot(v, &w_lds[c0]);
    }
    float s = 0.f;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) s += acc[u];
    s = wave_sum(s) + bias;
    if (lane == 0) scores[row] = (s == 0.f) ? 0.f : s;  // -0 -> +0
  }
}

// Widths of whole wave-wide loads, d == NB * PB * (64 lanes * elements per load): a wavefront keeps the weight vector in
// registers as it is in memory (4 per load) and reads a row in NB batches of PB loads; the next batch (same row, or the
// wavefront's next row) is in flight while the current one is multiplied and reduced.  No LDS and no barrier: the first
// row is requested before the weights, which is most of the time where a wavefront gets a row or two, and bf16 takes one
// instruction per pair (two exact products and the fp32 sum), unpacking neither side.  Measured, 4096 channels in bf16,
// against weights staged in LDS as fp32: 64 rows 3.1 -> 2.5 us, 3200 rows 9.3 -> 7.7 us, 15000 rows 21.9 -> 19.4 us
// (6.3 TB/s), 32768 rows 41.9 -> 41.5 us (6.5 TB/s: bound by memory).
// A weight vector that does not start on a 16-byte boundary (kStaged) reaches the registers through LDS, as it is in
// memory: the arithmetic, and so every score, is the same for any alignment.  kInLds (fp32 beyond 8192 channels, where
// registers would not do): it stays there.
enum WeightsIn { kDirect, kStaged, kInLds };
template <int DTYPE, int PB, int NB, WeightsIn WEIGHTS>
__global__ __launch_bounds__(kScoreThreads) void score_pipelined_kernel(const void* __restrict__ hidden_all,
                                                                        const void* __restrict__ w_all, float bias,
                                                                        int64_t N, int64_t row_stride,
                                                                        float* __restrict__ scores_all, LayerDim ld) {
  using E = Elems<DTYPE>;
  // all arguments in one round of scalar loads (the compiler would fetch them a few at a time, before each first use)
  asm volatile("" ::"s"(hidden_all), "s"(w_all), "s"(bias), "s"(N), "s"(row_stride), "s"(scores_all),
               "s"(ld.hidden_ls), "s"(ld.w_ls), "s"(ld.scores_ls), "s"(ld.biases));
  const int64_t layer = blockIdx.y;
  constexpr int64_t esz = DTYPE == DODO_DTYPE_F32 ? 4 : 2;
  const char* hidden = static_cast<const char*>(hidden_all) + layer * ld.hidden_ls * esz;
  const char* w = static_cast<const char*>(w_all) + layer * ld.w_ls * esz;
  float* scores = scores_all + layer * ld.scores_ls;
  if (ld.biases != nullptr) bias = ld.biases[layer];

  const int lane = lane_id();
  const int64_t wave = static_cast<int64_t>(blockIdx.x) * (kScoreThreads / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t nwaves = static_cast<int64_t>(gridDim.x) * (kScoreThreads / kWave);

  // Loads are issued unconditionally: a branch around them would make the compiler wait for every outstanding load at
  // the merge.  A row past the end is a buffer of no bytes: its loads fetch nothing and return zeros (re-reading some
  // row instead would send every wavefront to the same few cache lines).
  auto load_batch = [&](uint4 (&v)[PB], int64_t row, int bi) {
    const char* rp = hidden + row * row_stride * esz;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(rp), 0, row < N ? NB * PB * kWave * 16 : 0, 0x00027000);
#pragma unroll
    for (int u = 0; u < PB; ++u) {
      const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16 + (bi * PB + u) * kWave * 16, 0, 2);  // (non-temporal)
      v[u] = make_uint4(t.x, t.y, t.z, t.w);
    }
  };
  uint4 buf[2][PB];  // used alternately, so that no copy has to wait for the loads in flight
  constexpr int kInRegs = WEIGHTS == kInLds ? 1 : NB * PB;
  uint4 wv[kInRegs];
  if (WEIGHTS != kInLds) load_batch(buf[0], wave, 0);
  const uint4* w_src = reinterpret_cast<const uint4*>(w);
  if (WEIGHTS != kDirect) {
    static_assert(WEIGHTS != kInLds || DTYPE == DODO_DTYPE_F32, "stage_weights converts to fp32");
    extern __shared__ uint4 w_raw[];
    if (WEIGHTS == kInLds)
      stage_weights<DTYPE>(w, NB * PB * kWave * E::kPerLoad, reinterpret_cast<float*>(w_raw));
    else
      stage_raw_weights<DTYPE>(w, NB * PB * kWave * E::kPerLoad, w_raw);
    __syncthreads();
    w_src = w_raw;
  }
  if (WEIGHTS != kInLds) {
#pragma unroll
    for (int u = 0; u < kInRegs; ++u) wv[u] = w_src[u * kWave + lane];
  } else {
    load_batch(buf[0], wave, 0);
  }
  constexpr int kRows = WEIGHTS == kInLds && NB % 2 == 0 ? 1 : 2;  // as many as leave which buffer is which known below
  for (int64_t row = wave; row < N; row += kRows * nwaves) {
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < kRows * NB; ++i) {
      if (WEIGHTS == kInLds && i == NB && row + nwaves >= N) break;  // (many loads that would fetch nothing)
      load_batch(buf[(i + 1) & 1], row + (i + 1) / NB * nwaves, (i + 1) % NB);
      __builtin_amdgcn_sched_barrier(0);  // keep the loads ahead of the arithmetic
      const int64_t r = row + i / NB * nwaves;
      const int bi = i % NB;
      if (i < NB || r < N) {
        float part[PB];
#pragma unroll
        for (int u = 0; u < PB; ++u)
          part[u] = E::dot(buf[i & 1][u], WEIGHTS == kInLds ? w_src[(bi * PB + u) * kWave + lane] : wv[(bi * PB + u) % kInRegs]);
#pragma unroll
        for (int u = 0; u < PB; ++u) acc += part[u];
        // (or the compiler puts the arithmetic of the batches behind the loads of the whole row: 256 registers and spills)
        if (WEIGHTS == kInLds) asm volatile("" : "+v"(acc));
        if (bi == NB - 1) {  // the row is complete
          const float s = wave_sum(acc) + bias;
          if (lane == 0) scores[r] = (s == 0.f) ? 0.f : s;  // -0 -> +0
          acc = 0.f;
        }
      }
    }
  }
}

// Workgroups of `kernel` that fit on the device at once (all resident: the kernels stride over the
// rows, so a grid a little larger than this would run in uneven rounds).
template <typename K>
int resident_blocks(K kernel, size_t lds) {
  return compute_units() * resident_blocks_per_cu(reinterpret_cast<const void*>(kernel), kScoreThreads, lds, 2);
}

template <int DTYPE, int PB, int NB, WeightsIn WEIGHTS>
void launch_pipelined(const void* hidden, const void* w, float bias, int64_t N, int64_t row_stride, float* scores,
                      unsigned blocks, hipStream_t s, int L, const LayerDim& ld) {
  const size_t lds = WEIGHTS != kDirect ? PB * NB * kWave * sizeof(uint4) : 0;
  const int cap = resident_blocks(score_pipelined_kernel<DTYPE, PB, NB, WEIGHTS>, lds);
  // What is resident at once, or, from two such rounds on, workgroups of kRowsPerWave rows per wavefront: wavefronts that
  // stride over hundreds of rows drift apart, and reads that are spread over the whole tensor are slower than a front that
  // moves through it.  bf16: 4096 channels, 400000 rows 525 -> 486 us (6.7 TB/s), 100000 rows 124 -> 119 us; 5120 channels,
  // 200000 rows 327 -> 299 us, 32768 rows 50.7 -> 50.2 us; 1024 channels, 400000 rows 140 -> 124 us.  A workgroup that
  // starts has to be hidden by others on its compute unit: where fewer than four fit, the grid stays at one round (8192
  // channels, 100000 rows: 248 us, 264 us with 2048 workgroups), and where it fetches as much of the weights as of a row,
  // and beyond the 2^32 threads that a launch may have.
  const int64_t per_block = kRowsPerWave * (kScoreThreads / kWave);
  const int64_t many = (N + per_block - 1) / per_block;
  if (WEIGHTS != kInLds && cap >= 4 * compute_units() && many >= 2 * static_cast<int64_t>(cap) && many <= 0xffffffffLL / kScoreThreads)
    blocks = static_cast<unsigned>(many);
  else if (blocks > static_cast<unsigned>(cap))
    blocks = cap;
  hipLaunchKernelGGL((score_pipelined_kernel<DTYPE, PB, NB, WEIGHTS>), dim3(blocks, L), dim3(kScoreThreads), lds, s, hidden, w,
                     bias, N, row_stride, scores, ld);
}

// (up to 4 batches of 8 loads: 128 registers of weights; fp32 has rows of up to twice that)
template <int DTYPE>
bool try_pipelined(const void* hidden, const void* w, float bias, int64_t N, int d, int64_t row_stride, float* scores,
                   unsigned blocks, hipStream_t s, int L, const LayerDim& ld) {
  constexpr int kChunk = kWave * Elems<DTYPE>::kPerLoad;
  if (d % kChunk != 0) return false;
  // (every layer's weights have to be aligned for the direct form; the scores do not depend on which of the two runs)
  const bool aligned = aligned16(w) && (ld.w_ls * (DTYPE == DODO_DTYPE_F32 ? 4 : 2)) % 16 == 0;
  switch (d / kChunk) {
#define DODO_SCORE_WIDTH(CHUNKS, PB, NB)                                                            \
  case CHUNKS:                                                                                      \
    static_assert(CHUNKS == PB * NB, "");                                                           \
    if (aligned)                                                                                    \
      launch_pipelined<DTYPE, PB, NB, kDirect>(hidden, w, bias, N, row_stride, scores, blocks, s, L, ld); \
    else                                                                                            \
      launch_pipelined<DTYPE, PB, NB, kStaged>(hidden, w, bias, N, row_stride, scores, blocks, s, L, ld); \
    return true
    DODO_SCORE_WIDTH(1, 1, 1);
    DODO_SCORE_WIDTH(2, 2, 1);
    DODO_SCORE_WIDTH(3, 3, 1);
    DODO_SCORE_WIDTH(4, 4, 1);
    DODO_SCORE_WIDTH(5, 5, 1);
    DODO_SCORE_WIDTH(6, 6, 1);
    DODO_SCORE_WIDTH(7, 7, 1);
    DODO_SCORE_WIDTH(8, 8, 1);
    DODO_SCORE_WIDTH(10, 5, 2);
    DODO_SCORE_WIDTH(12, 6, 2);
    DODO_SCORE_WIDTH(14, 7, 2);
    DODO_SCORE_WIDTH(16, 8, 2);
    DODO_SCORE_WIDTH(18, 6, 3);
    DODO_SCORE_WIDTH(20, 5, 4);
    DODO_SCORE_WIDTH(21, 7, 3);
    DODO_SCORE_WIDTH(24, 8, 3);
    DODO_SCORE_WIDTH(28, 7, 4);
    DODO_SCORE_WIDTH(32, 8, 4);
#undef DODO_SCORE_WIDTH
#define DODO_SCORE_WIDTH(CHUNKS, PB, NB)                                                            \
  case CHUNKS:                                                                                      \
    static_assert(CHUNKS == PB * NB, "");                                                           \
    if constexpr (DTYPE == DODO_DTYPE_F32) {                                                        \
      launch_pipelined<DTYPE, PB, NB, kInLds>(hidden, w, bias, N, row_stride, scores, blocks, s, L, ld); \
      return true;                                                                                  \
    }                                                                                               \
    return false
    DODO_SCORE_WIDTH(35, 7, 5);
    DODO_SCORE_WIDTH(40, 8, 5);
    DODO_SCORE_WIDTH(42, 7, 6);
    DODO_SCORE_WIDTH(48, 8, 6);
    DODO_SCORE_WIDTH(49, 7, 7);
    DODO_SCORE_WIDTH(56, 8, 7);
    DODO_SCORE_WIDTH(64, 8, 8);
#undef DODO_SCORE_WIDTH
    default: return false;
  }
}

}  // namespace
}  // namespace dodo

namespace dodo {
namespace {

int score_entry(const void* hidden, const void* w, float bias, int dtype, int64_t N, int32_t d, int64_t row_stride,
                float* scores, int32_t L, const LayerDim& ld, void* stream) {
  if (N < 0 || d <= 0 || row_stride < d || L < 0) return DODO_ERR_INVALID_ARG;
  if (N == 0 || L == 0) return DODO_OK;
  if (!hidden || !w || !scores) return DODO_ERR_INVALID_ARG;
  if (!dtype_ok(dtype)) return DODO_ERR_UNSUPPORTED;
  const int es = elem_bytes(dtype);
  if (d % 8 != 0 || d > 16384 || L > 65535) return DODO_ERR_UNSUPPORTED;
  if (!aligned16(hidden) || (row_stride * es) % 16 != 0 || (ld.hidden_ls * es) % 16 != 0) return DODO_ERR_UNSUPPORTED;

  const int waves_per_block = kScoreThreads / kWave;
  int64_t blocks = (N + waves_per_block - 1) / waves_per_block;
  const int64_t cap = 256 * 8;  // upper bound; each kernel fits it to what is resident at once
  if (blocks > cap) blocks = cap;
  const size_t lds = static_cast<size_t>(d) * sizeof(float);
  hipStream_t s = static_cast<hipStream_t>(stream);
  // widths that split evenly into batches of 5 to 8 (up to 8 loads: one batch) wave-wide loads (4096, 5120, 8192, ...) take
  // the pipelined kernel
  const unsigned nblk = static_cast<unsigned>(blocks);
  if (dtype == DODO_DTYPE_BF16
          ? try_pipelined<DODO_DTYPE_BF16>(hidden, w, bias, N, d, row_stride, scores, nblk, s, L, ld)
          : try_pipelined<DODO_DTYPE_F32>(hidden, w, bias, N, d, row_stride, scores, nblk, s, L, ld))
    return launch_status();
  if (dtype == DODO_DTYPE_BF16) {
    const int64_t fit = resident_blocks(score_kernel<DODO_DTYPE_BF16>, lds);
    hipLaunchKernelGGL(score_kernel<DODO_DTYPE_BF16>, dim3(static_cast<unsigned>(blocks < fit ? blocks : fit), L),
                       dim3(kScoreThreads), lds, s, hidden, w, bias, N, d, row_stride, scores, ld);
  } else {
    const int64_t fit = resident_blocks(score_kernel<DODO_DTYPE_F32>, lds);
    hipLaunchKernelGGL(score_kernel<DODO_DTYPE_F32>, dim3(static_cast<unsigned>(blocks < fit ? blocks : fit), L),
                       dim3(kScoreThreads), lds, s, hidden, w, bias, N, d, row_stride, scores, ld);
  }
  return launch_status();
}

}  // namespace
}  // namespace dodo

extern "C" int dodo_score(const void* hidden, const void* w, float bias, int dtype, int64_t N, int32_t d,
                          int64_t row_stride, float* scores, void* stream) {
  return dodo::score_entry(hidden, w, bias, dtype, N, d, row_stride, scores, 1, dodo::LayerDim{0, 0, 0, nullptr}, stream);
}

extern "C" int dodo_score_layers(const void* hidden, const void* w, const float* biases, int dtype, int32_t L, int64_t N,
                                 int32_t d, int64_t row_stride, int64_t hidden_layer_stride, int64_t w_layer_stride,
                                 int64_t scores_layer_stride, float* scores, void* stream) {
  if (hidden_layer_stride < 0 || w_layer_stride < 0 || scores_layer_stride < 0) return DODO_ERR_INVALID_ARG;
  if (L > 1 && scores_layer_stride < N) return DODO_ERR_INVALID_ARG;
  return dodo::score_entry(hidden, w, 0.f, dtype, N, d, row_stride, scores, L,
                           dodo::LayerDim{hidden_layer_stride, w_layer_stride, scores_layer_stride, biases}, stream);
}
