// Nugget attention for a few query vectors that read the same K/V rows, on the matrix cores (Eq. 13 / Eq. 9 of
// the Dodo paper with q_b small): the G query heads of one KV head (grouped-query attention) times the rows of a
// small query block -- at most 32 vectors, the width of one MFMA tile.  bf16, d_h = 128 or 64 (a template
// parameter: tile sizes, LDS layout and fragment counts follow from it).
//
// The work is bandwidth-bound (every K and V row is read once, and serves all the vectors), so the layout is built
// around keeping loads in flight: a workgroup owns one (sequence, KV head, split); each of its wavefronts streams
// its own share of the keys, 32 at a time, through a private two-stage LDS buffer filled by direct global->LDS
// loads -- no workgroup barrier in the loop, the wavefront's own vmcnt is all the synchronisation there is.  Per 32
// keys and wavefront:
//   S^T = K Q^T     8 x v_mfma_f32_32x32x16_bf16, A = K rows (LDS), B = Q^T (registers): lane <-> query vector
//   online softmax in base 2 on the accumulators (row statistics are lane-local, one exchange with lane^32)
//   O^T += V^T P^T  16 MFMAs, A = V^T through the transposing LDS read, B = P^T straight from the accumulators, in two parts (or three)
// Up to 16 vectors take v_mfma_f32_16x16x32_bf16 instead: half of the matrix work, exponentials and registers.
// (the LDS swizzles and the k-slot <-> key permutation are those of the query-block kernel).  The wavefronts'
// partial (m, l, O) meet in LDS and are merged in wavefront order; with several splits the workgroup writes a
// partial record and the last split merges the records in split order, as in the split-K kernel (same workspace
// format), so results are deterministic.
//
// What bounds it: memory, from about 20 us on; below, the start (2 us of launch, 3 to 4 until the first tiles of all compute
// units are there), and where keys are split the merge.  Narrow tiles, query vectors through LDS (so that the first tile is
// not waited for together with the second), no request past a wavefront's last tile, merges of four channels per thread and
// split counts by expected time, before / after, 64 heads over 8, caches in turn: 16 sequences of 667 rows 21.6 -> 14.8 us, 24 of 667
// 31.2 -> 17.1, 33 of 1897 72.4 -> 58.4, 96 of 667 58.5 -> 48.6, 64 of 667 36.0 -> 33.3 (5.2 TB/s); 4 query rows of 32 heads, 8 sequences of
// 667 rows 27.3 -> 17.9.
#include <algorithm>
#include <type_traits>

#include "dodo_attn.h"

namespace dodo {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short shortx4;
typedef __attribute__((ext_vector_type(8))) float floatx8;
typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kKeys = 32;        // keys per tile
constexpr int kMaxVectors = 32;  // query vectors per workgroup: the N side of one MFMA tile, which is NV = 32 or 16 wide
// What follows from the head size DH (128 or 64) and the width NV of the MFMA tiles
template <int DH, int NV>
struct GroupDims {
  static constexpr int kRowBytes = DH * 2;
  static constexpr int kP = kRowBytes / 16;           // 16-byte pieces of a row
  static constexpr int kPLog2 = DH == 128 ? 4 : 3;
  // rows of 128 bytes cover half of the LDS banks: two consecutive rows sit side by side and the swizzles take the
  // row's index from bit 1 on; rows of 256 bytes use the index as it is
  static constexpr int kRowShift = DH == 128 ? 0 : 1;
  static constexpr int kCB = DH / NV;                 // blocks of NV channels of O^T, each a granule of 2 NV bytes of a V row
  static constexpr int kGranPieces = NV / 8;          // 16-byte pieces of a granule
  static constexpr int kSteps = DH * NV / 512;        // 16-byte fragments of a query vector per lane: MFMAs of S^T per key block
  static constexpr int kKeyBlocks = kKeys / NV;       // key blocks of S^T per tile
  static constexpr int kPvSteps = NV / 16;            // MFMAs of O^T per tile and channel block (32 / their depth in keys)
  static constexpr int kRowsPerInstr = 64 / kP;       // a load instruction brings 1 KiB: 4 or 8 rows
  static constexpr int kInstrPerTensor = kKeys / kRowsPerInstr;
  static constexpr int kTensorBytes = kKeys * kRowBytes;  // K or V part of a stage: 8 or 4 KiB
  static constexpr int kStageBytes = 2 * kTensorBytes;
  static constexpr int kWaveLds = 2 * kStageBytes;        // two stages per wavefront: 32 or 16 KiB
  static constexpr int kQBytes = NV * kRowBytes;          // the workgroup's query vectors, behind the wavefronts' stages
  static constexpr int kLoadsPerTile = 2 * kInstrPerTensor;
  static constexpr int kPartStride = DH + 4;              // floats per vector of a partial in LDS (spreads the banks)
  static constexpr int kPartBytes = (NV * kPartStride + 2 * NV) * 4;  // a partial: O, then m and l
  // splits of the keys of a (sequence, KV head) pair over workgroups: the last split's staging (one float per
  // vector and other split in each of the first two wavefronts' regions, behind the partials) bounds their number
  static constexpr int kMaxSplits = DH == 128 ? 64 : 32;
  static_assert(kPartBytes + (NV * (kMaxSplits - 1) + 3 * NV) * 4 <= kWaveLds, "the merge's staging fits behind the partials");
};
constexpr float kNegInf = -__builtin_inff();

__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }  // exp2(-inf) = 0
constexpr int vmcnt_imm(int n) { return 0x0f70 | (n & 15) | ((n >> 4) << 14); }         // s_waitcnt vmcnt(n) only

typedef __attribute__((ext_vector_type(4))) float floatx4;
template <int NV>
struct Mfma;  // accumulator of NV x NV floats; a product is 16 (NV = 32) or 32 (NV = 16) deep
template <>
struct Mfma<32> {
  typedef floatx16 Acc;
  static constexpr int kRegs = 16;
  __device__ static __forceinline__ Acc mul(const bf16x8& a, const bf16x8& b, const Acc& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma<16> {
  typedef floatx4 Acc;
  static constexpr int kRegs = 4;
  __device__ static __forceinline__ Acc mul(const bf16x8& a, const bf16x8& b, const Acc& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// Largest / sum of x over the lanes of a query vector (the lanes of equal index modulo NV).
template <int NV>
__device__ __forceinline__ float vector_max(float x) {
  float a, b;
  if (NV == 16) {
    lane_pair<16>(x, a, b);
    x = fmaxf(a, b);
  }
  lane_pair<32>(x, a, b);
  return fmaxf(a, b);
}
template <int NV>
__device__ __forceinline__ float vector_sum(float x) {
  float a, b;
  if (NV == 16) {
    lane_pair<16>(x, a, b);
    x = a + b;
  }
  lane_pair<32>(x, a, b);
  return a + b;
}

// Online-softmax update for one 32-key tile.  acc holds the raw S^T accumulators: register v <-> key 8 (v / 4) + 4 g + v % 4
// (NV = 32, g = lane / 32) or 16 (v / 4) + 4 g + v % 4 (NV = 16, g = lane / 16).  MASK: keys at or beyond `limit` are masked.
// Returns P^T as the MFMA B operands (NV = 32: k-step t covers keys 16t .. 16t+15) in PARTS parts: the weights' upper 8 bits of
// mantissa, and what they lack, in bf16 again.  With two they count with 16 bits, and O's error is that of its own rounding to
// bf16 (2-norm against 64 bits 1.66e-3; 2.1e-3 to 2.3e-3 with weights rounded to bf16); the matrix pipe, which is idle three
// quarters of the time here, does twice the work for V (64 sequences of 667 rows, 64 heads over 8: 32.4 -> 33.3 us).  With three they
// are whole, as in the split-K kernel: calls that come here only to be faster than there have these (with two, one value of O in 250
// rounded to another neighbour than the 64-bit result does, with three one in 6000, as there; 6 sequences of 357 rows, 64 heads over 8
// 6.6 -> 6.7 us, 14 of 457 9.2 -> 9.6).  No part of a weight is negative, nor zero unless the weight is: with an
// infinity in V their products are that infinity.
// The exponent offset m_run of a vector is moved (and its sum and output accumulators rescaled) only when the tile's
// maximum exceeds it by more than kSlack: the result does not depend on the offset, the weights stay below
// 2^kSlack, and after the first tiles of a vector the output accumulators are hardly ever touched again (the rescale is
// a wavefront-uniform branch: taken if any vector of the wavefront moves).
constexpr float kSlack = 8.f;
template <bool MASK, int NV, int CB, int REGS, int PARTS>
__device__ __forceinline__ void softmax_tile32(float (&acc)[REGS], int limit, int g, float scale_log2e, float& m_run,
                                               float& l_run, typename Mfma<NV>::Acc (&acc_o)[CB], bf16x8 (&pf)[PARTS][REGS / 8]) {
  float tmax = kNegInf;
#pragma unroll
  for (int v = 0; v < REGS; ++v) {
    float s = acc[v] * scale_log2e;
    if (MASK) {
      const int key = (NV == 32 ? 8 : 16) * (v >> 2) + 4 * g + (v & 3);
      s = (key < limit) ? s : kNegInf;
    }
    acc[v] = s;
    tmax = fmaxf(tmax, s);
  }
  tmax = vector_max<NV>(tmax);                // all lanes of a vector decide alike
  const bool move = tmax > m_run + kSlack;  // (m_run = -inf: any finite maximum moves it)
  if (__any(move)) {
    const float m_new = move ? tmax : m_run;
    const float alpha = exp2_hw(m_run - ((m_new == kNegInf) ? 0.f : m_new));  // 1 where nothing moves, 0 from -inf
    l_run *= alpha;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int v = 0; v < Mfma<NV>::kRegs; ++v) acc_o[cb][v] *= alpha;
    m_run = m_new;
  }
  const float m_use = (m_run == kNegInf) ? 0.f : m_run;
  float psum = 0.f;
#pragma unroll
  for (int half = 0; half < REGS / 8; ++half) {
    floatx8 low;
    uint32_t high[PARTS - 1][4];
#pragma unroll
    for (int v = 0; v < 8; v += 2) {
      const float p0 = exp2_hw(acc[8 * half + v] - m_use), p1 = exp2_hw(acc[8 * half + v + 1] - m_use);
      psum += p0;
      psum += p1;
      float r0 = p0, r1 = p1;
#pragma unroll
      for (int part = 0; part < PARTS - 1; ++part) {
        const uint32_t b0 = __float_as_uint(r0), b1 = __float_as_uint(r1);
        high[part][v / 2] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);  // the upper halves: rounded towards zero
        r0 = __builtin_amdgcn_fmed3f(r0 - __uint_as_float(b0 & 0xffff0000u), 1e-30f, p0);
        r1 = __builtin_amdgcn_fmed3f(r1 - __uint_as_float(b1 & 0xffff0000u), 1e-30f, p1);
      }
      low[v] = r0;
      low[v + 1] = r1;
    }
#pragma unroll
    for (int part = 0; part < PARTS - 1; ++part)
      pf[part][half] = __builtin_bit_cast(bf16x8, make_uint4(high[part][0], high[part][1], high[part][2], high[part][3]));
    pf[PARTS - 1][half] = __builtin_convertvector(low, bf16x8);  // hardware round-to-nearest-even pack
  }
  l_run += psum;
}

// NWV wavefronts per workgroup; STREAM: K/V rows with the non-temporal hint; NV: width of the MFMA tiles; PARTS: of a weight.
// Grid: (KV head, sequence, split).
template <int DH, int NWV, bool STREAM, int NV, int PARTS>
__global__ __launch_bounds__(NWV * kWave) void group_attention_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ Kn, const uint16_t* __restrict__ Vn,
    const uint16_t* __restrict__ Kl, const uint16_t* __restrict__ Vl, const int32_t* __restrict__ cu_q,
    const int32_t* __restrict__ cu_nuggets, const int32_t* __restrict__ nug_len, const int32_t* __restrict__ cu_local,
    const int32_t* __restrict__ loc_len, int H, int H_kv, int G, FastDiv div_G, int max_q, int row0, int rows_per,
    int nsplit,
    int64_t nug_tok_stride, int64_t nug_head_stride, float scale_log2e, uint16_t* __restrict__ O,
    float* __restrict__ lse, float* __restrict__ ws, uint32_t* __restrict__ flags) {
  using GD = GroupDims<DH, NV>;
  using Acc = typename Mfma<NV>::Acc;
  constexpr int kDH = DH, kRowBytes = GD::kRowBytes, kP = GD::kP, kRowShift = GD::kRowShift, kCB = GD::kCB, kSteps = GD::kSteps;
  constexpr int kTensorBytes = GD::kTensorBytes, kStageBytes = GD::kStageBytes, kWaveLds = GD::kWaveLds;
  constexpr int kPartStride = GD::kPartStride, kPartBytes = GD::kPartBytes, kMaxSplits = GD::kMaxSplits;
  constexpr int kInstr = GD::kInstrPerTensor, kLoads = GD::kLoadsPerTile, kRowsPerInstr = GD::kRowsPerInstr;
  constexpr int kThreads = NWV * kWave;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  // all arguments in one round of scalar loads, then all of the sequence's boundaries
  asm volatile("" ::"s"(Q), "s"(Kn), "s"(Vn), "s"(Kl), "s"(Vl), "s"(cu_q), "s"(cu_nuggets), "s"(nug_len), "s"(cu_local),
               "s"(loc_len), "s"(H), "s"(H_kv), "s"(G), "s"(div_G.mul), "s"(div_G.shift), "s"(max_q), "s"(row0), "s"(rows_per),
               "s"(nsplit), "s"(nug_tok_stride), "s"(nug_head_stride), "s"(scale_log2e));
  const int kvh = blockIdx.x, b = blockIdx.y, split = blockIdx.z;

  const int32_t* k_end_p = nug_len != nullptr ? nug_len + b : cu_nuggets + b + 1;
  const int32_t* l_end_p = loc_len != nullptr ? loc_len + b : cu_local + b + 1;
  const int q0 = cu_q[b], q_end = cu_q[b + 1];
  const int k0 = cu_nuggets[b], k_end = *k_end_p;
  const int l0 = cu_local[b], l_end = *l_end_p;
  asm volatile("" ::"s"(q0), "s"(q_end), "s"(k0), "s"(k_end), "s"(l0), "s"(l_end));  // one round of loads
  const int q_b = min(q_end - q0, max_q);  // query rows of the sequence; this launch takes rows row0 .. row0 + rows_per
  const int k_b = nug_len != nullptr ? k_end : k_end - k0;
  const int m_b = loc_len != nullptr ? l_end : l_end - l0;
  if (q_b <= row0) return;  // uniform over the workgroup and over the splits: nothing to write, nothing to wait for
  const int q_cnt = min(rows_per, q_b - row0);

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave;
  const int j = lane % NV, g = lane / NV;
  const int nv = q_cnt * G;  // query vectors of this workgroup: vector v = (row row0 + v / G, head kvh * G + v % G)
  const int my_i = row0 + static_cast<int>(fast_div(static_cast<uint32_t>(j < nv ? j : 0), div_G));
  // causal rule, bottom-right aligned: query row i sees local rows j <= m_b - q_b + i (the sequence's last row sees
  // all); the launch's last row bounds the local tiles
  const int wg_vis = max(0, min(m_b, m_b - q_b + row0 + q_cnt));
  const int my_vis = max(0, min(m_b, m_b - q_b + my_i + 1));  // (spare lanes: vector 0's, so that whole tiles need no mask)

  const int n_nug_tiles = (k_b + kKeys - 1) / kKeys;
  const int n_loc_tiles = (wg_vis + kKeys - 1) / kKeys;
  const int n_tiles = n_nug_tiles + n_loc_tiles;
  const int per_split = (n_tiles + nsplit - 1) / nsplit;
  const int t0 = min(n_tiles, split * per_split), t1 = min(n_tiles, t0 + per_split);
  // this wavefront's tiles: t0 + wave, t0 + wave + NWV, ...
  const int first = t0 + wave;
  const int n_mine = first < t1 ? (t1 - first + NWV - 1) / NWV : 0;

  const uint16_t* nugK = Kn + static_cast<int64_t>(k0) * nug_tok_stride + static_cast<int64_t>(kvh) * nug_head_stride;
  const uint16_t* nugV = Vn + static_cast<int64_t>(k0) * nug_tok_stride + static_cast<int64_t>(kvh) * nug_head_stride;
  const int64_t loc_stride = static_cast<int64_t>(H_kv) * kDH;
  const uint16_t* locK = Kl + (static_cast<int64_t>(l0) * H_kv + kvh) * kDH;
  const uint16_t* locV = Vl + (static_cast<int64_t>(l0) * H_kv + kvh) * kDH;

  // Loads: an instruction brings 1 KiB (4 or 8 rows) of K, of V or of the query vectors; the lane at LDS position (row, pos)
  // fetches the 16-byte piece that the swizzle stores there (K and Q: pos ^ r; V: granule (pos / granule) ^ r; r = row >>
  // kRowShift, taken modulo the number of pieces or granules).  They go through a buffer that ends with the tile's last
  // row: what lies beyond fetches nothing and reads as zeros (masked later).
  char* const lds_w = lds + wave * kWaveLds;
  const uint32_t lds_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void*)lds));
  const uint32_t lds_w_addr = lds_addr + static_cast<uint32_t>(wave * kWaveLds);
  const int ld_row0 = lane >> GD::kPLog2;
  const uint32_t ld_pos = lane & (kP - 1);
  auto k_piece_of = [&](int row) -> uint32_t { return (ld_pos ^ ((row >> kRowShift) & (kP - 1))) * 16u; };
  auto v_piece_of = [&](int row) -> uint32_t {
    return (((ld_pos / GD::kGranPieces) ^ ((row >> kRowShift) & (kCB - 1))) * GD::kGranPieces + ld_pos % GD::kGranPieces) * 16u;
  };
  uint32_t k_off[kInstr], v_off[kInstr], off_stride = 0;
  auto issue_tile = [&](int tile, int stage) {
    const bool nug = tile < n_nug_tiles;
    const int base = nug ? tile * kKeys : (tile - n_nug_tiles) * kKeys;
    const int cnt = min(kKeys, (nug ? k_b : m_b) - base);
    const int64_t stride = nug ? nug_tok_stride : loc_stride;
    const uint32_t stride_bytes = static_cast<uint32_t>(stride) * 2u;
    if (off_stride != stride_bytes) {  // (uniform: the first tile, and where the cache's stride is not the local rows')
      off_stride = stride_bytes;
#pragma unroll
      for (int u = 0; u < kInstr; ++u) {
        const int row = ld_row0 + kRowsPerInstr * u;
        k_off[u] = static_cast<uint32_t>(row) * stride_bytes + k_piece_of(row);
        v_off[u] = static_cast<uint32_t>(row) * stride_bytes + v_piece_of(row);
      }
    }
    const uint32_t range = static_cast<uint32_t>(cnt - 1) * stride_bytes + kRowBytes;
    const u32x4_t kbuf = buffer_of((nug ? nugK : locK) + base * stride, range);
    const u32x4_t vbuf = buffer_of((nug ? nugV : locV) + base * stride, range);
    const uint32_t dst = lds_w_addr + stage * kStageBytes;
#pragma unroll
    for (int u = 0; u < kInstr; ++u) {
      dma16_buffer<STREAM>(kbuf, k_off[u], __builtin_amdgcn_readfirstlane(dst + u * 1024));
      dma16_buffer<STREAM>(vbuf, v_off[u], __builtin_amdgcn_readfirstlane(dst + kTensorBytes + u * 1024));
    }
  };

  // The query vectors go through LDS like a tile of K: loads into registers would have the compiler, which does not count the
  // tiles' loads, wait for both tiles in flight before the first product (64 sequences of 667 rows: 5.9 us into the launch).
  // Every wavefront enqueues the same number of loads.
  constexpr int kQInstr = (GD::kQBytes / 1024 + NWV - 1) / NWV;
  {
    // (offsets below 32 rows of the K/V heads' bytes, which group_attention_applies holds below 2^32)
    const u32x4_t qbuf = buffer_of(Q + (static_cast<int64_t>(q0 + row0) * H + kvh * G) * kDH, 0xffffffffu);
#pragma unroll
    for (int u = 0; u < kQInstr; ++u) {
      const int chunk = min(wave * kQInstr + u, GD::kQBytes / 1024 - 1);
      const int v = chunk * kRowsPerInstr + ld_row0, jv = v < nv ? v : 0;  // spare rows repeat vector 0; nothing of them is stored
      const int il = static_cast<int>(fast_div(static_cast<uint32_t>(jv), div_G));
      dma16_buffer(qbuf, static_cast<uint32_t>(il * H + jv - il * G) * kRowBytes + k_piece_of(v),
                   __builtin_amdgcn_readfirstlane(lds_addr + NWV * kWaveLds + chunk * 1024));
    }
  }
  // Two tiles in flight per wavefront
  if (n_mine > 0) issue_tile(first, 0);
  if (n_mine > 1) issue_tile(first + NWV, 1);
  if (n_mine > 1) {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * kLoads));
  } else if (n_mine > 0) {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(kLoads));
  } else {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  }
  __syncthreads();  // every wavefront's part of the query vectors has landed
  // Q^T fragments: lane (j, g) holds 8 channels of its vector from (1024 / NV / 2) ds + 8 g on, for each step ds
  constexpr int kPiecesPerStep = 64 / NV;
  bf16x8 qf[kSteps];
  {
    const char* q_lds = lds + NWV * kWaveLds + j * kRowBytes;
#pragma unroll
    for (int ds = 0; ds < kSteps; ++ds)
      qf[ds] = *reinterpret_cast<const bf16x8*>(q_lds + (((kPiecesPerStep * ds + g) ^ ((j >> kRowShift) & (kP - 1))) << 4));
  }

  Acc acc_o[kCB];
#pragma unroll
  for (int cb = 0; cb < kCB; ++cb)
#pragma unroll
    for (int v = 0; v < Mfma<NV>::kRegs; ++v) acc_o[cb][v] = 0.f;
  float m_run = kNegInf, l_run = 0.f;

  // V^T through the transposing read: 16 lanes read 4 rows of 16 channels, the lane supplies row (lane % 16) / 4 of them,
  // 8 bytes at channel 4 (lane % 4).  NV = 32: rows 16t + 8e + 4g, channels 32cb + 16 ((lane / 16) % 2); NV = 16: rows 16e +
  // 4g, channels 16cb -- the keys of P^T's registers in either case.
  const int v_r = 4 * g + ((lane & 15) >> 2);
  const int v_in = (NV == 32 ? 32 * ((lane >> 4) & 1) : 0) + 8 * (lane & 3);

  for (int n = 0; n < n_mine; ++n) {
    const int tile = first + n * NWV, stage = n & 1;
    if (n + 1 < n_mine) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(kLoads));  // this tile has landed, the next one is in flight
    } else {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    }
    asm volatile("" ::: "memory");
    const char* kbuf = lds_w + stage * kStageBytes;
    const char* vbuf = kbuf + kTensorBytes;
    // all fragment reads of the tile are requested up front
    bf16x8 kf[GD::kKeyBlocks][kSteps], vt[GD::kPvSteps][kCB];
#pragma unroll
    for (int kb = 0; kb < GD::kKeyBlocks; ++kb)
#pragma unroll
      for (int ds = 0; ds < kSteps; ++ds)
        kf[kb][ds] = *reinterpret_cast<const bf16x8*>(kbuf + (NV * kb + j) * kRowBytes +
                                                      (((kPiecesPerStep * ds + g) ^ (((NV * kb + j) >> kRowShift) & (kP - 1))) << 4));
#pragma unroll
    for (int t = 0; t < GD::kPvSteps; ++t)
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) {
        shortx4 a[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int r = 16 * t + (NV == 32 ? 8 : 16) * e + v_r;
          const char* p = vbuf + r * kRowBytes + ((cb ^ ((r >> kRowShift) & (kCB - 1))) * (2 * NV)) + v_in;
          a[e] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p));
        }
        vt[t][cb] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a[0], a[1], 0, 1, 2, 3, 4, 5, 6, 7));
      }
    // with every fragment of the tile in registers its stage is free: the tile after next is requested before the
    // arithmetic, so two tiles are in flight while the wavefront computes
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    if (n + 2 < n_mine) issue_tile(tile + 2 * NWV, stage);
    __builtin_amdgcn_sched_barrier(0);
    Acc acc_s[GD::kKeyBlocks];
#pragma unroll
    for (int kb = 0; kb < GD::kKeyBlocks; ++kb)
#pragma unroll
      for (int v = 0; v < Mfma<NV>::kRegs; ++v) acc_s[kb][v] = 0.f;
#pragma unroll
    for (int ds = 0; ds < kSteps; ++ds)
#pragma unroll
      for (int kb = 0; kb < GD::kKeyBlocks; ++kb) acc_s[kb] = Mfma<NV>::mul(kf[kb][ds], qf[ds], acc_s[kb]);
    const bool nug = tile < n_nug_tiles;
    const int base = nug ? tile * kKeys : (tile - n_nug_tiles) * kKeys;
    const int limit = nug ? k_b - base : my_vis - base;  // keys [0, limit) of the tile are visible to this lane's vector
    constexpr int kRegs = GD::kKeyBlocks * Mfma<NV>::kRegs;
    float sv[kRegs];
#pragma unroll
    for (int v = 0; v < kRegs; ++v) sv[v] = acc_s[v / Mfma<NV>::kRegs][v % Mfma<NV>::kRegs];
    bf16x8 pf[PARTS][kRegs / 8];
    if (__all(limit >= kKeys)) {
      softmax_tile32<false, NV>(sv, limit, g, scale_log2e, m_run, l_run, acc_o, pf);
    } else {
      softmax_tile32<true, NV>(sv, limit, g, scale_log2e, m_run, l_run, acc_o, pf);
    }
#pragma unroll
    for (int part = 0; part < PARTS; ++part)
#pragma unroll
      for (int t = 0; t < GD::kPvSteps; ++t)
#pragma unroll
        for (int cb = 0; cb < kCB; ++cb) acc_o[cb] = Mfma<NV>::mul(vt[t][cb], pf[part][t], acc_o[cb]);
  }

  // ---- the wavefronts' partials meet in LDS: [vector][channel] floats, then m and l per vector ----
  // lane (j, g) holds channels 32cb + 8(v/4) + 4g + v%4 (NV = 32) or 16cb + 4g + v (NV = 16) of vector j
  {
    float* part = reinterpret_cast<float*>(lds_w);
    const float l_tot = vector_sum<NV>(l_run);
#pragma unroll
    for (int cb = 0; cb < kCB; ++cb)
#pragma unroll
      for (int qd = 0; qd < Mfma<NV>::kRegs / 4; ++qd)
        *reinterpret_cast<float4*>(part + j * kPartStride + NV * cb + 8 * qd + 4 * g) =
            make_float4(acc_o[cb][4 * qd], acc_o[cb][4 * qd + 1], acc_o[cb][4 * qd + 2], acc_o[cb][4 * qd + 3]);
    if (g == 0) {
      part[NV * kPartStride + j] = m_run;
      part[NV * kPartStride + NV + j] = l_tot;
    }
  }
  __syncthreads();

  // Four neighbouring channels of a vector per thread and step, the wavefronts merged in wavefront order.
  auto merged = [&](int v, int c, float& M, float& S, float4& o) {
    float mw[NWV];
    M = kNegInf;
#pragma unroll
    for (int w = 0; w < NWV; ++w) {
      mw[w] = reinterpret_cast<const float*>(lds + w * kWaveLds)[NV * kPartStride + v];
      M = fmaxf(M, mw[w]);
    }
    S = 0.f;
    o = make_float4(0.f, 0.f, 0.f, 0.f);
    if (M != kNegInf) {
#pragma unroll
      for (int w = 0; w < NWV; ++w) {
        const float* part = reinterpret_cast<const float*>(lds + w * kWaveLds);
        const float wgt = exp2_hw(mw[w] - M);
        S = fmaf(part[NV * kPartStride + NV + v], wgt, S);
        const float4 p = *reinterpret_cast<const float4*>(part + v * kPartStride + c);
        o.x = fmaf(p.x, wgt, o.x); o.y = fmaf(p.y, wgt, o.y); o.z = fmaf(p.z, wgt, o.z); o.w = fmaf(p.w, wgt, o.w);
      }
    }
  };
  auto out_row_of = [&](int v, int& i_out, int& h_out) -> int64_t {
    const int il = static_cast<int>(fast_div(static_cast<uint32_t>(v), div_G));
    i_out = row0 + il;
    h_out = kvh * G + (v - il * G);
    return static_cast<int64_t>(q0 + i_out) * H + h_out;
  };
  // (S, lse_m: the row's sum and exponent offset; NaN everywhere if a partial is missing)
  auto store_out = [&](int v, int c, const float4& o, float S, float lse_m, bool whole) {
    int i_out, h_out;
    const int64_t out_row = out_row_of(v, i_out, h_out);
    const float nan = __builtin_nanf("");
    auto val = [&](float x) { return !whole ? nan : (S > 0.f) ? x / S : 0.f; };
    *reinterpret_cast<uint2*>(O + out_row * kDH + c) = make_uint2(pack_bf16(val(o.x), val(o.y)), pack_bf16(val(o.z), val(o.w)));
    if (lse != nullptr && c == 0) lse[out_row] = !whole ? nan : (S > 0.f) ? (lse_m + __log2f(S)) * 0.6931471805599453f : kNegInf;
  };
  const int n_quads = nv * (kDH / 4);

  if (nsplit == 1) {
    for (int e = tid; e < n_quads; e += kThreads) {
      const int v = e / (kDH / 4), c = 4 * (e % (kDH / 4));
      float M, S;
      float4 o;
      merged(v, c, M, S, o);
      store_out(v, c, o, S, M, true);
    }
    return;
  }

  // ---- several splits: partial records [m, s, o[0..DH)] per (sequence, row, head, split); the last split
  // waits for the others' flags and merges in split order (device-scope accesses, as in the split-K kernel) ----
  const int64_t b_row0 = static_cast<int64_t>(b) * max_q;
  constexpr int kRecWords = partial_floats<kDH>() / 2;  // a record in 8-byte words, as it is read and written
  auto row_slot = [&](int v) -> int64_t {
    int i_out, h_out;
    out_row_of(v, i_out, h_out);
    return ((b_row0 + i_out) * H + h_out) * nsplit;
  };
  auto word_of = [](float lo, float hi) -> uint64_t { return static_cast<uint64_t>(__float_as_uint(hi)) << 32 | __float_as_uint(lo); };
  auto lo_of = [](uint64_t w) -> float { return __uint_as_float(static_cast<uint32_t>(w)); };
  auto hi_of = [](uint64_t w) -> float { return __uint_as_float(static_cast<uint32_t>(w >> 32)); };
  uint64_t* const recs = reinterpret_cast<uint64_t*>(ws);
  if (split + 1 < nsplit) {
    for (int e = tid; e < n_quads; e += kThreads) {
      const int v = e / (kDH / 4), c = 4 * (e % (kDH / 4));
      float M, S;
      float4 o;
      merged(v, c, M, S, o);
      uint64_t* rec = recs + (row_slot(v) + split) * kRecWords;
      if (c == 0) __hip_atomic_store(rec, word_of(M, S), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(rec + 1 + c / 2, word_of(o.x, o.y), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(rec + 2 + c / 2, word_of(o.z, o.w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // this thread's stores are acknowledged
    __syncthreads();
    if (tid < nv)
      __hip_atomic_store(flags + row_slot(tid) + split, kPartialReady, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  // ---- the last split ----
  // (1) All flags are polled at once (one per thread and round: a device-scope load is a round trip past the
  // XCD's L2); the thread that sees the flag of (vector, split) fetches that record's m and s right away.  They go
  // to LDS behind the wavefronts' partials (room for NV vectors x kMaxSplits - 1 splits in each of the first two regions).
  float* const st_m = reinterpret_cast<float*>(lds + kPartBytes);
  float* const st_s = reinterpret_cast<float*>(lds + kWaveLds + kPartBytes);
  float* const tot_s = st_m + NV * (kMaxSplits - 1);  // per vector: the total sum and the weight of the own partial
  float* const own_w = tot_s + NV;
  float* const tot_m = own_w + NV;
  const int ns1 = nsplit - 1;
  const int n_flags = nv * ns1;
  int ok = 1;
  for (int f = tid; f < n_flags; f += kThreads) {
    const int v = f / ns1, sp = f - v * ns1;
    const int64_t slot = row_slot(v) + sp;
    int polls = 0;
    while (__hip_atomic_load(flags + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != kPartialReady) {
      if (++polls > kMaxPolls) {
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    const uint64_t ms = __hip_atomic_load(recs + slot * kRecWords, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    st_m[f] = lo_of(ms);
    st_s[f] = hi_of(ms);
  }
  const bool complete = __syncthreads_and(ok) != 0;
  // (2) One thread per vector: the total maximum, every partial's weight (kept where its maximum was) and the total
  // sum, added in split order with the own partial (the last split) last.
  if (tid < nv) {
    const int v = tid;
    float M_own, S_own;
    float4 unused;
    merged(v, 0, M_own, S_own, unused);
    float M = M_own;
    for (int sp = 0; sp < ns1; ++sp) M = fmaxf(M, st_m[v * ns1 + sp]);
    float S = 0.f;
    for (int sp = 0; sp < ns1; ++sp) {
      const float w = (M == kNegInf) ? 0.f : exp2_hw(st_m[v * ns1 + sp] - M);
      st_m[v * ns1 + sp] = w;
      S = fmaf(st_s[v * ns1 + sp], w, S);
    }
    const float w_own = (M == kNegInf) ? 0.f : exp2_hw(M_own - M);
    tot_s[v] = fmaf(S_own, w_own, S);
    own_w[v] = w_own;
    tot_m[v] = M;
  }
  __syncthreads();
  // (3) Outputs: four neighbouring channels of a vector per thread and step; the records of STEPS steps and up to BATCH
  // splits are requested before the first is used, so the merge costs a few round trips, not one per record.  (No more
  // requests than that: 64 whatever the count made the merge of two splits 4 of a call's 20 us.)
  auto merge_outputs = [&](auto steps_tag, auto batch_tag) {
    constexpr int STEPS = decltype(steps_tag)::value, BATCH = decltype(batch_tag)::value;
    for (int e0 = tid; e0 < n_quads; e0 += STEPS * kThreads) {
      int vv[STEPS], cc[STEPS];
      const uint64_t* rec[STEPS];
      float4 acc[STEPS];
#pragma unroll
      for (int k = 0; k < STEPS; ++k) {
        const int e = e0 + k * kThreads;
        const int ee = e < n_quads ? e : e0;  // spare steps repeat the first one; nothing of them is stored
        vv[k] = ee / (kDH / 4);
        cc[k] = 4 * (ee % (kDH / 4));
        rec[k] = recs + row_slot(vv[k]) * kRecWords + 1 + cc[k] / 2;
        acc[k] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
      for (int s0 = 0; s0 < ns1; s0 += BATCH) {
        uint64_t w0[STEPS][BATCH], w1[STEPS][BATCH];
#pragma unroll
        for (int k = 0; k < STEPS; ++k)
#pragma unroll
          for (int u = 0; u < BATCH; ++u) {
            const uint64_t* r = rec[k] + static_cast<int64_t>(min(s0 + u, ns1 - 1)) * kRecWords;
            w0[k][u] = __hip_atomic_load(r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            w1[k][u] = __hip_atomic_load(r + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
#pragma unroll
        for (int k = 0; k < STEPS; ++k)
#pragma unroll
          for (int u = 0; u < BATCH; ++u)
            if (s0 + u < ns1) {
              const float w = st_m[vv[k] * ns1 + s0 + u];
              acc[k].x = fmaf(lo_of(w0[k][u]), w, acc[k].x);
              acc[k].y = fmaf(hi_of(w0[k][u]), w, acc[k].y);
              acc[k].z = fmaf(lo_of(w1[k][u]), w, acc[k].z);
              acc[k].w = fmaf(hi_of(w1[k][u]), w, acc[k].w);
            }
      }
#pragma unroll
      for (int k = 0; k < STEPS; ++k) {
        if (e0 + k * kThreads >= n_quads) continue;
        const int v = vv[k], c = cc[k];
        float M_own, S_own;
        float4 o;
        merged(v, c, M_own, S_own, o);
        const float w = own_w[v];
        o.x = fmaf(o.x, w, acc[k].x); o.y = fmaf(o.y, w, acc[k].y); o.z = fmaf(o.z, w, acc[k].z); o.w = fmaf(o.w, w, acc[k].w);
        store_out(v, c, o, tot_s[v], tot_m[v], complete);  // (a partial never arrived: fail loudly)
      }
    }
  };
  if (ns1 == 1) {
    merge_outputs(std::integral_constant<int, 2>{}, std::integral_constant<int, 1>{});
  } else if (ns1 <= 4) {
    merge_outputs(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
  } else {
    merge_outputs(std::integral_constant<int, 2>{}, std::integral_constant<int, 16>{});
  }
  // the flags are left cleared for the next call on this workspace
  for (int f = tid; f < n_flags; f += kThreads) {
    const int v = f / ns1, sp = f - v * ns1;
    __hip_atomic_store(flags + row_slot(v) + sp, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

template <int DH, int NWV, bool STREAM, int NV, int PARTS>
int launch_nwv(const AttnParams& p, int row0, int rows_per, int nsplit, uint32_t* flags) {
  constexpr int kLds = NWV * GroupDims<DH, NV>::kWaveLds + GroupDims<DH, NV>::kQBytes;
  const auto kernel = &group_attention_kernel<DH, NWV, STREAM, NV, PARTS>;
  const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), kLds);
  if (rc != DODO_OK) return rc;
  const int G = p.H / p.H_kv;
  const dim3 grid(static_cast<unsigned>(p.H_kv), static_cast<unsigned>(p.B), static_cast<unsigned>(nsplit));
  hipLaunchKernelGGL(kernel, grid, dim3(NWV * kWave), kLds, p.stream,
                     static_cast<const uint16_t*>(p.Q), static_cast<const uint16_t*>(p.Kn),
                     static_cast<const uint16_t*>(p.Vn), static_cast<const uint16_t*>(p.Kl),
                     static_cast<const uint16_t*>(p.Vl), p.cu_q, p.cu_nuggets, p.nug_len, p.cu_local, p.loc_len, p.H,
                     p.H_kv, G, make_fast_div(static_cast<uint32_t>(G)), p.max_q, row0, rows_per, nsplit, p.nug_tok_stride,
                     p.nug_head_stride, p.scale_log2e, static_cast<uint16_t*>(p.O), p.lse, static_cast<float*>(p.ws),
                     flags);
  return launch_status();
}

template <int DH, int NV, int PARTS>
int launch_dh(const AttnParams& p, bool two, bool stream, int row0, int rows_per, int nsplit, uint32_t* flags) {
  if (stream) {
    return two ? launch_nwv<DH, 2, true, NV, PARTS>(p, row0, rows_per, nsplit, flags) : launch_nwv<DH, 4, true, NV, PARTS>(p, row0, rows_per, nsplit, flags);
  }
  return two ? launch_nwv<DH, 2, false, NV, PARTS>(p, row0, rows_per, nsplit, flags) : launch_nwv<DH, 4, false, NV, PARTS>(p, row0, rows_per, nsplit, flags);
}

// Whether the K/V rows are requested with the non-temporal hint: where the call reads them once and they are more than a quarter
// of the 256 MB last-level cache, so that little of them would be found there by the next call (another layer as a rule).
// 64 heads over 8, caches in turn, plain / hint: 32 sequences of 667 rows (87 MB), four or more caches 19.8 / 17.7 us, three
// or fewer 17.2 / 17.1; 14 of 1897 (109 MB) three or more 26.4 / 24.0, fewer 22.7 / 23.5; 64 of 667 (175 MB) 36.1 / 32.6.
// Below that a cache that stays resident loses more (16 of 667, 44 MB, up to four 11.8 / 13.4, eight 14.5 / 13.5), and so do
// calls of several passes (64 sequences, 15 query rows 154.6 / 156.8).  The bounds count a sequence's rows as its own, which
// those of segments are not: the segments of a text share its nuggets and overlap in its local rows (4 texts of 4096 tokens in
// segments of 8, 295 MB of rows counted as 18 GB: 1599 -> 1686 us with the hint; 2 of 2048 117 -> 123).  In the cached form max_k
// may be a capacity far above the fill, so it takes half of the cache there: 64 caches of 2048 rows full 116 -> 97 us, half full
// 70 -> 60, a tenth full 30.2 -> 27.6 (4 layers in turn); 16 caches of 4096 a tenth full, 4 layers in turn 20.3 -> 21.0, 8 layers
// 22.0 -> 21.1; 64 of 2048 with 20 rows each, 4 layers in turn 14.2 -> 15.9, one layer 13.3 -> 12.5.
bool streams_rows(const AttnParams& p, int rows_per) {
  if (p.loc_len != nullptr) return false;  // the segment form
  const int64_t bytes = static_cast<int64_t>(p.B) * (static_cast<int64_t>(p.max_k) + p.max_local) * p.H_kv * p.d_h * 4;
  return p.max_q <= rows_per && bytes >= (p.nug_len != nullptr ? 128ll << 20 : 64ll << 20);
}

int64_t most_splits(const AttnParams& p) { return p.d_h == 128 ? GroupDims<128, 32>::kMaxSplits : GroupDims<64, 32>::kMaxSplits; }

// Splits for these bounds, if the workspace were no limit: the count of least expected time.  A compute unit that has the memory
// system to itself streams a 32-key tile of 16 KiB in 440 ns; with all units at it, the memory gives each a tile in 660.
// Units run their workgroups side by side and at the same pace, so while some have a workgroup more than the others they go on
// alone with it: 264 workgroups take as long as 512 (33 sequences over 8 KV heads, 1897 rows, whole / in two / three / four:
// 63.5 / 57.8 / 54.0 / 53.4 us; 667 rows 28.0 / 28.6 / 27.1 / 27.4, where 24 sequences take 16.9 whole and 20.8 in two).
// Merging costs 5 us (up to five splits; beyond, 6 and 0.3 for every one over four): 8 sequences, 1897 rows 27.9 whole, 20.9 / 20.1 /
// 18.7 in 2 / 3 / 4, 24.1 in 8; 667 rows 10.6 whole, 11.1 in two; 2 sequences, 1897 rows 19.8 / 15.5 / 14.5 / 12.7 in 1 / 2 / 3 / 4, 13.4
// in 8, 14.3 in 13.
struct Wanted {
  int64_t splits, ns;  // and the time
};
Wanted wanted(const AttnParams& p) {
  const int64_t pairs = static_cast<int64_t>(p.B) * p.H_kv, cus = compute_units();
  const int64_t tiles = (static_cast<int64_t>(p.max_k) + kKeys - 1) / kKeys + (static_cast<int64_t>(p.max_local) + kKeys - 1) / kKeys;
  const int64_t most = most_splits(p);
  const int64_t alone_ns = p.d_h == 128 ? 440 : 220, shared_ns = p.d_h == 128 ? 660 : 330;
  Wanted best{1, 0};
  for (int64_t n = 1; n <= most && (n == 1 || (4 * n <= tiles && n * pairs <= 8 * cus)); ++n) {
    const int64_t rounds = (n * pairs + cus - 1) / cus, rest = n * pairs - (rounds - 1) * cus;  // `rest` units have one more
    const int64_t last_ns = std::max(alone_ns, shared_ns * rest / cus);
    const int64_t t = (tiles + n - 1) / n * ((rounds - 1) * shared_ns + last_ns) + (n == 1 ? 0 : n <= 5 ? 5000 : 6000 + 300 * (n - 4));
    if (n == 1 || t < best.ns) best = Wanted{n, t};
  }
  return best;
}

// Splits that the caller's workspace has records for (none if it is not 8-byte aligned: records are read in 8-byte words).
int64_t splits_that_fit(const AttnParams& p) {
  const int64_t records_per_split = static_cast<int64_t>(p.B) * p.max_q * p.H;
  int64_t fit;
  if (p.ws_flags != nullptr) {  // records and flags in separate regions of ws_slots entries each
    fit = p.ws_slots / records_per_split;
  } else {  // one region: records of d_h + 2 floats, then a flag each
    const bool usable = p.ws != nullptr && (reinterpret_cast<uintptr_t>(p.ws) & 7) == 0;
    fit = usable ? static_cast<int64_t>(p.ws_bytes / (records_per_split * (p.d_h + 3) * sizeof(float))) : 0;
  }
  return fit;
}

// Splits of eight tiles or more that would make a workgroup for every compute unit, with at most `fit` (see group_attention_applies).
int64_t routing_splits(const AttnParams& p, int64_t fit) {
  const int64_t cus = compute_units(), pairs = static_cast<int64_t>(p.B) * p.H_kv;
  const int64_t rows = static_cast<int64_t>(p.max_k) + p.max_local, wanted = ((pairs >= cus ? 2 * cus : cus) + pairs - 1) / pairs;
  return std::max<int64_t>(1, std::min({wanted, rows / (8 * kKeys), most_splits(p), fit}));
}
// Whether that is one for every other compute unit at least.
bool fills_units(const AttnParams& p, int64_t fit) {
  return static_cast<int64_t>(p.B) * p.H_kv * routing_splits(p, fit) * 2 >= compute_units();
}
int group_split_count(const AttnParams& p) { return static_cast<int>(std::max<int64_t>(1, std::min(wanted(p).splits, splits_that_fit(p)))); }

}  // namespace

size_t group_workspace_bytes(int32_t B, int32_t H, int32_t H_kv, int32_t d_h, int32_t max_q, int32_t max_k,
                             int32_t max_local) {
  AttnParams p{};
  p.B = B; p.H = H; p.H_kv = H_kv; p.d_h = d_h; p.max_q = max_q; p.max_k = max_k; p.max_local = max_local;
  const int64_t n = std::max(wanted(p).splits, routing_splits(p, most_splits(p)));
  return n <= 1 ? 0 : static_cast<size_t>(B) * max_q * H * static_cast<size_t>(n) * (d_h + 3) * sizeof(float);
}

// Launches that cover the query rows of a call: each takes as many rows as fit the 32 vectors of a tile with G
// heads per row.  0: the kernel does not take such a call (fewer than 4 vectors share a row, more than 32 heads
// per KV head, or more than four passes over the keys, where the K/V rows would be read too often).
int group_launches(int32_t H, int32_t H_kv, int32_t max_q) {
  const int64_t G = H / H_kv;
  if (G > kMaxVectors || G * max_q < 4) return 0;
  const int rows_per = static_cast<int>(kMaxVectors / G);
  const int launches = (max_q + rows_per - 1) / rows_per;
  return launches <= 4 ? launches : 0;
}

bool group_attention_applies(const AttnParams& p) {
  if (p.dtype != DODO_DTYPE_BF16 || (p.d_h != 128 && p.d_h != 64) || p.nug_idx != nullptr) return false;
  if (group_launches(p.H, p.H_kv, p.max_q) == 0) return false;
  if (p.B > 65535) return false;  // second grid dimension
  // a row number times a stride in bytes is kept in 32 bits
  if (p.nug_tok_stride * 2 * kKeys > 0xffffffffLL || static_cast<int64_t>(p.H_kv) * p.d_h * 2 * kKeys > 0xffffffffLL)
    return false;
  // a workgroup for every other compute unit ...
  const int64_t fit = splits_that_fit(p);
  if (fills_units(p, fit)) return true;
  // ... or, where the narrow tiles hold all vectors and the workspace every wanted split, enough vectors times rows for the
  // split-K kernel, which works on each of them, to be the slower one.  It takes 4.5 us and 7.3 ns (5.3 for heads of 64 channels) for
  // each row of a workgroup's share and each workgroup that a compute unit gets, and 2 more where the shares are merged; this kernel 1.5 beyond
  // the time above, or 2.3 with several splits.  64 heads over 8, split-K / this kernel: 4 x 357 rows 7.1 / 7.7 us, 4 x 579 9.3 / 9.4,
  // 4 x 667 9.3 / 10.1, 2 x 1099 11.2 / 10.1, 5 x 454 11.5 / 8.5, 6 x 357 9.8 / 6.7, 13 x 204 11.4 / 6.0; 40 over 8, 2 x 1887 12.0 / 13.7; 32 over 8, 7 x
  // 687 10.4 / 10.9; 32 over 4, 9 x 627 15.7 / 9.8, heads of 64 2 x 3168 11.1 / 13.5, 5 x 1242 9.6 / 8.9.  (Below 128 Ki of vectors times rows little is won.)
  // (One query row per sequence only: rows that a vector does not see are not read there.)
  const int64_t vectors = static_cast<int64_t>(p.H) * p.max_q, rows = static_cast<int64_t>(p.max_k) + p.max_local;
  const Wanted here = wanted(p);
  if (p.max_q > 1 || vectors > 16 * static_cast<int64_t>(p.H_kv) || std::max<int64_t>(1, fit) < here.splits || vectors * p.B * rows < 128 * 1024) return false;
  const int64_t shares = splitk_count(p.B, p.H, p.d_h, p.max_q, p.max_k, p.max_local, p.dtype), cus = compute_units();
  const int64_t splitk_ns = 4500 + (rows + shares - 1) / shares * (p.d_h == 128 ? 73 : 53) / 10 * ((vectors * p.B * shares + cus - 1) / cus) + (shares > 1 ? 2000 : 0);
  if (here.ns + (here.splits > 1 ? 2300 : 1500) > splitk_ns) return false;
  // (a call that the split-K kernel refuses for want of a workspace is refused whichever kernel would take it)
  const int64_t records = vectors * p.B * shares;
  return records == vectors * p.B || rows < 512 || p.ws_flags != nullptr ||
         (p.ws != nullptr && p.ws_bytes >= static_cast<size_t>(records) * splitk_record_bytes(p.d_h));
}

int launch_group_attention(const AttnParams& p) {
  const int nsplit = group_split_count(p);
  uint32_t* flags = p.ws_flags != nullptr
                        ? static_cast<uint32_t*>(p.ws_flags)
                        : reinterpret_cast<uint32_t*>(static_cast<float*>(p.ws) +
                                                      static_cast<int64_t>(p.B) * p.max_q * p.H * nsplit * (p.d_h + 2));
  // Workgroups of four wavefronts, one on a compute unit at a time, where no unit gets a second one, and of narrow tiles where
  // there are many; of two wavefronts, two at a time, otherwise.  (Not by the rows: a bound that says more than there is changes
  // no bit.)  Two / four wavefronts: 8 sequences over 8 KV heads, 667 rows 13.4 / 10.6 us; 33 sequences, 1897 rows in four 53.4 /
  // 61.4, 667 rows whole 28.0 / 29.4; 64 sequences, 357 / 667 / 1897 rows 21.6 / 23.4, 33.3 / 34.4, 82.6 / 78.8; 96 sequences 30.7 /
  // 32.0, 48.3 / 47.0, 127 / 116; wide tiles (4 query rows), 64 sequences, 667 rows 35.3 / 42.2.
  const int64_t wgs = static_cast<int64_t>(p.B) * p.H_kv * nsplit, cus = compute_units();
  const bool narrow_all = static_cast<int64_t>(p.H) * std::min<int64_t>(p.max_q, kMaxVectors / (p.H / p.H_kv)) <= 16 * static_cast<int64_t>(p.H_kv);
  const bool two = wgs > cus && (nsplit > 1 || !narrow_all || 2 * wgs < 5 * cus);
  const int rows_per = kMaxVectors / (p.H / p.H_kv);
  const bool stream = streams_rows(p, rows_per);
  const bool whole = !fills_units(p, splits_that_fit(p));  // weights in three parts: a call that the split-K kernel could take
  for (int row0 = 0; row0 < p.max_q; row0 += rows_per) {  // (records and flags of different rows are apart)
    // the narrow tiles where their 16 columns hold the launch's vectors: half of the matrix work, and half of the registers
    const bool narrow = std::min(rows_per, p.max_q - row0) * (p.H / p.H_kv) <= 16;
    const auto launch = [&](auto dh_tag) {
      constexpr int DH = decltype(dh_tag)::value;
      return !narrow ? launch_dh<DH, 32, 2>(p, two, stream, row0, rows_per, nsplit, flags)
             : whole ? launch_dh<DH, 16, 3>(p, two, stream, row0, rows_per, nsplit, flags)
                     : launch_dh<DH, 16, 2>(p, two, stream, row0, rows_per, nsplit, flags);
    };
    const int rc = p.d_h == 128 ? launch(std::integral_constant<int, 128>{}) : launch(std::integral_constant<int, 64>{});
    if (rc != DODO_OK) return rc;
  }
  return DODO_OK;
}

}  // namespace dodo
