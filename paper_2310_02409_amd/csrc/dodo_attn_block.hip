// Query-block nugget attention on the matrix cores (Eq. 13 / Eq. 9 of the Dodo
// paper): each query row attends over all nuggets of its sequence, then over
// the causally visible part of the local (uncompressed) rows.  bf16 inputs,
// fp32 accumulation, d_h = 128 or 64 (a template parameter: the tile loops, LDS
// layout and fragment counts follow from it).  Inputs must be finite.
//
// Work split: query heads of one K/V head see the same keys, so that the rows of G such
// neighbours (G from 1 to H / H_kv, see plan_blocks) can go through the tiles together:
// row f of the group is head f % G of query row f / G.  One workgroup owns NW*32
// consecutive rows of one (sequence, group); each wavefront owns 32 of them.  Keys arrive in tiles of 64: first the
// dense nugget tiles, then the local tiles up to the causal diagonal.  K and V
// tiles go from global memory straight into LDS (16-byte direct loads issued as
// inline assembly, so that the compiler does not order every later LDS read behind
// all outstanding loads: the tile loops keep that count themselves; several
// tiles in flight), row-major with an XOR swizzle chosen so that both read
// patterns below are conflict-free.  Per tile and wavefront:
//   S^T = K Q^T     v_mfma_f32_32x32x16_bf16, A = K rows (LDS), B = Q^T (registers)
//   online softmax in base 2 on the accumulators: lane <-> query row, so row
//   statistics and rescaling are lane-local; one exchange with lane^32
//   O^T += V^T P^T  A = V^T through the transposing LDS read (ds_read_b64_tr_b16),
//   B = P^T taken straight from the S^T accumulators.
// Re-using the accumulators as the B operand fixes which key sits in which
// k-slot; the V^T reads follow the same permutation, so no data crosses lanes.
//
// A single wavefront runs its MFMA and its softmax (VALU) work one after the
// other, and two wavefronts that share a SIMD drift into the same phase, so the
// matrix pipe idles while both do softmax.  The 8-wavefront kernel therefore
// runs two groups of four wavefronts (one of each per SIMD) half a tile apart,
// separated by workgroup barriers: while one group issues the 32 MFMAs of
// "PV(t-1), then S(t)", the other does the softmax of its tile.  Small query
// blocks (<= 128 rows) use a plain 4-wavefront kernel, where the chip is not full one
// whose wavefronts share 64 rows in pairs, half of a tile's keys each (plan_blocks).
//
// What bounds the 8-wavefront kernel: the two phases are about equally long (cycle
// counter, 3277 nuggets: 1200 cycles of matrix instructions, 1088 of them the pipe's
// own; softmax 920 and tile requests 320 beside them; 75 for the barrier).  Row sums
// from 16x16x32 products (a 33rd block of V^T took twice the matrix cycles), tile
// requests whose limits are the buffer's range instead of clamps per lane, masks by
// bit selects, the row maximum taken in the first tile only: 2048 rows, 103 nuggets,
// 16 x 40 heads 812 -> 772 us (931 -> 981 TFLOP/s); 1024 rows, 3277 nuggets, 2 x 32
// heads 119 -> 113 us; 512 rows, 410 nuggets, 8 x 32 heads 75.5 -> 72.6 us.
#include <algorithm>
#include <type_traits>

#include "dodo_attn.h"

namespace dodo {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short shortx4;
typedef __attribute__((ext_vector_type(8))) short shortx8;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(8))) float floatx8;
typedef __attribute__((ext_vector_type(16))) float floatx16;

constexpr int kBN = 64;   // keys per tile
// What follows from the head size DH (128 or 64)
template <int DH>
struct HeadDims {
  static constexpr int kRowBytes = DH * 2;
  static constexpr int kTileBytes = kBN * kRowBytes;  // 16 KiB (DH = 128) or 8 KiB (DH = 64) per K or V tile
  static constexpr int kPieces = kRowBytes / 16;      // 16-byte pieces of a row
  static constexpr int kPiecesLog2 = DH == 128 ? 4 : 3;
  // Rows of 128 bytes cover half of the LDS banks, so two consecutive rows sit side by side and the swizzles take
  // the row's index from bit 1 on; rows of 256 bytes cover all banks and use the index as it is.
  static constexpr int kRowShift = DH == 128 ? 0 : 1;
  static constexpr int kChannelBlocks = DH / 32;      // 32-channel blocks of O^T = 64-byte granules of a V row
  static constexpr int kSteps = DH / 8;               // MFMAs per tile of S^T = K Q^T (2 key blocks x DH/16), and of
                                                      // O^T += V^T P^T (4 key steps x DH/32 channel blocks)
};
constexpr float kNegInf = -__builtin_inff();

typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  typedef __attribute__((ext_vector_type(2))) float floatx2;
  const floatx2 f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));  // hardware round-to-nearest-even pack
}

// Per-lane part of the tile loads.  A 64 x DH tile is 64 * P pieces of 16 bytes (P = 16 or 8 per row); wavefront
// w of NW fills LDS rows (64/NW)*w ..., 64/P rows (1 KiB) per instruction.  The lane at LDS position
// (row, pos) fetches the piece that the swizzle stores there:
//   K: piece = pos ^ (r & (P-1))                      (16-byte granules, for the 16-byte row reads)
//   V: piece = ((pos/4) ^ (r & (P/4-1)))*4 + pos%4    (64-byte granules, for the transposing reads)
// with r = row >> kRowShift.
template <int NW, int DH>
struct TileLoader {
  static constexpr int kP = HeadDims<DH>::kPieces;
  static constexpr int kRowsPerInstr = 64 / kP;
  static constexpr int kGranMask = HeadDims<DH>::kChannelBlocks - 1;
  static constexpr int kRowShift = HeadDims<DH>::kRowShift;
  static constexpr int kPerWave = (kBN / kRowsPerInstr) / NW;  // load instructions per wavefront per tile and tensor
  int row0;                // LDS row of this lane in the wavefront's first instruction
  uint32_t pos;            // 16-byte position inside the row
  uint32_t v_piece_bytes;  // the V swizzle term is the same for all of the wavefront's instructions
  uint32_t lds_chunk0;     // byte offset of the wavefront's first 1 KiB chunk inside a tile

  __device__ __forceinline__ void init(int wave, int lane) {
    row0 = wave * kPerWave * kRowsPerInstr + (lane >> HeadDims<DH>::kPiecesLog2);
    pos = lane & (kP - 1);
    v_piece_bytes = ((((pos >> 2) ^ ((row0 >> kRowShift) & kGranMask)) << 2) | (pos & 3)) * 16u;
    lds_chunk0 = wave * kPerWave * 1024;
  }
  template <bool IS_V>
  __device__ __forceinline__ uint32_t piece_bytes(int row) const {
    return IS_V ? v_piece_bytes : (pos ^ ((row >> kRowShift) & (kP - 1))) * 16u;
  }
  // Byte offsets of this lane's loads from the tile's first row, `stride_bytes` apart
  template <bool IS_V>
  __device__ __forceinline__ void offsets(uint32_t stride_bytes, uint32_t (&off)[kPerWave]) const {
#pragma unroll
    for (int u = 0; u < kPerWave; ++u) {
      const int row = row0 + kRowsPerInstr * u;
      off[u] = static_cast<uint32_t>(row) * stride_bytes + piece_bytes<IS_V>(row);
    }
  }
  // The same with the rows taken through an index list: row r of the tile is token idx[r] (idx points into LDS at the
  // tile's first entry; rows past the last of `cnt` re-read that one)
  template <bool IS_V>
  __device__ __forceinline__ void offsets_idx(uint32_t stride_bytes, int cnt, const int32_t* idx, uint32_t (&off)[kPerWave]) const {
#pragma unroll
    for (int u = 0; u < kPerWave; ++u) {
      const int row = row0 + kRowsPerInstr * u;
      off[u] = static_cast<uint32_t>(idx[min(row, cnt - 1)]) * stride_bytes + piece_bytes<IS_V>(row);
    }
  }
  // V's offsets from K's of the same rows
  __device__ __forceinline__ void k_to_v(const uint32_t (&k)[kPerWave], uint32_t (&v)[kPerWave]) const {
#pragma unroll
    for (int u = 0; u < kPerWave; ++u) v[u] = k[u] + (v_piece_bytes - piece_bytes<false>(row0 + kRowsPerInstr * u));
  }
  // 64 rows at base + off, requested through a buffer that ends `range` bytes after base: what lies beyond fetches
  // nothing and reads as zeros, so that neither the rows past a tile's last one nor a tile past the last need a test per
  // lane.  Every call enqueues the same number of loads.
  __device__ __forceinline__ void issue(const uint16_t* base, uint32_t range, const uint32_t (&off)[kPerWave], uint32_t lds_dst) const {
    const u32x4_t buf = buffer_of(base, range);
#pragma unroll
    for (int u = 0; u < kPerWave; ++u) dma16_buffer(buf, off[u], __builtin_amdgcn_readfirstlane(lds_dst + lds_chunk0 + u * 1024));
  }
};

// One bit per key of a 32-key block, set for the first `limit` of them (any limit).
__device__ __forceinline__ uint32_t first_keys(int limit) {
  const int n = min(32, max(0, limit));
  return n == 32 ? 0xffffffffu : (1u << n) - 1u;
}
// x where bit `key` (a constant) is set, -inf elsewhere: a field extract and a bit select (a comparison would go through
// the scalar registers, with two idle slots before each select)
__device__ __forceinline__ float visible_or_neg_inf(float x, uint32_t bits, int key) {
  const uint32_t m = static_cast<uint32_t>(static_cast<int32_t>(bits << (31 - key)) >> 31);
  return __uint_as_float((__float_as_uint(x) & m) | (0xff800000u & ~m));
}

// Online-softmax update of one 32-row block for one 64-key tile.  acc holds the raw
// S^T accumulators (two 32-key blocks); accumulator v of block kb <-> key 32kb + 8(v/4) + 4g + v%4.
// Returns P^T as MFMA B operands: pf[2kb + half] = accumulators 8*half .. 8*half+7 of block kb.
template <bool MASK, int NCB, int NKB>
__device__ __forceinline__ void softmax_tile(floatx16 (&acc)[NKB], int limit, int g, float scale_log2e, float& m_run,
                                             float& l_run, floatx16 (&acc_o)[NCB], bf16x8 (&pf)[2 * NKB]) {
  float tmax = kNegInf;
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb) {
    // (the lane's part of the key index, 4 g, is taken off the limit, so that the bits' positions are constants)
    const uint32_t bits = first_keys(limit - 4 * g - 32 * kb);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      float s = acc[kb][v] * scale_log2e;
      if (MASK) s = visible_or_neg_inf(s, bits, 8 * (v >> 2) + (v & 3));
      acc[kb][v] = s;
      tmax = fmaxf(tmax, s);
    }
  }
  tmax = fmaxf(tmax, __shfl_xor(tmax, 32, kWave));
  const float m_new = fmaxf(m_run, tmax);
  const float m_use = (m_new == kNegInf) ? 0.f : m_new;
  float psum = 0.f;
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      floatx8 p;
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        p[v] = exp2_hw(acc[kb][8 * half + v] - m_use);
        psum += p[v];
      }
      pf[2 * kb + half] = __builtin_convertvector(p, bf16x8);  // hardware RNE pack
    }
  // The running sums are rescaled unconditionally: a data-dependent skip would add a branch around
  // 64 live accumulators, which costs more in register copies than the multiplies it saves.
  const float alpha = exp2_hw(m_run - m_use);  // m_run = -inf -> 0
  l_run *= alpha;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc_o[cb][v] *= alpha;
  m_run = m_new;
  l_run += psum;
}

// Keys [0, limit) of the tile are visible to this lane's row.
__device__ __forceinline__ void mask_tile(floatx16 (&acc)[2], int limit, int g) {
  const uint32_t bits[2] = {first_keys(limit - 4 * g), first_keys(limit - 4 * g - 32)};
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[kb][v] = visible_or_neg_inf(acc[kb][v], bits[kb], 8 * (v >> 2) + (v & 3));
}
__device__ __forceinline__ float tile_max(const floatx16 (&acc)[2]) {
  float tmax = kNegInf;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int v = 0; v < 16; ++v) tmax = fmaxf(tmax, acc[kb][v]);
  return fmaxf(tmax, __shfl_xor(tmax, 32, kWave));
}
// Softmax with a fixed exponent offset per row (used by the two-group kernel): the offset m_off is the row maximum of
// the first tile -- every row that sees anything sees keys of it -- and is never moved afterwards, so the output
// accumulators are not rescaled: O = sum(p v) / sum(p) does not depend on the offset.  Logits far above the fixed offset
// show up as a row sum beyond kMostSum (or one that is not finite) at the end, in which case the caller redoes the rows with
// softmax_tile, as it does where every logit of a row's first tile is -inf, which leaves the row no offset.  The sum stays finite
// for a while after sum(p v) has overflowed; below kMostSum that takes values of V beyond 2^63.  Needs scale_log2e > 0.
constexpr float kMostSum = 0x1p64f;
__device__ __forceinline__ void softmax_fixed(const floatx16 (&acc)[2], float scale_log2e, float m_off, bf16x8 (&pf)[4]) {
  const float neg = (m_off == kNegInf) ? 0.f : -m_off;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    floatx8 p;
#pragma unroll
    for (int v = 0; v < 8; ++v) p[v] = exp2_hw(fmaf(acc[i >> 1][8 * (i & 1) + v], scale_log2e, neg));
    pf[i] = __builtin_convertvector(p, bf16x8);  // hardware RNE pack
  }
}

// KG = 1, NW = 4: plain loop, two workgroups per CU.  NW = 8: two groups of four wavefronts in
// alternating MFMA / softmax phases, one workgroup per CU.  KG = 2: plain loop, each 32 rows have two wavefronts, which
// take half of every tile's keys each.
template <int NW, int DH, int KG>
struct BlockCfg {
  static constexpr bool kTwoGroups = NW == 8 && KG == 1;
  static constexpr int kThreads = NW * kWave;
  static constexpr int kBM = NW * 32 / KG;            // query rows per workgroup
  static constexpr int kStages = kTwoGroups ? 4 : 2;  // K/V tiles resident in LDS
  static constexpr int kLdsBytes = kStages * 2 * HeadDims<DH>::kTileBytes;
  static constexpr int kMinBlocks = NW == 4 ? 2 : 1;
  // gather-free form: the sequence's index list sits in LDS after the stages (160 KiB per compute unit in all; the 8-wavefront
  // kernel has 1 KiB of static LDS besides).  Up to kShortIdx entries leave two workgroups of 4 wavefronts room on a compute unit.
  static constexpr int kIdxCap = 7680, kShortIdx = 4096;
  static int idx_entries(int32_t max_k) { return kMinBlocks == 2 && max_k <= kShortIdx ? kShortIdx : kIdxCap; }
  static_assert(kMinBlocks * (kLdsBytes + (kMinBlocks == 2 ? kShortIdx : kIdxCap) * 4) <= 160 * 1024 && kLdsBytes + kIdxCap * 4 <= 159 * 1024,
                "a compute unit has LDS for the workgroups that plan_blocks puts there");
  // KG = 2: the second halves' channels, offsets and sums meet the first halves' in the stages
  static constexpr int kMergeO = NW / 2 * 32 * DH * 4;
  static_assert(KG == 1 || kMergeO + NW / 2 * kWave * 8 <= kLdsBytes, "the merge of the halves fits into the stages");
};

// What a query block needs to know of its sequence: first rows and lengths of its queries, nuggets and local rows
// (and, gather-free form, the first token of its context).  Read with scalar loads by load_seq_geom, for both query
// blocks of a workgroup at the kernel's start, so that no block begins with a chain of dependent loads.
struct SeqGeom {
  int b, grp;
  int q0, q_b, k0, k_b, l0, m_b;
  int64_t ctx0;
};
template <bool IDX>
__device__ __forceinline__ SeqGeom load_seq_geom(int bh, FastDiv div_groups, int n_groups,
                                                 const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_nuggets,
                                                 const int32_t* __restrict__ nug_len, const int32_t* __restrict__ cu_local,
                                                 const int32_t* __restrict__ loc_len, const int32_t* __restrict__ cu_ctx) {
  SeqGeom g;
  g.b = static_cast<int>(fast_div(static_cast<uint32_t>(bh), div_groups));
  g.grp = bh - g.b * n_groups;
  const int32_t* k_end_p = nug_len != nullptr ? nug_len + g.b : cu_nuggets + g.b + 1;
  const int32_t* l_end_p = loc_len != nullptr ? loc_len + g.b : cu_local + g.b + 1;
  g.q0 = cu_q[g.b];
  const int q_end = cu_q[g.b + 1];
  g.k0 = cu_nuggets[g.b];
  const int k_end = *k_end_p;
  g.l0 = cu_local[g.b];
  const int l_end = *l_end_p;
  g.ctx0 = IDX ? cu_ctx[g.b] : 0;
  asm volatile("" ::"s"(g.q0), "s"(q_end), "s"(g.k0), "s"(k_end), "s"(g.l0), "s"(l_end), "s"(g.ctx0));  // one round of loads
  g.q_b = q_end - g.q0;
  g.k_b = nug_len != nullptr ? k_end : k_end - g.k0;
  g.m_b = loc_len != nullptr ? l_end : l_end - g.l0;
  return g;
}

// In the place of a sum: the share has no tile that the row's wavefront looked at.  (Of a sum that is 0 or NaN the channels count
// all the same: a NaN or an infinity in K or V makes them NaN, and the row's result with them, as without sharing.)
constexpr float kNoKeys = -1.f;

// What a workgroup knows of its share of a query block's keys, and where its partial results go (split form only).
struct SplitArgs {
  int split, nsplit;
  float* o;        // [split][row slot][DH], not normalised; nothing where ml holds kNoKeys
  float2* ml;      // [split][row slot]: exponent offset (base 2) and sum, or kNoKeys
  int64_t slots;   // row slots: (row of the call, head)
  int64_t first_row;  // the call's first query row
};

// One block (kBM rows) of one (sequence, group of G heads); called by the whole workgroup.
// SPLIT (4 wavefronts): the workgroup takes an equal share of the key tiles and leaves its sums to
// combine_splits_kernel.
// IDX: Kn / Vn are the context's K / V and nugget j of sequence b is its token cu_ctx[b] + nug_idx[cu_nuggets[b] + j].
// GROUPED: G_ heads go through the tiles together (else one).
template <int NW, int KG, bool IDX, int DH, bool SPLIT, bool GROUPED>
__device__ __forceinline__ void attend_query_block(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ Kn, const uint16_t* __restrict__ Vn,
    const uint16_t* __restrict__ Kl, const uint16_t* __restrict__ Vl, const int32_t* __restrict__ nug_idx, int idx_cap,
    int H, int H_kv, int G_, FastDiv div_G, FastDiv div_kv, const SeqGeom& geom, int qblk,
    int64_t nug_tok_stride, int64_t nug_head_stride, float scale_log2e, uint16_t* __restrict__ O,
    float* __restrict__ lse, const SplitArgs& sp) {
  static_assert(NW == 4 || !SPLIT, "the 8-wavefront kernel does not share the keys out");
  using Cfg = BlockCfg<NW, DH, KG>;
  using HD = HeadDims<DH>;
  constexpr int kDH = DH, kRowBytes = HD::kRowBytes, kTileBytes = HD::kTileBytes;
  constexpr int kP = HD::kPieces;           // 16-byte pieces of a row
  constexpr int kRowShift = HD::kRowShift;  // swizzles use row >> kRowShift
  constexpr int kNCB = HD::kChannelBlocks;  // 32-channel blocks of the output
  constexpr int kSteps = HD::kSteps;        // MFMAs of S^T per tile, and of O^T += V^T P^T
  constexpr int kBM = Cfg::kBM;
  constexpr bool kTwoGroups = Cfg::kTwoGroups;
  constexpr int NKB = 2 / KG;               // 32-key blocks of a tile per wavefront
  constexpr int kStages = Cfg::kStages;
  extern __shared__ __attribute__((aligned(1024))) char lds[];  // stage s: K at 2s, V at 2s+1 (tiles of 16 KiB)
  const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void*)lds));

  const int G = GROUPED ? G_ : 1;
  const int h0 = geom.grp * G, kvh = static_cast<int>(fast_div(static_cast<uint32_t>(geom.grp), div_kv));
  const int q0 = geom.q0, q_b = geom.q_b, k0 = geom.k0, k_b = geom.k_b, l0 = geom.l0, m_b = geom.m_b;
  const int rows_b = q_b * G;
  const int i0 = qblk * kBM;
  if (i0 >= rows_b) return;  // uniform over the workgroup
  // a row's query row inside the sequence, and its place among the call's (query row, head) pairs
  auto query_of = [&](int f) -> int { return GROUPED ? static_cast<int>(fast_div(static_cast<uint32_t>(f), div_G)) : f; };
  auto place_of = [&](int f, int i) -> int64_t { return static_cast<int64_t>(q0 + i) * H + h0 + (f - i * G); };

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave;
  const int j = lane & 31, g = lane >> 5;
  const int row_wave = KG == 2 ? wave % (NW / 2) : wave, half = KG == 2 ? wave / (NW / 2) : 0;
  const int w_i0 = i0 + row_wave * 32;  // first row of this wavefront
  // A wavefront past the sequence's last row only brings tiles: its matrix instructions would take the pipe and the LDS from the
  // others (8 x 530 rows, 200 nuggets, 32 heads 90.3 -> 80.0 us; 129 rows, 410 nuggets 28.7 -> 26.5; 16 x 32 rows 27.9 -> 25.9).
  const bool has_rows = w_i0 < rows_b;
  const int shift = m_b - q_b + 1;  // query row i sees local rows [0, i + shift)
  const int my_f = w_i0 + j;        // this lane's row and query row
  const int my_i = query_of(my_f);
  const bool row_ok = my_f < rows_b;
  const int my_vis = row_ok ? max(0, min(m_b, my_i + shift)) : 0;
  // local rows visible to the first / last row of this wavefront and to the whole workgroup
  const int w_lo = max(0, min(m_b, query_of(w_i0) + shift));
  const int w_hi = max(0, min(m_b, query_of(min(w_i0 + 31, rows_b - 1)) + shift));
  const int wg_vis = max(0, min(m_b, query_of(min(i0 + kBM, rows_b) - 1) + shift));

  const int n_nug_tiles = (k_b + kBN - 1) / kBN;
  const int n_loc_tiles = (wg_vis + kBN - 1) / kBN;
  const int n_tiles = n_nug_tiles + n_loc_tiles;
  // the tiles of this workgroup: an even number per split, because a tile's stage follows from its index
  const int per_split = SPLIT ? 2 * ((n_tiles + 2 * sp.nsplit - 1) / (2 * sp.nsplit)) : n_tiles;
  const int t_begin = SPLIT ? min(n_tiles, sp.split * per_split) : 0;
  const int t_end = SPLIT ? min(n_tiles, t_begin + per_split) : n_tiles;

  const int64_t nug_row0 = IDX ? geom.ctx0 : k0;  // IDX: the index list holds tokens of the sequence that starts here
  const uint16_t* nugK = Kn + nug_row0 * nug_tok_stride + static_cast<int64_t>(kvh) * nug_head_stride;
  const uint16_t* nugV = Vn + nug_row0 * nug_tok_stride + static_cast<int64_t>(kvh) * nug_head_stride;
  const int32_t* idx_l = reinterpret_cast<const int32_t*>(lds + Cfg::kLdsBytes);
  if (IDX) {
    // (a previous query block of this workgroup is past its last tile request: the caller's barrier)
    int32_t* dst = reinterpret_cast<int32_t*>(lds + Cfg::kLdsBytes);
    for (int t = threadIdx.x; t < min(k_b, idx_cap); t += Cfg::kThreads) dst[t] = nug_idx[k0 + t];
    __syncthreads();
  }
  const int64_t loc_stride = static_cast<int64_t>(H_kv) * kDH;
  const uint16_t* locK = Kl + (static_cast<int64_t>(l0) * H_kv + kvh) * kDH;
  const uint16_t* locV = Vl + (static_cast<int64_t>(l0) * H_kv + kvh) * kDH;

  // Who brings what of a tile: in the 4-wavefront kernel every wavefront a part of K and of V; in the 8-wavefront kernel
  // the wavefronts of group 1 K and those of group 0 V.  Every request enqueues the same number of loads per lane (a tile
  // past the end fetches nothing), so the vmcnt arithmetic of the loops is uniform.
  using Loader = TileLoader<kTwoGroups ? 4 : NW, DH>;
  Loader loader;
  loader.init(kTwoGroups ? wave & 3 : wave, lane);
  constexpr int kPer = Loader::kPerWave;
  constexpr int kLoadsPerTile = kTwoGroups ? kPer : 2 * kPer;
  uint32_t off[kPer];       // of the tensor that this wavefront's group brings (4 wavefronts: of K)
  uint32_t off_stride = 0;  // the token stride that they were made for
  auto request = [&](int tile, auto v_tag, auto both_tag) {
    constexpr bool IS_V = decltype(v_tag)::value, BOTH = decltype(both_tag)::value;
    const bool nug = tile < n_nug_tiles;
    const int base = nug ? tile * kBN : (tile - n_nug_tiles) * kBN;
    const int cnt = min(kBN, (nug ? k_b : wg_vis) - base);  // no more than 0 past the last tile
    const int64_t stride = nug ? nug_tok_stride : loc_stride;
    const uint32_t stride_bytes = static_cast<uint32_t>(stride) * 2u;
    const uint32_t dst = lds_base + (2 * (tile % kStages) + (IS_V ? 1 : 0)) * kTileBytes;
    const uint16_t* ptr = nug ? (IS_V ? nugV : nugK) : (IS_V ? locV : locK);
    const uint16_t* ptr_v = nug ? nugV : locV;
    auto issue = [&](int64_t first, uint32_t range) {  // the region's row at element `first` is offset 0
      loader.issue(ptr + first, range, off, dst);
      if (BOTH) {
        uint32_t off_v[kPer];
        loader.k_to_v(off, off_v);
        loader.issue(ptr_v + first, range, off_v, dst + kTileBytes);
      }
    };
    if (IDX && nug) {
      loader.template offsets_idx<IS_V>(stride_bytes, cnt, idx_l + base, off);
      off_stride = 0;
      issue(0, 0x7fffffffu);  // (offsets from the sequence's first token, below 2^31: checked on the host)
    } else {
      if (off_stride != stride_bytes) {
        loader.template offsets<IS_V>(stride_bytes, off);
        off_stride = stride_bytes;
      }
      issue(base * stride, cnt > 0 ? static_cast<uint32_t>(cnt - 1) * stride_bytes + kRowBytes : 0u);
    }
  };
  using K = std::false_type;
  using V = std::true_type;
  using Alone = std::false_type;
  using WithV = std::true_type;
  auto issue_tile = [&](int tile) {
    if (!kTwoGroups) {
      if (!SPLIT || tile < t_end) request(tile, K{}, WithV{});
    } else if (wave < 4) {
      request(tile, V{}, Alone{});
    } else {
      request(tile, K{}, Alone{});
    }
  };
  // per-tile bookkeeping shared by the phases
  struct TileInfo {
    bool visible, need_mask;
    int limit;
  };
  auto tile_info = [&](int tile) -> TileInfo {
    const bool is_nug = tile < n_nug_tiles;
    const int base = is_nug ? tile * kBN : (tile - n_nug_tiles) * kBN;
    const int cnt = min(kBN, (is_nug ? k_b : wg_vis) - base);
    TileInfo ti;
    ti.visible = has_rows && (is_nug || base < w_hi);  // some key of this tile is visible to this wavefront
    ti.need_mask = cnt < kBN || (!is_nug && base + kBN > w_lo);
    ti.limit = is_nug ? cnt : min(cnt, my_vis - base);  // keys [0, limit) are visible to this lane's row
    return ti;
  };

  // Prologue.  The first tile is requested before anything else; the workgroup's query rows follow,
  // through LDS like a K tile (whole rows per request; a lane fetching its own row from global
  // memory would touch 32 rows per instruction), into the stages that tiles 1.. (NW = 4) or 2..
  // (NW = 8) use later.  Q^T fragments: lane (j, g) holds Q[my_i][16*ds + 8*g .. +8) for ds = 0..7.
  // Rows past the end of the sequence read as zeros, and their lanes take the last row's fragments instead: zeros would make NaN of
  // an infinite key, which spreads through the row sums below and has the block done twice.  Nothing of them is stored.
  constexpr int kQSlot0 = kTwoGroups ? 4 : 2;  // first 16 KiB slot of the query rows
  bf16x8 qf[kDH / 16];
  if (t_begin < t_end) {
    issue_tile(t_begin);
    TileLoader<NW, DH> q_loader;
    q_loader.init(wave, lane);
    uint32_t q_off[TileLoader<NW, DH>::kPerWave];
    if (!GROUPED) q_loader.template offsets<false>(static_cast<uint32_t>(H) * kRowBytes, q_off);
#pragma unroll
    for (int c = 0; c < kBM / kBN; ++c) {
      const int f0 = i0 + kBN * c, first = query_of(f0);
      const int rows = min(kBN, rows_b - f0);
      uint32_t range = 0;
      if (!GROUPED) {
        if (rows > 0) range = static_cast<uint32_t>(rows - 1) * static_cast<uint32_t>(H) * kRowBytes + kRowBytes;
      } else {  // (offsets from the first row's token and the group's first head: they grow with the row)
        auto offset_of = [&](int f) -> uint32_t {
          const int i = query_of(f);
          return (static_cast<uint32_t>(i - first) * static_cast<uint32_t>(H) + static_cast<uint32_t>(f - i * G)) * kRowBytes;
        };
        if (rows > 0) range = offset_of(f0 + rows - 1) + kRowBytes;
#pragma unroll
        for (int u = 0; u < TileLoader<NW, DH>::kPerWave; ++u) {
          const int row = q_loader.row0 + TileLoader<NW, DH>::kRowsPerInstr * u;
          q_off[u] = offset_of(f0 + row) + q_loader.template piece_bytes<false>(row);
        }
      }
      q_loader.issue(Q + (static_cast<int64_t>(q0 + first) * H + h0) * kDH, range, q_off, lds_base + (kQSlot0 + c) * kTileBytes);
    }
    if (kTwoGroups) {
      issue_tile(1);
      __builtin_amdgcn_s_waitcnt(0x0f70 | kLoadsPerTile);  // tile 0 and Q landed, tile 1 in flight
    } else {
      __builtin_amdgcn_s_waitcnt(0x0f70);
    }
    __syncthreads();
    const int j_q = max(0, min(j, rows_b - 1 - w_i0));
    const char* qbuf = lds + kQSlot0 * kTileBytes + (row_wave * 32 + j_q) * kRowBytes;
#pragma unroll
    for (int ds = 0; ds < kDH / 16; ++ds)
      qf[ds] = *reinterpret_cast<const bf16x8*>(qbuf + (((2 * ds + g) ^ ((j_q >> kRowShift) & (kP - 1))) << 4));
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the fragments are in registers
    if (kTwoGroups) {
      __syncthreads();  // everyone has its fragments: the stages are free again
      issue_tile(2);
      issue_tile(3);
    }
  } else {
#pragma unroll
    for (int ds = 0; ds < kDH / 16; ++ds) qf[ds] = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
  }

  floatx16 acc_o[kDH / 32];
#pragma unroll
  for (int cb = 0; cb < kDH / 32; ++cb)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc_o[cb][v] = 0.f;
  float m_run = kNegInf, l_run = 0.f;

  // per-lane constants of the LDS read patterns
  const int k_row_off = j * kRowBytes;  // K: row 32kb + j, piece (2ds + g) ^ swizzle(row); swizzle(32kb + j) == swizzle(j)
  const int k_sw = (j >> kRowShift) & (kP - 1);
  // V^T via transposing read: lane supplies row 16t + 8e + 4g + (lane%16)/4, 8 bytes at channel 32cb + 16*half + 4*(lane%4)
  const int v_r = 4 * g + ((lane & 15) >> 2);
  const int v_in = 32 * ((lane >> 4) & 1) + 8 * (lane & 3);

  // Fragments are requested kAhead MFMAs before their use; the scheduling barriers keep the
  // compiler from hoisting every LDS read of a tile to the front (which would not fit in registers).
  constexpr int kAhead = 6;
  // S^T = K Q^T of one tile: K fragment s = 2*ds + kb is row 32kb + j, 16 bytes at the swizzled piece 2ds + g
  auto read_k = [&](int tile, int s) -> bf16x8 {
    const char* kbuf = lds + (2 * (tile % kStages)) * kTileBytes + k_row_off;
    return *reinterpret_cast<const bf16x8*>(kbuf + (s & 1) * 32 * kRowBytes + ((((s >> 1) * 2 + g) ^ k_sw) << 4));
  };
  auto compute_s = [&](int tile, floatx16 (&acc_s)[NKB]) {  // (KG = 2: the keys of block `half`)
    constexpr int kAll = kSteps / KG;
    const auto frag = [&](int s) { return read_k(tile, KG == 2 ? 2 * s + half : s); };
    bf16x8 kf[kAhead];
#pragma unroll
    for (int s = 0; s < kAhead && s < kAll; ++s) kf[s] = frag(s);
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc_s[kb][v] = 0.f;
#pragma unroll
    for (int s = 0; s < kAll; ++s) {
      const bf16x8 cur = kf[s % kAhead];
      if (s + kAhead < kAll) kf[s % kAhead] = frag(s + kAhead);
      acc_s[s % NKB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, qf[s / NKB], acc_s[s % NKB], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // O^T += V^T P^T of one tile: V^T fragment s = 4*t + cb; slot 8g+4e+r of k-step t <-> key 16t + 8e + 4g + r.
  // The two-group kernel takes the row sums of P from the matrix pipe as well, of the bf16-rounded P, exactly what O^T is
  // accumulated from: one 16x16x32 product per P^T fragment (half the cycles of a 33rd block of V^T).  Read as a 32 x 16
  // operand, lane l of the fragment holds column l % 16 and keys of group l / 16: groups 0 and 2 are the keys of queries
  // 0 .. 15, groups 1 and 3 those of queries 16 .. 31, so row 0 of the left operand has ones in groups 0 and 2, row 1 in
  // groups 1 and 3, and accumulators 0 and 1 of lane n < 16 collect the sums of queries n and n + 16 over all keys.
  floatx4 acc_l = {0.f, 0.f, 0.f, 0.f};
  const bool sel_one = (lane & 15) == ((lane >> 4) & 1);
  const bf16x8 sel_frag = __builtin_bit_cast(
      bf16x8, sel_one ? make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u) : make_uint4(0, 0, 0, 0));
  auto read_vt = [&](int tile, int s) -> bf16x8 {
    const char* vbuf = lds + (2 * (tile % kStages) + 1) * kTileBytes + v_in;
    const int t = s / kNCB, cb = s % kNCB;
    shortx4 a[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int r = 16 * t + 8 * e + v_r;
      const char* p = vbuf + r * kRowBytes + ((cb ^ ((r >> kRowShift) & (kNCB - 1))) << 6);
      a[e] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p));
    }
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a[0], a[1], 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto compute_pv = [&](int tile, const bf16x8 (&pf)[2 * NKB]) {  // (KG = 2: k-steps 2 half and 2 half + 1)
    constexpr int kAll = kSteps / KG;
    const auto frag = [&](int s) { return read_vt(tile, s + (KG == 2 ? half * kAll : 0)); };
    bf16x8 vf[kAhead];
#pragma unroll
    for (int s = 0; s < kAhead && s < kAll; ++s) vf[s] = frag(s);
#pragma unroll
    for (int s = 0; s < kAll; ++s) {
      const bf16x8 cur = vf[s % kAhead];
      if (s + kAhead < kAll) vf[s % kAhead] = frag(s + kAhead);
      acc_o[s % kNCB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, pf[s / kNCB], acc_o[s % kNCB], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  bool bail = false;
  auto softmax = [&](const TileInfo& ti, floatx16 (&acc_s)[NKB], bf16x8 (&pf)[2 * NKB]) {
    if (ti.need_mask) {
      softmax_tile<true, kNCB, NKB>(acc_s, ti.limit - 32 * half, g, scale_log2e, m_run, l_run, acc_o, pf);
    } else {
      softmax_tile<false, kNCB, NKB>(acc_s, kBN, g, scale_log2e, m_run, l_run, acc_o, pf);
    }
  };

  bool saw_keys = false;  // (split form)
  if constexpr (!kTwoGroups) {
    // ---- plain loop: one barrier per tile, next tile in flight ----
    // (the first barrier also tells that every wavefront has taken its Q fragments out of stage 1)
    for (int tile = t_begin; tile < t_end; ++tile) {
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wavefront's part of the tile has landed
      __syncthreads();                      // everyone's part has landed; the other stage is free
      issue_tile(tile + 1);
      const TileInfo ti = tile_info(tile);
      if (!ti.visible) continue;
      saw_keys = true;
      floatx16 acc_s[NKB];
      bf16x8 pf[2 * NKB];
      compute_s(tile, acc_s);
      softmax(ti, acc_s, pf);
      compute_pv(tile, pf);
    }
  } else {
    // ---- two groups of four wavefronts, half a tile apart ----
    // Phase p ends with a workgroup barrier.  Group 0 does in even phases 2t "PV(t-1) then S(t)"
    // (32 MFMAs) and in odd phases 2t+1 the softmax of tile t; group 1 does the softmax of tile
    // t-1 in phase 2t and the MFMAs in phase 2t+1, so in every phase one group feeds the matrix
    // pipe while the other runs VALU work.  Tile t is read during phases 2t .. 2t+3 and sits in
    // stage t % 4; tile t+4 is requested during phases 2t+4 (K) and 2t+5 (V) and has to be visible
    // at the barrier that ends phase 2t+7.
    const int grp = wave >> 2;
    floatx16 acc_s[2];
    bf16x8 pf[4];
    // One iteration = phases 2t and 2t+1.  The two groups run separate copies of the loop (same
    // number of barriers) so that each copy is straight-line code for the compiler.
    // The MFMA phase is one software pipeline over 32 fragments (16 of V^T, then 16 of K), each
    // requested kAhead MFMAs before its use into a ring of registers: slot i of the phase lives
    // in ring[i % kAhead].  The first kAhead fragments of V^T are requested at the end of the
    // softmax phase before, so no MFMA phase starts by waiting for LDS.  A tile that is invisible
    // to a wavefront (above the causal diagonal) is followed by invisible tiles only.
    bf16x8 ring[kAhead];
    auto pv_steps = [&](int t, auto k_prefetch_tag) {  // PV(t-1); requests the first K fragments of tile t
      constexpr bool K_PREFETCH = decltype(k_prefetch_tag)::value;
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        const bf16x8 cur = ring[s % kAhead];
        if (s + kAhead < kSteps) {
          ring[s % kAhead] = read_vt(t - 1, s + kAhead);
        } else if (K_PREFETCH) {
          ring[s % kAhead] = read_k(t, s + kAhead - kSteps);
        }
        acc_o[s % kNCB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, pf[s / kNCB], acc_o[s % kNCB], 0, 0, 0);
        if ((s % kNCB) == kNCB - 1)
          acc_l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sel_frag, pf[s / kNCB], acc_l, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto s_steps = [&](int t) {  // S(t); its first kAhead fragments are in the ring already
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_s[kb][v] = 0.f;
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        const bf16x8 cur = ring[(kSteps + s) % kAhead];
        if (s + kAhead < kSteps) ring[(kSteps + s) % kAhead] = read_k(t, s + kAhead);
        acc_s[s & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, qf[s >> 1], acc_s[s & 1], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto valu_work = [&](int t) {  // softmax of tile t, then the first V^T fragments for PV(t)
      const TileInfo ti = tile_info(t);
      if (ti.need_mask) mask_tile(acc_s, ti.limit, g);
      if (t == 0) m_run = tile_max(acc_s) * scale_log2e;  // (-inf: no key visible)
      softmax_fixed(acc_s, scale_log2e, m_run, pf);
#pragma unroll
      for (int s = 0; s < kAhead; ++s) ring[s] = read_vt(t, s);
    };
    // In the loop a wavefront requests tiles in its softmax phase: a request can take hundreds of cycles to issue when the
    // memory pipeline is backed up.  The wavefronts of group 1 bring K of tile t+2 (during phase 2t), those of group 0 its V
    // (during phase 2t+1).
    auto end_odd_phase = [&](int t) {  // ends phase 2t+1: tile t+1 must have landed
      // younger requests of this wavefront in flight: two tiles' worth while the prologue's are pending, else one
      if (t == 0) {
        __builtin_amdgcn_s_waitcnt(0x0f70 | (2 * kLoadsPerTile));
      } else {
        __builtin_amdgcn_s_waitcnt(0x0f70 | (1 * kLoadsPerTile));
      }
      __syncthreads();
    };
    if (n_tiles > 0 && scale_log2e > 0.f) {
      // Tiles [0, n_vis) are visible to this wavefront.  Iteration t is one of four kinds, so that
      // each loop body is straight-line code: 0 = S(0) only, 1 = PV(t-1) and S(t) (the steady
      // state), 2 = PV(n_vis-1) only, 3 = nothing but the barriers the other wavefronts count on.
      const int n_vis = has_rows ? n_nug_tiles + min(n_loc_tiles, (w_hi + kBN - 1) / kBN) : 0;
      auto iteration = [&](int t, auto grp_tag, auto kind_tag) {
        constexpr int GRP = decltype(grp_tag)::value, KIND = decltype(kind_tag)::value;
        if (GRP == 1) {
          if (t >= 2) request(t + 2, K{}, Alone{});
          if (KIND == 1 || KIND == 2) valu_work(t - 1);
          __syncthreads();
        }
        __builtin_amdgcn_s_setprio(1);
        if (KIND == 0) {
#pragma unroll
          for (int s = 0; s < kAhead; ++s) ring[(kSteps + s) % kAhead] = read_k(t, s);
          s_steps(t);
        } else if (KIND == 1) {
          pv_steps(t, std::true_type{});
          s_steps(t);
        } else if (KIND == 2) {
          pv_steps(t, std::false_type{});
        }
        __builtin_amdgcn_s_setprio(0);
        if (GRP == 0) {
          __syncthreads();
          if (t >= 2) request(t + 2, V{}, Alone{});
          if (KIND == 0 || KIND == 1) valu_work(t);
        }
        end_odd_phase(t);
      };
      auto run = [&](auto grp_tag) {
        using K0 = std::integral_constant<int, 0>;
        using K1 = std::integral_constant<int, 1>;
        using K2 = std::integral_constant<int, 2>;
        using K3 = std::integral_constant<int, 3>;
        int t = 0;
        if (n_vis > 0) {
          iteration(0, grp_tag, K0{});
          for (t = 1; t < n_vis; ++t) iteration(t, grp_tag, K1{});
          iteration(t, grp_tag, K2{});
          ++t;
        }
        for (; t <= n_tiles; ++t) iteration(t, grp_tag, K3{});
      };
      if (grp == 0) {
        run(std::integral_constant<int, 0>{});
      } else {
        run(std::integral_constant<int, 1>{});
      }
      const float sum_lo = __shfl(acc_l[0], lane & 15, kWave), sum_hi = __shfl(acc_l[1], lane & 15, kWave);
      const float l_row = (j & 16) ? sum_hi : sum_lo;
      l_run = (g == 0) ? l_row : 0.f;
      bail = !(l_row <= kMostSum) ||  // or NaN: some logit is too far above the row's fixed offset
             (m_run == kNegInf && row_ok && (k_b > 0 || my_vis > 0));  // no offset, though the row sees keys
    } else {
      bail = n_tiles > 0;
    }
    // Rare: some logit is too far above its row's fixed offset, or a row has none (or the scale is not positive).  Redo the
    // workgroup's rows with the exact running-maximum softmax, one tile at a time.
    __builtin_amdgcn_s_waitcnt(0x0f70);
    if (__syncthreads_or(bail)) {
#pragma unroll
      for (int cb = 0; cb < kDH / 32; ++cb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_o[cb][v] = 0.f;
      m_run = kNegInf;
      l_run = 0.f;
      for (int tile = 0; tile < n_tiles; ++tile) {
        issue_tile(tile);
        __builtin_amdgcn_s_waitcnt(0x0f70);
        __syncthreads();
        const TileInfo ti = tile_info(tile);
        if (ti.visible) {
          compute_s(tile, acc_s);
          softmax(ti, acc_s, pf);
          compute_pv(tile, pf);
        }
        __syncthreads();
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);  // drain the look-ahead loads before the wavefront ends

  // ---- epilogue: lane (j, g) holds channels 32cb + 8(v/4) + 4g + v%4 of query row my_i ----
  // The 32 x 128 block of a wavefront goes through LDS (free by now) so that O is written with
  // full 256-byte rows, 16 bytes per lane; 16-byte pieces are XOR-swizzled with the row to keep
  // both the 8-byte writes and the 16-byte reads free of bank conflicts.
  if (!kTwoGroups) __syncthreads();  // every wavefront is done with the K/V stages
  if constexpr (KG == 2) {
    // The second halves' offsets, sums and channels go to the first halves through the stages (16 bytes per lane and access).
    // (Behind the stages their offsets and sums would take the index list's workgroups the second place on a compute unit: 12 x 64
    // rows, 300 nuggets, 32 heads through the list 30.4 us there, 21.9 here; 9 x 64 rows, 100 nuggets 20.2 / 13.9.)
    float2* ml = reinterpret_cast<float2*>(lds + Cfg::kMergeO) + row_wave * kWave + lane;
    float4* o = reinterpret_cast<float4*>(lds + row_wave * (32 * kDH * 4)) + lane;
    if (half == 1) {
      *ml = make_float2(m_run, l_run);
#pragma unroll
      for (int cb = 0; cb < kNCB; ++cb)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq)
          o[(4 * cb + vq) * kWave] = make_float4(acc_o[cb][4 * vq], acc_o[cb][4 * vq + 1], acc_o[cb][4 * vq + 2], acc_o[cb][4 * vq + 3]);
    }
    __syncthreads();
    if (half == 0) {
      const float2 other = *ml;
      const float m_new = fmaxf(m_run, other.x), m_use = (m_new == kNegInf) ? 0.f : m_new;
      const float a = exp2_hw(m_run - m_use), b = exp2_hw(other.x - m_use);
      l_run = l_run * a + other.y * b;
      m_run = m_new;
#pragma unroll
      for (int cb = 0; cb < kNCB; ++cb)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          const float4 p = o[(4 * cb + vq) * kWave];
          acc_o[cb][4 * vq] = acc_o[cb][4 * vq] * a + p.x * b;
          acc_o[cb][4 * vq + 1] = acc_o[cb][4 * vq + 1] * a + p.y * b;
          acc_o[cb][4 * vq + 2] = acc_o[cb][4 * vq + 2] * a + p.z * b;
          acc_o[cb][4 * vq + 3] = acc_o[cb][4 * vq + 3] * a + p.w * b;
        }
    }
    __syncthreads();  // the stages are free again
    if (half == 1) return;
  }
  const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
  if constexpr (SPLIT) {
    // (slots follow from max_q: rows of a sequence that is longer have none and are not written, rather than past the workspace)
    const int64_t row_slot = place_of(my_f, my_i) - sp.first_row * H;
    if (row_ok && row_slot < sp.slots) {
      // A workspace may serve a call with flags next, and no flag may hold the ready value: neither does a record.
      auto word = [](float x) { return __float_as_uint(x) == kPartialReady ? __uint_as_float(kPartialReady + 1) : x; };
      const int64_t slot = static_cast<int64_t>(sp.split) * sp.slots + row_slot;
      if (g == 0) sp.ml[slot] = make_float2(word(m_run), saw_keys ? word(l_tot) : kNoKeys);
      if (saw_keys) {
        float* o = sp.o + slot * DH + 4 * g;
#pragma unroll
        for (int cb = 0; cb < kNCB; ++cb)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq)
            *reinterpret_cast<float4*>(o + 32 * cb + 8 * vq) =
                make_float4(word(acc_o[cb][4 * vq]), word(acc_o[cb][4 * vq + 1]), word(acc_o[cb][4 * vq + 2]), word(acc_o[cb][4 * vq + 3]));
      }
    }
    return;
  }
  {
    const float inv = (l_tot > 0.f) ? 1.f / l_tot : 0.f;
    char* obuf = lds + row_wave * (32 * kRowBytes);
#pragma unroll
    for (int cb = 0; cb < kDH / 32; ++cb)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        const int piece = 4 * cb + vq;  // 16-byte piece of the row: channels 8*piece .. 8*piece+7; g picks the half
        uint2 out;
        out.x = pack2_bf16(acc_o[cb][4 * vq + 0] * inv, acc_o[cb][4 * vq + 1] * inv);
        out.y = pack2_bf16(acc_o[cb][4 * vq + 2] * inv, acc_o[cb][4 * vq + 3] * inv);
        *reinterpret_cast<uint2*>(obuf + j * kRowBytes + ((piece ^ ((j >> kRowShift) & (kP - 1))) << 4) + 8 * g) = out;
      }
    __builtin_amdgcn_wave_barrier();
    const int n_rows = min(32, rows_b - w_i0);  // valid rows of this wavefront (may be <= 0)
#pragma unroll
    for (int it = 0; it < kP / 2; ++it) {  // 64 / kP rows per iteration, 16 bytes per lane
      const int row = (64 / kP) * it + (lane >> HD::kPiecesLog2), piece = lane & (kP - 1);
      const uint4 val = *reinterpret_cast<const uint4*>(obuf + row * kRowBytes + ((piece ^ ((row >> kRowShift) & (kP - 1))) << 4));
      const int f = w_i0 + row;
      if (row < n_rows) *reinterpret_cast<uint4*>(O + place_of(f, query_of(f)) * kDH + piece * 8) = val;
    }
  }
  if (row_ok && lse != nullptr && g == 0) {
    lse[place_of(my_f, my_i)] =
        (l_tot > 0.f) ? (m_run + __log2f(l_tot)) * 0.6931471805599453f : kNegInf;
  }
}

// Workgroups are handed to the 8 XCDs round-robin, each XCD has an L2 of its own: the blocks
// of one (sequence, group of heads) go to one XCD back to back (heaviest first), so that they start together
// and share the K/V tiles in that L2.  With pair != 0 a workgroup takes two query blocks, one
// after the other: a block i from the end and a block i from the start, so that under the causal
// mask all workgroups carry the same load (new workgroups are handed out in order, and a compute
// unit that finishes early is not refilled before the ones ahead of it in that order).
template <int NW, int KG, bool IDX, int DH, bool SPLIT, bool GROUPED>
__global__ __launch_bounds__((BlockCfg<NW, DH, KG>::kThreads), (BlockCfg<NW, DH, KG>::kMinBlocks)) void block_attention_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ Kn, const uint16_t* __restrict__ Vn,
    const uint16_t* __restrict__ Kl, const uint16_t* __restrict__ Vl, const int32_t* __restrict__ cu_q,
    const int32_t* __restrict__ cu_nuggets, const int32_t* __restrict__ nug_len,
    const int32_t* __restrict__ cu_local, const int32_t* __restrict__ loc_len, const int32_t* __restrict__ nug_idx,
    const int32_t* __restrict__ cu_ctx, int idx_cap,
    int B, int H, int H_kv, int G, int HG, int n_qblocks, int pair, int sorted, int heavy_last, int heads_xcd, FastDiv div_heads_xcd, FastDiv div_slots,
    FastDiv div_pairs, FastDiv div_HG, FastDiv div_G, FastDiv div_kv,
    int64_t nug_tok_stride, int64_t nug_head_stride, float scale_log2e, uint16_t* __restrict__ O,
    float* __restrict__ lse, float* __restrict__ part_o, float2* __restrict__ part_ml, int64_t slots) {
  // all arguments in one round of scalar loads (the compiler would fetch them a few at a time, before each first use)
  asm volatile("" ::"s"(Q), "s"(Kn), "s"(Vn), "s"(Kl), "s"(Vl), "s"(cu_q), "s"(cu_nuggets), "s"(nug_len), "s"(cu_local),
               "s"(loc_len), "s"(nug_idx), "s"(cu_ctx), "s"(B), "s"(H), "s"(H_kv), "s"(G), "s"(HG), "s"(n_qblocks), "s"(pair), "s"(sorted),
               "s"(heavy_last), "s"(heads_xcd));
  asm volatile("" ::"s"(div_heads_xcd.mul), "s"(div_heads_xcd.shift), "s"(div_slots.mul), "s"(div_slots.shift), "s"(div_pairs.mul),
               "s"(div_pairs.shift), "s"(div_HG.mul), "s"(div_HG.shift), "s"(div_G.mul), "s"(div_G.shift), "s"(div_kv.mul),
               "s"(div_kv.shift), "s"(nug_tok_stride), "s"(nug_head_stride), "s"(scale_log2e), "s"(O), "s"(lse));
  const int n_slots = pair ? (n_qblocks + 1) >> 1 : n_qblocks, n_pairs = B * HG;  // (div_slots and div_pairs divide by these)
  // The i-th (sequence, group) of an XCD: heads_xcd consecutive groups of every sequence (ragged sequences weigh on all
  // XCDs alike), starting at another one in each sequence, or every eighth (heads_xcd = 0).
  auto pair_of = [&](int i, int x) -> int {
    if (heads_xcd == 0) return i * 8 + x;
    const int b = static_cast<int>(fast_div(static_cast<uint32_t>(i), div_heads_xcd));
    return b * HG + ((x + b) & 7) * heads_xcd + (i - b * heads_xcd);
  };
  // sorted: the heaviest block of every (sequence, group), then the next ones of all; else an XCD's (sequence, group)s one after
  // the other
  const int turn = sorted ? static_cast<int>(fast_div(blockIdx.x, div_pairs)) : 0;
  const int place = static_cast<int>(blockIdx.x) - turn * n_pairs;
  const int xcd = place & 7, slot = place >> 3;
  const int j = sorted ? slot : static_cast<int>(fast_div(static_cast<uint32_t>(slot), div_slots));
  const int bh = pair_of(j, xcd);
  const int heavy = n_qblocks - 1 - (sorted ? turn : slot - j * n_slots), light = n_qblocks - 1 - heavy;
  if (bh >= n_pairs) return;
  // Two neighbouring workgroups of an XCD (j even and odd) share two (sequence, head) pairs
  // crosswise: one takes the heavy block of the first pair and then the light block of the second,
  // the other the light block of the first and then the heavy block of the second.  Both carry the
  // same load, the two blocks that read the same K/V run at the same time and share it in L2, and
  // the bursts of first loads come from half of the compute units at a time.
  const int bh_other = pair_of(j ^ 1, xcd);
  const bool cross = pair && light != heavy && bh_other < n_pairs;
  int bh1 = bh, q1 = heavy, bh2 = bh, q2 = (pair && light != heavy) ? light : -1;
  if (cross) {
    if (j & 1) {
      bh1 = bh_other;
      q1 = light;
      q2 = heavy;
    } else {
      bh2 = bh_other;
    }
  }
  // heavy_last: the batch's entries grow in cost with their index (segments of a text see more and more nuggets);
  // workgroups are handed out in index order, so the entries are walked from the back to keep the tail light
  if (heavy_last) {
    bh1 = n_pairs - 1 - bh1;
    bh2 = n_pairs - 1 - bh2;
  }
  // both blocks' sequence data are requested here, before the first block's work
  const SeqGeom g1 = load_seq_geom<IDX>(bh1, div_HG, HG, cu_q, cu_nuggets, nug_len, cu_local, loc_len, cu_ctx);
  const SeqGeom g2 = load_seq_geom<IDX>(q2 >= 0 ? bh2 : bh1, div_HG, HG, cu_q, cu_nuggets, nug_len, cu_local, loc_len, cu_ctx);
  SplitArgs sp{0, 1, nullptr, nullptr, 0, 0};
  if (SPLIT) sp = SplitArgs{static_cast<int>(blockIdx.y), static_cast<int>(gridDim.y), part_o, part_ml, slots, cu_q[0]};
  attend_query_block<NW, KG, IDX, DH, SPLIT, GROUPED>(Q, Kn, Vn, Kl, Vl, nug_idx, idx_cap, H, H_kv, G, div_G, div_kv, g1, q1, nug_tok_stride, nug_head_stride,
                                         scale_log2e, O, lse, sp);
  if (!SPLIT && q2 >= 0) {
    __syncthreads();  // the first block's use of LDS is over
    attend_query_block<NW, KG, IDX, DH, SPLIT, GROUPED>(Q, Kn, Vn, Kl, Vl, nug_idx, idx_cap, H, H_kv, G, div_G, div_kv, g2, q2, nug_tok_stride, nug_head_stride,
                                           scale_log2e, O, lse, sp);
  }
}

// The splits' partial results of a row, merged in split order: DH / 4 lanes per row, four channels each.
constexpr int kCombineThreads = 256;
template <int DH>
__global__ __launch_bounds__(kCombineThreads) void combine_splits_kernel(
    const float* __restrict__ part_o, const float2* __restrict__ part_ml, int64_t slots, int nsplit, const int32_t* __restrict__ cu_q,
    int B, int H, uint16_t* __restrict__ O, float* __restrict__ lse) {
  constexpr int kLanes = DH / 4;
  const int64_t slot = static_cast<int64_t>(blockIdx.x) * (kCombineThreads / kLanes) + threadIdx.x / kLanes;
  const int c = threadIdx.x % kLanes;
  const int64_t row0 = cu_q[0], rows = cu_q[B] - row0;
  if (slot >= min(slots, rows * H)) return;
  float M = kNegInf;
  for (int s = 0; s < nsplit; ++s) M = fmaxf(M, part_ml[s * slots + slot].x);
  const float M_use = M == kNegInf ? 0.f : M;
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
  float sum = 0.f;
  for (int s = 0; s < nsplit; ++s) {
    const float2 ml = part_ml[s * slots + slot];
    if (ml.y == kNoKeys) continue;
    const float w = exp2_hw(ml.x - M_use);
    const float4 p = *reinterpret_cast<const float4*>(part_o + (s * slots + slot) * DH + 4 * c);
    sum = fmaf(ml.y, w, sum);
    o.x = fmaf(p.x, w, o.x); o.y = fmaf(p.y, w, o.y); o.z = fmaf(p.z, w, o.z); o.w = fmaf(p.w, w, o.w);
  }
  const float inv = sum > 0.f ? 1.f / sum : 0.f;
  const int64_t at = row0 * H + slot;
  *reinterpret_cast<uint2*>(O + at * DH + 4 * c) = make_uint2(pack2_bf16(o.x * inv, o.y * inv), pack2_bf16(o.z * inv, o.w * inv));
  if (lse != nullptr && c == 0) lse[at] = sum > 0.f ? (M + __log2f(sum)) * 0.6931471805599453f : kNegInf;
}

inline size_t split_bytes(int32_t B, int32_t H, int32_t d_h, int32_t max_q, int64_t n) {
  return static_cast<size_t>(B) * max_q * H * n * (static_cast<size_t>(d_h) + 2) * sizeof(float);
}

// How a call's rows become workgroups.
struct BlockPlan {
  int32_t G = 1;        // query heads of a K/V head that go through the tiles together
  int32_t waves = 4;    // wavefronts per workgroup: 4 or 8, for 32 rows each
  int32_t KG = 1;       // or 2 of them for 32 rows
  int32_t nsplit = 1;   // workgroups that share the keys of a block (4 wavefronts)
  bool pair = false;    // two blocks per workgroup, a heavy and a light one
  bool sorted = false;  // all heavy blocks before the next ones
};

// The plan of least expected time, with at most max_splits shares of the keys.  Measured (ns): a 64-key tile 1350 in the
// 4-wavefront kernel, 1.6 times that with two workgroups on a compute unit; in the 8-wavefront kernel 1200, 1600 where more than
// half of the compute units run it, 2100 where hardly any two of them at work share their keys; heads of 64 channels two thirds
// of that; a block's start and end 4000 and 6200.  With two wavefronts per 32 rows, blocks of 64, a tile takes 1110, and 1900 with two
// workgroups on a compute unit (shares of keys 1800, heads of 64 channels 950).
//
// Two wavefronts per 32 rows, each half of a tile's keys (KG = 2): a wavefront alone on its SIMD works through a tile as one chain of
// matrix and vector instructions.  32 heads, one wavefront / two: 64 rows, 200 nuggets 13.7 / 11.7 us, 4 x 64 rows, 80 nuggets 10.2 /
// 9.4, 170 rows, 358 nuggets 20.1 (the 8-wavefront kernel) / 16.8; 12 x 64 rows, 300 nuggets (two workgroups on a compute unit) 21.7 /
// 19.4; on a full chip they only share its units: 24 x 64 rows 39.5 / 41.8.
//
// Heads together (G): where one head's blocks are more than the chip takes at once and leave lanes without a row or end far from
// each other's causal limits.  One head / together: 64 heads over 8, 16 sequences of 34 rows over 460 nuggets 42.9 / 26.1 us, of 16
// rows over 100 21.9 / 10.5; 8 of 336 rows, 143 nuggets 68.4 / 56.3; 32 heads over 8, 16 of 64 rows, 200 nuggets 19.6 / 17.0.  On a
// chip that is not full a head per workgroup is faster (8 heads of 16 rows 9.5 / 10.1 us, of 64 rows 13.8 / 15.8).
//
// Two blocks per workgroup, heavy and light, or all heavy blocks first (sorted): pairs fill the last round badly where the blocks
// of a group are odd in number or few; 8 sequences of 546 rows, 64 heads over 8 together 127.8 (pairs of one head's) / 92.1 us
// (sorted), 32 over 8 65.6 / 51.4.  But blocks of one group, which read the same keys, are then seldom at work together: 1100
// rows, 100 nuggets, 8 x 32 heads 146 (pairs) / 155 us (sorted).
//
// Keys shared by several workgroups: costs a launch and two passes over the partial results (one write, one read), so it is for few
// rows and many keys.  64 rows, 3000 nuggets, 40 heads 56 (whole) -> 23.4 us; 3 x 23 rows, 2700 nuggets, 40 heads 59 -> 41; 128 rows,
// 1000 nuggets, 32 heads 27.4 -> 18.6.  512 rows, 400 nuggets, 32 heads (17 MB of partial results for two splits) stay whole: 23.7 us
// against 25.5.  Blocks of 64 rows with KG = 2 or, where these are too many or would get too few shares, of 128 with KG = 1; 64 / 128:
// 128 rows, 1000 nuggets, 32 heads 19.1 / 22.5, 1500 nuggets, 64 heads over 8 24.7 / 23.5, 83 rows, 671 nuggets, 2 x 32 heads 18.6 / 20.4; 549
// rows, 3578 nuggets, 32 heads - / 62.7 (8 wavefronts, whole: 79.6), 466 rows, 3747 nuggets, 32 heads 87.5 (whole) / 61.6.  Starts and ends, the
// second launch, 400 ns for every share and 4 TB/s for the partial results: fitted to 206 shapes, all share counts of both timed.
// The bounds decide, also where they promise more than there is: in the cached form max_k may be a capacity.  64 rows, 32 heads over
// a cache of 8192 rows, whole / shared: empty 6.8 / 12.5 us, 1% full 9.7 / 13.2, 5% 16.4 / 15.6, 10% 24.4 / 18.5, full 179 / 41;
// 4 sequences over 4096 rows each: 1% 8.6 / 15.5, 10% 17.6 / 19.5, 25% 29.6 / 27.0, full 96 / 58.
BlockPlan plan_blocks(int32_t B, int32_t H, int32_t H_kv, int32_t d_h, int32_t max_q, int32_t max_k, int32_t max_local, bool heavy_last,
                      int64_t max_splits) {
  const int64_t cus = compute_units(), nug_tiles = (static_cast<int64_t>(max_k) + kBN - 1) / kBN;
  const int64_t tiles = nug_tiles + (static_cast<int64_t>(max_local) + kBN - 1) / kBN;
  const auto scaled = [&](int64_t ns) { return d_h == 128 ? ns : ns * 2 / 3; };
  constexpr int64_t kStart4 = 4000, kStart8 = 6200;
  BlockPlan best;
  int64_t best_ns = -1;
  const auto consider = [&](int64_t ns, int32_t G, int32_t waves, int32_t KG, int64_t nsplit, bool pair, bool sorted) {
    if (best_ns >= 0 && ns * 20 >= best_ns * 19) return;
    best_ns = ns;
    best = BlockPlan{G, waves, KG, static_cast<int32_t>(nsplit), pair, sorted};
  };
  // Few rows and many keys stay with an offset that follows the row's maximum (O's error against 64 bits, 549 rows, 3578 nuggets, 32
  // heads 2.23e-3, with the 8-wavefront kernel's fixed offset 2.34e-3), also where that kernel is about as fast: wherever blocks of 128
  // rows that share their keys are, at 2 TB/s for the partial results, faster than that kernel's tiles.
  bool follow = false;
  const int64_t blocks128 = static_cast<int64_t>(B) * H * ((static_cast<int64_t>(max_q) + 127) / 128);
  for (int64_t s = 2; s <= 16 && max_splits > 1 && blocks128 <= cus && s * blocks128 <= 2 * cus && 2 * s <= tiles; ++s)
    follow |= (tiles + s - 1) / s * scaled(s * blocks128 <= cus ? 1350 : 2160) + 5000 +
                  static_cast<int64_t>(split_bytes(B, H, d_h, max_q, s) / 2000) < tiles * scaled(1200);
  for (int32_t G = 1; G <= H / H_kv; ++G) {
    if ((H / H_kv) % G != 0) continue;
    const int64_t pairs = static_cast<int64_t>(B) * (H / G), rows = static_cast<int64_t>(max_q) * G;
    const bool few = pairs % 8 != 0 && pairs < 64 && !heavy_last;  // (see launch_nw)
    for (int32_t waves = 8; waves >= 4; waves -= 4) {
      // (up to 128 query rows the offset follows the row's maximum, whose weight is then 1 and not rounded: 16 x 34 rows over 460
      // nuggets, 64 heads over 8, error against 64 bits 2.19e-3, with the 8-wavefront kernel's fixed offset 2.30e-3)
      if (waves == 8 ? max_q <= 128 || follow : (rows > 128 && max_q > 128 && G == 1)) continue;
      const int64_t bm = 32 * waves, n = (rows + bm - 1) / bm, units = pairs * n, at_once = waves == 8 ? cus : 2 * cus;
      const int64_t tile_ns = scaled(waves == 8 ? (2 * units <= cus ? 1200 : 1600) : units <= cus ? 1350 : 2160);
      const auto block_ns = [&](int64_t blk) {  // the nuggets and what the block's last row sees of the local rows
        const int64_t seen = max_local - max_q + (std::min((blk + 1) * bm, rows) + G - 1) / G;
        return (nug_tiles + (std::max<int64_t>(0, seen) + kBN - 1) / kBN) * tile_ns + (waves == 8 ? kStart8 : kStart4);
      };
      const int64_t rounds = (units + at_once - 1) / at_once;
      if (rounds <= 1) {
        consider(block_ns(n - 1), G, waves, 1, 1, false, false);
        continue;
      }
      int64_t in_turn = 0, paired = -1;  // (blocks of one (sequence, group) run together in the latter only)
      if (rounds <= 16 && !heavy_last) {
        for (int64_t r = 0; r < rounds; ++r) in_turn += block_ns(n - 1 - r * at_once / pairs);
      } else {
        in_turn = rounds * (block_ns(0) + block_ns(n - 1)) / 2;
      }
      if (waves == 8 && 2 * pairs > cus) in_turn = in_turn * 21 / 16;
      const int64_t wgs = (pairs + 7) / 8 * 8 * ((n + 1) / 2);
      if (n >= 2 && wgs >= cus && !few) paired = (wgs + at_once - 1) / at_once * (block_ns(0) + block_ns(n - 1));
      if (paired >= 0 && (heavy_last || rounds > 16 || paired * 20 <= in_turn * 21)) {
        consider(paired, G, waves, 1, 1, true, false);
      } else {
        consider(in_turn, G, waves, 1, 1, false, n >= 2 && !heavy_last);
      }
    }
    // two wavefronts per 32 rows: where that leaves a workgroup per compute unit at most, or up to 64 rows, which have the same
    // workgroups either way, two
    const int64_t units = pairs * ((rows + 63) / 64);
    if (units <= (rows <= 64 ? 2 : 1) * cus) consider(tiles * scaled(units > cus ? 1900 : 1110) + kStart4, G, 4, 2, 1, false, false);
    // keys shared by several workgroups, over blocks of 128 or 64 rows: the better of the two
    int64_t shared_ns = -1, shared_n = 1;
    int32_t shared_KG = 1;
    for (int32_t KG = 1; KG <= 2; ++KG) {
      const int64_t blocks = pairs * ((rows + 128 / KG - 1) / (128 / KG));
      for (int64_t s = 2; s <= std::min<int64_t>(16, max_splits) && blocks <= cus && s * blocks <= 2 * cus && 2 * s <= tiles; ++s) {
        const bool two = s * blocks > cus;  // workgroups on a compute unit
        const int64_t one_ns = KG == 1 ? scaled(two ? 2160 : 1350) : two ? (d_h == 128 ? 1800 : 950) : scaled(1110);
        const int64_t ns = (tiles + 2 * s - 1) / (2 * s) * 2 * one_ns + (KG == 2 ? 7300 : 9000) + 400 * s +
                           static_cast<int64_t>(split_bytes(B, H, d_h, max_q, s) / 4000);
        if (shared_ns >= 0 && ns >= shared_ns) continue;
        shared_ns = ns;
        shared_n = s;
        shared_KG = KG;
      }
    }
    if (shared_ns >= 0) consider(shared_ns, G, 4, shared_KG, shared_n, false, false);
  }
  return best;
}

// Heads that an XCD gets of every sequence, next to each other (0: the pairs of sequence and head go to the XCDs in turn).
// Heads are neighbours in a token's row of 256-byte pieces: with every eighth of them a tile's rows come from two of an
// L2's sixteen channels, which the 8-wavefront kernel feels (8 sequences of 512 rows, 410 nuggets, 32 heads 72.7 -> 70.4 us;
// 2048 rows, 103 nuggets, 40 heads the same), and the query heads of one K/V head are spread over all L2s (64 heads over 8:
// 512 rows 66.7 -> 63.7 us, 128 rows 36.3 -> 33.1; 32 heads over 8, 64 rows 22.2 -> 19.3).  The 4-wavefront kernel, a few
// tiles long, does better without where heads are not grouped (64 rows, 80 nuggets 11.05 against 11.2 us, 128 rows, 410
// nuggets 26.45 against 26.8).
int heads_per_xcd(const AttnParams& p, const BlockPlan& plan) {
  const int HG = p.H / plan.G;
  return HG % 8 == 0 && (plan.waves == 8 || HG != p.H_kv) ? HG / 8 : 0;
}

// nsplit > 1: the keys are shared by that many workgroups per query block, whose partial results the workspace holds.
template <int NW, int KG, bool IDX, int DH, bool SPLIT, bool GROUPED>
int launch_nw(const AttnParams& p, BlockPlan plan) {
  using Cfg = BlockCfg<NW, DH, KG>;
  if (IDX && p.max_k > Cfg::kIdxCap) return DODO_ERR_UNSUPPORTED;
  const int idx_cap = IDX ? Cfg::idx_entries(p.max_k) : 0, lds_bytes = Cfg::kLdsBytes + idx_cap * 4;
  const int HG = p.H / plan.G, nsplit = plan.nsplit;
  const int64_t pairs = static_cast<int64_t>(p.B) * HG, blocks = (static_cast<int64_t>(p.max_q) * plan.G + Cfg::kBM - 1) / Cfg::kBM;
  // few (sequence, group)s that don't deal out evenly would leave XCDs idle: their blocks go to all of them in turn
  if (pairs % 8 != 0 && pairs < 64 && !p.heavy_last) plan.sorted = true;
  const int64_t n_slots = plan.pair ? (blocks + 1) / 2 : blocks;
  const int64_t grid = (plan.sorted ? pairs : (pairs + 7) / 8 * 8) * n_slots;
  if (pairs > 0x7fffffffLL || grid > 0x7fffffffLL) return DODO_ERR_UNSUPPORTED;
  const int n_qblocks = static_cast<int>(blocks), heads_xcd = heads_per_xcd(p, plan);
  auto kern = block_attention_kernel<NW, KG, IDX, DH, SPLIT, GROUPED>;
  const int64_t slots = SPLIT ? static_cast<int64_t>(p.B) * p.max_q * p.H : 0;
  float* part_o = SPLIT ? static_cast<float*>(p.ws) : nullptr;
  float2* part_ml = SPLIT ? reinterpret_cast<float2*>(part_o + slots * nsplit * DH) : nullptr;
  if (lds_bytes > 64 * 1024) {
    const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds_bytes);
    if (rc != DODO_OK) return rc;
  }
  const auto div = [](int64_t d) { return make_fast_div(static_cast<uint32_t>(d)); };
  hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(grid), SPLIT ? nsplit : 1), dim3(Cfg::kThreads), lds_bytes, p.stream,
                     static_cast<const uint16_t*>(p.Q), static_cast<const uint16_t*>(p.Kn),
                     static_cast<const uint16_t*>(p.Vn), static_cast<const uint16_t*>(p.Kl),
                     static_cast<const uint16_t*>(p.Vl), p.cu_q, p.cu_nuggets, p.nug_len, p.cu_local, p.loc_len, p.nug_idx, p.cu_ctx, idx_cap, p.B, p.H, p.H_kv,
                     plan.G, HG, n_qblocks, plan.pair ? 1 : 0, plan.sorted ? 1 : 0, p.heavy_last, heads_xcd, div(heads_xcd > 0 ? heads_xcd : 1),
                     div(n_slots), div(pairs), div(HG), div(plan.G), div(HG / p.H_kv), p.nug_tok_stride, p.nug_head_stride, p.scale_log2e,
                     static_cast<uint16_t*>(p.O), p.lse, part_o, part_ml, slots);
  const int rc = launch_status();
  if (rc != DODO_OK || !SPLIT) return rc;
  constexpr int kRows = kCombineThreads / (DH / 4);
  hipLaunchKernelGGL(combine_splits_kernel<DH>, dim3(static_cast<unsigned>((slots + kRows - 1) / kRows)), dim3(kCombineThreads), 0,
                     p.stream, part_o, part_ml, slots, nsplit, p.cu_q, p.B, p.H, static_cast<uint16_t*>(p.O), p.lse);
  return launch_status();
}

template <int DH>
int launch_dh(const AttnParams& p) {
  // the K/V row offsets inside one tile are kept in 32 bits
  if (p.nug_tok_stride * 2 * kBN > 0x7fffffffLL || static_cast<int64_t>(p.H_kv) * DH * 2 * kBN > 0x7fffffffLL ||
      static_cast<int64_t>(p.H) * DH * 2 * kBN > 0x7fffffffLL)
    return DODO_ERR_UNSUPPORTED;
  int64_t max_splits = p.ws != nullptr && aligned16(p.ws) ? static_cast<int64_t>(p.ws_bytes / split_bytes(p.B, p.H, p.d_h, p.max_q, 1)) : 1;
  const bool idx = p.nug_idx != nullptr;
  if (idx) {
    // a token's byte offset from its sequence's first row is kept in 32 bits as well
    if (static_cast<int64_t>(p.max_n) * p.nug_tok_stride * 2 > 0x7fffffffLL) return DODO_ERR_UNSUPPORTED;
  }
  // (up to 128 query rows a longer list is refused; beyond, the plan is that of the packed form, and so are the bits)
  if (idx && p.max_k > BlockCfg<4, DH, 1>::kShortIdx && p.max_q <= 128) return DODO_ERR_UNSUPPORTED;
  const BlockPlan plan = plan_blocks(p.B, p.H, p.H_kv, p.d_h, p.max_q, p.max_k, p.max_local, p.heavy_last != 0, max_splits);
  const auto launch = [&](auto grouped_tag) {
    constexpr bool GROUPED = decltype(grouped_tag)::value;
    const auto form = [&](auto waves_tag, auto kg_tag, auto split_tag) {
      constexpr int NW = decltype(waves_tag)::value, KG = decltype(kg_tag)::value;
      constexpr bool SPLIT = decltype(split_tag)::value;
      return idx ? launch_nw<NW, KG, true, DH, SPLIT, GROUPED>(p, plan) : launch_nw<NW, KG, false, DH, SPLIT, GROUPED>(p, plan);
    };
    using I4 = std::integral_constant<int, 4>;
    using I8 = std::integral_constant<int, 8>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using Whole = std::false_type;
    using Split = std::true_type;
    if (plan.nsplit > 1) return plan.KG == 2 ? form(I4{}, I2{}, Split{}) : form(I4{}, I1{}, Split{});
    if (plan.KG == 2) return form(I4{}, I2{}, Whole{});
    return plan.waves == 4 ? form(I4{}, I1{}, Whole{}) : form(I8{}, I1{}, Whole{});
  };
  return plan.G > 1 ? launch(std::true_type{}) : launch(std::false_type{});
}

}  // namespace

size_t block_workspace_bytes(int32_t B, int32_t H, int32_t H_kv, int32_t d_h, int32_t max_q, int32_t max_k, int32_t max_local) {
  // (never less than for as many K/V heads as query heads: smaller calls are served with it too)
  int32_t n = 1;
  for (int32_t h = H_kv > 0 ? H_kv : 1; h <= H; ++h)
    if (h == H || h == H_kv || (H_kv <= 0 && H % h == 0))
      n = std::max(n, plan_blocks(B, H, h, d_h, max_q, max_k, max_local, false, 16).nsplit);
  return n > 1 ? split_bytes(B, H, d_h, max_q, n) : 0;
}

int launch_block_attention(const AttnParams& p) {
  if (p.dtype != DODO_DTYPE_BF16) return DODO_ERR_UNSUPPORTED;
  if (p.d_h == 128) return launch_dh<128>(p);
  if (p.d_h == 64) return launch_dh<64>(p);
  return DODO_ERR_UNSUPPORTED;
}

}  // namespace dodo
