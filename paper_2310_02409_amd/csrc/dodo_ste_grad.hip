// dodo_ste_score_grad: the gradient that the straight-through estimator hands
// to the scores (Sec. 2.5, Eq. 17-18 of the Dodo paper).  The score s_i is
// added to the attention logits of nugget i (minus a detached copy, so the
// forward pass is unchanged); its gradient is therefore the sum, over query rows
// j and heads h (and layers: one call per layer, accumulating), of the gradient
// of the loss in the softmax input xi[j, i]:
//     grad[i] = grad_scale * sum_h sum_j P[j,i] * (dP[j,i] - D[j]),
//     P[j,i] = exp(scale q_j.k_i - lse[j]),  dP[j,i] = dO[j].v_i,  D[j] = dO[j].O[j],
// with O and lse as the forward attention call returned them (lse covers the
// local keys as well, so only nugget columns are touched here).
//
// Two contractions (Q K^T and dO V^T) restricted to the nugget columns:
// 4 k q d_h flop per (sequence, head).  bf16 with d_h = 128 or 64 runs on the
// matrix cores: each of a workgroup's 4 wavefronts owns 64 (or 32) nuggets of one
// (sequence, head), whose K and V fragments stay in its registers; the workgroup
// walks over the sequence's query rows in tiles of 32 (Q, dO and O rows stream into
// a 3-stage LDS ring by 16-byte direct loads, two tiles ahead, shared by the 4
// wavefronts), and a wavefront computes S and dP with v_mfma_f32_32x32x16_bf16 so
// that a nugget is a lane and a query row an accumulator register, and adds
// P (dP - D) into a per-lane sum.  D of the next tile's rows comes from its dO and O
// tiles, 8 rows per wavefront, while the matrix cores run; with many nugget tiles, each
// of which would read O and form D again, from a kernel of its own before it (the rule
// is at the launch).  No atomics: per-head sums go to the workspace and a last kernel
// adds them in head order.  Other types and head sizes take a plain kernel, with D from
// the same kernel of its own.
// What bounds it (cycle counter, 8 x 410 nuggets, 512 rows, 32 heads of 128): 24 K of
// a workgroup's 86 K cycles are the wait for K, V and the first tiles; a tile of
// 32 rows takes some 3600 cycles, 2048 of them the matrix instructions of a SIMD's
// two wavefronts, the sums for D 470 and the softmax 780 beside them.  That shape:
// 44 us, 49 to 51 us with the sum over heads (56.5 us before its loop was reworked,
// 41.5 us after a 14 us kernel that made D and lse before that).  2 x 3277 nuggets,
// 1024 rows: 130 us (136 us).  Heads of 64, 4 x 250 nuggets, 300 rows, 16 heads:
// 17.3 us, 2249 us in the plain kernel.  Error against 64 bits (2-norm), 512 rows,
// 410 / 3277 nuggets: 2.9e-7 / 4.1e-7 (were 4.2e-7 / 4.7e-7).
#include <type_traits>

#include "dodo_common.h"

namespace dodo {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kGradWaves = 4;
constexpr int kGradThreads = kGradWaves * kWave;
constexpr int nuggets_per_workgroup(int blocks) { return kGradWaves * 32 * blocks; }  // (blocks of 32 per wavefront)
constexpr int kQTile = 32;                         // query rows per step
constexpr int kStagesSte = 3;
constexpr int kLseChunk = 1024;                    // query rows whose lse sits in LDS at a time
// PRE: D comes from ste_rowdot_kernel instead of the dO and O tiles.
template <int DH, bool PRE>
struct SteDims {
  static constexpr int kRowBytes = DH * 2;
  static constexpr int kPieces = kRowBytes / 16;            // 16-byte pieces of a row
  static constexpr int kRowsPerInstr = 64 / kPieces;        // rows that one direct load instruction brings
  static constexpr int kRowShift = DH == 128 ? 0 : 1;       // rows of 128 bytes cover half of the banks: swizzle by pairs
  static constexpr int kTileBytes = kQTile * kRowBytes;
  static constexpr int kTensors = PRE ? 2 : 3;              // Q tile, dO tile, O tile
  static constexpr int kStageBytes = kTensors * kTileBytes;
  static constexpr int kInstr = 8 / kRowsPerInstr;          // instructions per wavefront, tile and tensor
  static constexpr int kLds = kStagesSte * kStageBytes + (kLseChunk + (PRE ? kLseChunk : 2 * kQTile)) * 4;
  // dP can start from -D, which saves a subtraction per element, but then every accumulation rounds away bits of D, the same
  // for all nuggets of a row; and a lane's sum over the tiles is a chain of rounded additions (4000 rows: 125 tiles).  Against
  // 64 bits (2-norm), 4000 rows, 16 heads of 64: 5.6e-7 so, 2.9e-7 with the subtraction and a compensated sum, in 2 to 8%
  // more time, 3.5e-7 in the plain kernel.  Heads of 128: 4.7e-7 as it is, 1.0e-6 with one chain over all rows; here the
  // 2% that the compensated sum takes alone buy nothing that was there before.
  static constexpr bool kExact = DH == 64;
};
constexpr float kLog2e = 1.4426950408889634f;

// D[h][row] = dO[row,h] . O[row,h] and lse2[h][row] = lse[row,h] * log2(e), head-major so that the rows of a head are
// contiguous.  16 lanes per (row, head), 8 channels per lane and step (d_h % 8 == 0).
template <int DTYPE>
__global__ __launch_bounds__(256) void ste_rowdot_kernel(const void* __restrict__ dO, const void* __restrict__ O,
                                                         const float* __restrict__ lse, int64_t Sq, int H, int d_h,
                                                         float* __restrict__ aux_lse2, float* __restrict__ aux_D) {
  const int64_t t = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / 16;
  const int sub = threadIdx.x % 16;
  const bool live = t < Sq * H;
  float acc = 0.f;
  if (live) {
    for (int c0 = sub * 8; c0 < d_h; c0 += 128) {
      float a[8], o[8];
      if (DTYPE == DODO_DTYPE_F32) {
        const float4* pa = reinterpret_cast<const float4*>(static_cast<const float*>(dO) + t * d_h + c0);
        const float4* po = reinterpret_cast<const float4*>(static_cast<const float*>(O) + t * d_h + c0);
        const float4 a0 = pa[0], a1 = pa[1], o0 = po[0], o1 = po[1];
        a[0] = a0.x; a[1] = a0.y; a[2] = a0.z; a[3] = a0.w; a[4] = a1.x; a[5] = a1.y; a[6] = a1.z; a[7] = a1.w;
        o[0] = o0.x; o[1] = o0.y; o[2] = o0.z; o[3] = o0.w; o[4] = o1.x; o[5] = o1.y; o[6] = o1.z; o[7] = o1.w;
      } else {
        const uint4 av = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(dO) + t * d_h + c0);
        const uint4 ov = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(O) + t * d_h + c0);
        const uint32_t aw[4] = {av.x, av.y, av.z, av.w}, ow[4] = {ov.x, ov.y, ov.z, ov.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[2 * e] = bf16_lo(aw[e]); a[2 * e + 1] = bf16_hi(aw[e]);
          o[2 * e] = bf16_lo(ow[e]); o[2 * e + 1] = bf16_hi(ow[e]);
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = fmaf(a[e], o[e], acc);
    }
  }
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, kWave);
  if (live && sub == 0) {
    const int64_t row = t / H;
    const int h = static_cast<int>(t % H);
    aux_D[h * Sq + row] = acc;
    aux_lse2[h * Sq + row] = lse[t] * kLog2e;
  }
}

template <int DH, bool PRE, int NB>
__global__ __launch_bounds__(kGradThreads, 2) void ste_grad_mfma_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ Kn, const uint16_t* __restrict__ Vn,
    const uint16_t* __restrict__ dO, const uint16_t* __restrict__ O, const float* __restrict__ lse,
    const float* __restrict__ aux_lse2, const float* __restrict__ aux_D, const int32_t* __restrict__ cu_q,
    const int32_t* __restrict__ cu_nuggets, int B, int H, int H_kv, int n_nug_tiles, int64_t Sq, int64_t Kt, int64_t nug_tok_stride, int64_t nug_head_stride, float scale_log2e, float* __restrict__ partial) {
  using SD = SteDims<DH, PRE>;
  constexpr int kWaveNug = 32 * NB, kNugTile = nuggets_per_workgroup(NB);
  constexpr int kRowBytes = SD::kRowBytes, kP = SD::kPieces, kRowShift = SD::kRowShift, kTileBytes = SD::kTileBytes;
  extern __shared__ __attribute__((aligned(1024))) char lds[];  // stages of (Q | dO | O tile), then lse2 of a chunk, D or -D of two tiles or of the chunk
  const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void*)lds));
  // block i runs on XCD i % 8: the nugget tiles of one (sequence, head) sit on one XCD and share Q / dO / O in its L2
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int bh = (slot / n_nug_tiles) * 8 + xcd;
  const int tile = slot % n_nug_tiles;
  if (bh >= B * H) return;
  const int b = bh / H, h = bh % H;
  const int k0 = cu_nuggets[b], k_b = cu_nuggets[b + 1] - k0;
  if (tile * kNugTile >= k_b) return;  // uniform over the workgroup
  const int q0 = cu_q[b], q_b = cu_q[b + 1] - q0;
  const int kvh = h / (H / H_kv);

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave;
  const int n = lane & 31, g = lane >> 5;
  const int nug0 = tile * kNugTile + wave * kWaveNug;  // this wavefront's first nugget
  const bool active = nug0 < k_b;                      // (the others only help to load and with D)

  // loader: a stage is 32 query rows of Q, dO and O; wavefront w brings rows 8w .. 8w+7 of each, whole rows; the 16-byte
  // piece at position pos of LDS row r is piece pos ^ ((r >> kRowShift) & (kP - 1)) of the row, which keeps the fragment
  // reads below conflict-free
  const int l_row = lane / kP, l_pos = lane % kP;
  const int64_t row_stride = static_cast<int64_t>(H) * DH;  // elements between query rows
  const int64_t row0 = (static_cast<int64_t>(q0) * H + h) * DH;
  const int n_qtiles = (q_b + kQTile - 1) / kQTile;
  constexpr int kLoads = SD::kTensors * SD::kInstr;  // direct loads per wavefront per tile
  // Requested through buffers that end with the tile's last row: the lanes' offsets are the same for every tile, and a tile past
  // the end fetches nothing.  Every row of a tile is one of the sequence: the last tile ends with the sequence and begins with
  // rows of the one before, and a sequence of fewer rows than a tile repeats its last one; such rows have weight 0.  (Zeros in
  // their place would make NaN of an infinite channel of K, which a weight of 0 does not take away; a copy in LDS before the last
  // tile cost 3% of a call, offsets clamped for it 1 to 2.5%, this nothing.)
  uint32_t voff[SD::kInstr];
#pragma unroll
  for (int u = 0; u < SD::kInstr; ++u) {
    const int row = 8 * wave + SD::kRowsPerInstr * u + l_row;
    voff[u] = static_cast<uint32_t>(min(row, q_b - 1)) * static_cast<uint32_t>(row_stride * 2) + ((l_pos ^ ((row >> kRowShift) & (kP - 1))) << 4);
  }
  const int last_first = max(0, q_b - kQTile);  // first row of the last tile
  const uint32_t tile_range = static_cast<uint32_t>(min(kQTile, q_b) - 1) * static_cast<uint32_t>(row_stride * 2) + kRowBytes;
  auto buffer_of = [&](const uint16_t* base, uint32_t first_byte, uint32_t range) {
    const uint64_t a = reinterpret_cast<uint64_t>(base) + first_byte;
    u32x4_t buf;
    buf.x = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a));
    buf.y = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32) & 0xffffu);
    buf.z = __builtin_amdgcn_readfirstlane(range);
    buf.w = 0x00027000u;
    return buf;
  };
  auto issue_tile = [&](int t) {
    const uint32_t range = t < n_qtiles ? tile_range : 0u;
    // (a sequence's rows span less than 2^31 bytes: checked on the host)
    const uint32_t first = static_cast<uint32_t>(min(t * kQTile, last_first)) * static_cast<uint32_t>(row_stride * 2);
    const u32x4_t qb = buffer_of(Q + row0, first, range), db = buffer_of(dO + row0, first, range);
    u32x4_t ob = db;
    if (!PRE) ob = buffer_of(O + row0, first, range);
    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_base + (t % kStagesSte) * SD::kStageBytes + 8 * wave * kRowBytes);
#pragma unroll
    for (int u = 0; u < SD::kInstr; ++u) {
      dma16_buffer(qb, voff[u], dst + u * 1024);
      dma16_buffer(db, voff[u], dst + kTileBytes + u * 1024);
      if (!PRE) dma16_buffer(ob, voff[u], dst + 2 * kTileBytes + u * 1024);
    }
  };
  if (n_qtiles > 0) {
    issue_tile(0);
    issue_tile(1);
  }

  // lse (base 2) of a chunk of this (sequence, head)'s query rows, in the tiles' order; +inf makes the weight of a row that has been
  // counted, or that repeats the last one, 0
  float* lse2_l = reinterpret_cast<float*>(lds + kStagesSte * SD::kStageBytes);
  float* dd_l = lse2_l + kLseChunk;
  auto load_lse = [&](int r0) {
    for (int r = tid; r < min(kLseChunk, n_qtiles * kQTile - r0); r += kGradThreads) {
      const int last = (n_qtiles - 1) * kQTile;
      const int row = r0 + r >= last ? last_first + (r0 + r - last) : r0 + r;
      const bool ok = row < q_b && (r0 + r < last || row >= last);
      if (PRE) {
        const int64_t at = static_cast<int64_t>(h) * Sq + q0 + row;
        const float D = ok ? aux_D[at] : 0.f;
        lse2_l[r] = ok ? aux_lse2[at] : __builtin_inff();
        dd_l[r] = SD::kExact ? D : -D;
      } else {
        lse2_l[r] = ok ? lse[static_cast<int64_t>(q0 + row) * H + h] * kLog2e : __builtin_inff();
      }
    }
  };
  load_lse(0);

  // K and V fragments of the 32-nugget blocks (B operands: lane (n, g) holds channels 16 ks + 8 g .. + 8 of
  // nugget row n); rows past the sequence's last nugget re-read it, their sums are not stored
  bf16x8 kf[NB][DH / 16], vf[NB][DH / 16];
#pragma unroll
  for (int blk = 0; blk < NB; ++blk) {
    const int r = min(nug0 + 32 * blk + n, k_b - 1);
    const int64_t off = static_cast<int64_t>(k0 + r) * nug_tok_stride + static_cast<int64_t>(kvh) * nug_head_stride + 8 * g;
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) {
      kf[blk][ks] = *reinterpret_cast<const bf16x8*>(Kn + off + 16 * ks);
      vf[blk][ks] = *reinterpret_cast<const bf16x8*>(Vn + off + 16 * ks);
    }
  }
  // The fragments are used here for the compiler's eyes: its waits for them then stand here.  (It does not take notice of
  // a wait written in assembly: with only that, it waited for them inside the loop, down to vmcnt(0) at the last matrix
  // instruction of every tile, that is for the tile that had just been requested.)
#pragma unroll
  for (int blk = 0; blk < NB; ++blk)
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) asm volatile("" : "+v"(kf[blk][ks]), "+v"(vf[blk][ks]));
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): tiles 0 and 1 too

  // D (kExact) or -D of tile t's rows, 8 lanes per row with DH / 8 channels each.  A wavefront takes the rows that it loaded itself, so
  // only its own loads have to have landed; the next tile's barrier hands the sums to the others.
  const int d_row = 8 * wave + (lane >> 3), d_sub = lane & 7;
  auto row_dots = [&](int t) {
    const char* rows = lds + (t % kStagesSte) * SD::kStageBytes + kTileBytes + d_row * kRowBytes;
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < kP / 8; ++i) {
      const int off = ((kP / 8 * d_sub + i) ^ ((d_row >> kRowShift) & (kP - 1))) << 4;
      const uint4 av = *reinterpret_cast<const uint4*>(rows + off);
      const uint4 ov = *reinterpret_cast<const uint4*>(rows + kTileBytes + off);
      const uint32_t aw[4] = {av.x, av.y, av.z, av.w}, ow[4] = {ov.x, ov.y, ov.z, ov.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc = fmaf(bf16_lo(aw[e]), bf16_lo(ow[e]), acc);
        acc = fmaf(bf16_hi(aw[e]), bf16_hi(ow[e]), acc);
      }
    }
    acc = lanes_sum<8>(acc);
    if (__builtin_expect(d_sub == 0, 1)) dd_l[(t & 1) * kQTile + d_row] = SD::kExact ? acc : -acc;
  };
  if (!PRE && n_qtiles > 0) row_dots(0);

  float ds[NB] = {}, lost[NB] = {};  // sum, and what its additions rounded away
  for (int t = 0; t < n_qtiles; ++t) {
    if (PRE) __builtin_amdgcn_s_waitcnt(0x0f70 | kLoads);  // this wavefront's part of tile t has landed, t+1 may be in flight
    __syncthreads();  // everyone's part of tile t has landed, its D is there; tile t-1 has been read by everyone
    const int c0 = t * kQTile % kLseChunk;
    if (__builtin_expect(c0 == 0 && t > 0, 0)) {  // (out of the loop's straight line: in it, 1 to 3% of a call)
      load_lse(t * kQTile);
      __syncthreads();
    }
    if (!active) issue_tile(t + 2);
    const float* dd_t = dd_l + (PRE ? c0 : (t & 1) * kQTile);
    const char* stg = lds + (t % kStagesSte) * SD::kStageBytes;
    floatx16 acc_s[NB], acc_p[NB];
    if (active) {
      // S starts from 0, dP from -D or from 0 (SteDims::kExact)
      floatx16 first;
#pragma unroll
      for (int v = 0; v < 16; ++v) first[v] = 0.f;
      if (!SD::kExact) {
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          const float4 dd = *reinterpret_cast<const float4*>(dd_t + 8 * vq + 4 * g);
          first[4 * vq] = dd.x; first[4 * vq + 1] = dd.y; first[4 * vq + 2] = dd.z; first[4 * vq + 3] = dd.w;
        }
      }
#pragma unroll
      for (int blk = 0; blk < NB; ++blk) {
        acc_p[blk] = first;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_s[blk][v] = 0.f;
      }
      const char* qrow = stg + n * kRowBytes;
      const char* drow = stg + kTileBytes + n * kRowBytes;
      // Fragments are requested two steps (eight matrix instructions) ahead, and the tile after next halfway through: at the
      // start of the tile the six requests of every wavefront held up the matrix instructions.  8 x 512 rows, 410 nuggets, 32
      // heads 51.5 -> 48.2 us with the head sums, 1638 nuggets 140.9 -> 136.4, 5 x 777 rows, 64 heads over 8 58.4 -> 54.7; the
      // requests alone 51.5 -> 50.5.
      bf16x8 qr[2], dr[2];
      auto read_frags = [&](int ks) {
        const int piece = ((2 * ks + g) ^ ((n >> kRowShift) & (kP - 1))) << 4;
        qr[ks & 1] = *reinterpret_cast<const bf16x8*>(qrow + piece);
        dr[ks & 1] = *reinterpret_cast<const bf16x8*>(drow + piece);
      };
      read_frags(0);
      read_frags(1);
#pragma unroll
      for (int ks = 0; ks < DH / 16; ++ks) {
        const bf16x8 qa = qr[ks & 1], da = dr[ks & 1];
        if (ks + 2 < DH / 16) read_frags(ks + 2);
        if (ks == DH / 32) issue_tile(t + 2);
#pragma unroll
        for (int blk = 0; blk < NB; ++blk) {
          acc_s[blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qa, kf[blk][ks], acc_s[blk], 0, 0, 0);
          acc_p[blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(da, vf[blk][ks], acc_p[blk], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);  // (the compiler would gather the reads again)
      }
    }
    if (!PRE) {
      __builtin_amdgcn_s_waitcnt(0x0f70 | kLoads);  // this wavefront's part of tile t+1 has landed, t+2 may be in flight
      row_dots(t + 1);  // (past the end: zeros, not used)
    }
    if (!active) continue;
    // accumulator v of a block is query row 8 (v / 4) + 4 g + v % 4 of the tile, for this lane's nugget; a tile's rows are
    // summed before they join the others (shorter chains of rounded additions)
    float part[NB] = {};
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) {
      const float4 l2 = *reinterpret_cast<const float4*>(lse2_l + c0 + 8 * vq + 4 * g);
      const float l2v[4] = {l2.x, l2.y, l2.z, l2.w};
      float ddv[4] = {0.f, 0.f, 0.f, 0.f};
      if (SD::kExact) {
        const float4 dd = *reinterpret_cast<const float4*>(dd_t + 8 * vq + 4 * g);
        ddv[0] = dd.x; ddv[1] = dd.y; ddv[2] = dd.z; ddv[3] = dd.w;
      }
#pragma unroll
      for (int blk = 0; blk < NB; ++blk)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p = __builtin_amdgcn_exp2f(acc_s[blk][4 * vq + e] * scale_log2e - l2v[e]);
          part[blk] = fmaf(p, SD::kExact ? acc_p[blk][4 * vq + e] - ddv[e] : acc_p[blk][4 * vq + e], part[blk]);
        }
    }
#pragma unroll
    for (int blk = 0; blk < NB; ++blk) {
      if (SD::kExact) {
        const float add = part[blk] - lost[blk], sum = ds[blk] + add;
        lost[blk] = (sum - ds[blk]) - add;
        ds[blk] = sum;
      } else {
        ds[blk] += part[blk];
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);  // drain the look-ahead loads before the wavefront ends

  // the two halves of a nugget's query rows sit in lanes n and n + 32
  if (active) {
#pragma unroll
    for (int blk = 0; blk < NB; ++blk) {
      const float both = ds[blk] + __shfl_xor(ds[blk], 32, kWave);
      const int i = nug0 + 32 * blk + n;
      if (g == 0 && i < k_b) partial[static_cast<int64_t>(h) * Kt + k0 + i] = both;
    }
  }
}

// One wavefront per (head, nugget): every lane takes query rows of its own and does the two dot products alone.
template <int DTYPE>
__global__ __launch_bounds__(kWave) void ste_grad_plain_kernel(
    const void* __restrict__ Q, const void* __restrict__ Kn, const void* __restrict__ Vn, const void* __restrict__ dO,
    const float* __restrict__ aux_lse2, const float* __restrict__ aux_D, const int32_t* __restrict__ cu_q,
    const int32_t* __restrict__ cu_nuggets, int B, int H, int H_kv, int d_h, int64_t Sq, int64_t Kt,
    int64_t nug_tok_stride, int64_t nug_head_stride, float scale_log2e, float* __restrict__ partial) {
  const int64_t kk = blockIdx.x;  // nugget (packed index)
  const int h = blockIdx.y;
  if (kk >= cu_nuggets[B]) return;
  int lo = 0, hi = B;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cu_nuggets[mid] <= kk) lo = mid; else hi = mid;
  }
  const int b = lo;
  const int q0 = cu_q[b], q_b = cu_q[b + 1] - q0;
  const int kvh = h / (H / H_kv);
  const int64_t koff = kk * nug_tok_stride + static_cast<int64_t>(kvh) * nug_head_stride;
  float acc = 0.f;
  for (int j = threadIdx.x; j < q_b; j += kWave) {
    const int64_t qoff = (static_cast<int64_t>(q0 + j) * H + h) * d_h;
    float s = 0.f, dp = 0.f;
    for (int c = 0; c < d_h; ++c) {
      s = fmaf(load_elem<DTYPE>(Q, qoff + c), load_elem<DTYPE>(Kn, koff + c), s);
      dp = fmaf(load_elem<DTYPE>(dO, qoff + c), load_elem<DTYPE>(Vn, koff + c), dp);
    }
    const float p = __builtin_amdgcn_exp2f(s * scale_log2e - aux_lse2[static_cast<int64_t>(h) * Sq + q0 + j]);
    acc = fmaf(p, dp - aux_D[static_cast<int64_t>(h) * Sq + q0 + j], acc);
  }
#pragma unroll
  for (int off = kWave / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, kWave);
  if (threadIdx.x == 0) partial[static_cast<int64_t>(h) * Kt + kk] = acc;
}

// grad[k] = (accumulate ? grad[k] : 0) + grad_scale * sum over heads, in head order.  A workgroup takes 8 nuggets:
// all of their per-head sums are fetched at once (thread (h mod 32, nugget)), then one thread per nugget adds them.
__global__ __launch_bounds__(256) void ste_reduce_heads_kernel(const float* __restrict__ partial, int H, int64_t Kt,
                                                               const int32_t* __restrict__ cu_nuggets, int B,
                                                               float grad_scale, int accumulate,
                                                               float* __restrict__ grad) {
  extern __shared__ float vals[];  // [H][8]
  const int kk = threadIdx.x & 7;
  const int64_t k = static_cast<int64_t>(blockIdx.x) * 8 + kk;
  const bool live = k < Kt && k < cu_nuggets[B];
  for (int h = threadIdx.x >> 3; h < H; h += 32) vals[h * 8 + kk] = live ? partial[static_cast<int64_t>(h) * Kt + k] : 0.f;
  __syncthreads();
  if (threadIdx.x < 8 && live) {
    float s = 0.f;
    for (int h = 0; h < H; ++h) s += vals[h * 8 + kk];
    s *= grad_scale;
    grad[k] = accumulate ? grad[k] + s : s;
  }
}

__global__ void fill_zero_kernel(float* __restrict__ p, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

}  // namespace
}  // namespace dodo

extern "C" size_t dodo_ste_score_grad_workspace_bytes(int64_t Sq, int32_t H, int64_t Kt) {
  if (Sq <= 0 || H <= 0 || Kt <= 0) return 0;
  return (static_cast<size_t>(2) * Sq * H + static_cast<size_t>(H) * Kt) * sizeof(float);
}

extern "C" int dodo_ste_score_grad(const void* Q, const void* Kn, const void* Vn, const void* dO, const void* O,
                                   const float* lse, const int32_t* cu_q, const int32_t* cu_nuggets, int32_t B,
                                   int32_t H, int32_t H_kv, int32_t d_h, int32_t max_q, int32_t max_k, int64_t Sq,
                                   int64_t Kt, float softmax_scale, float grad_scale, int accumulate, int dtype,
                                   int layout, float* grad_scores, void* ws, size_t ws_bytes, void* stream) {
  using namespace dodo;
  if (B < 0 || H <= 0 || H_kv <= 0 || d_h <= 0 || max_q < 0 || max_k < 0 || Sq < 0 || Kt < 0) return DODO_ERR_INVALID_ARG;
  if (H % H_kv != 0) return DODO_ERR_INVALID_ARG;
  if (layout != DODO_LAYOUT_TOKEN_MAJOR && layout != DODO_LAYOUT_HEAD_MAJOR) return DODO_ERR_INVALID_ARG;
  if (!(softmax_scale == softmax_scale) || !(grad_scale == grad_scale)) return DODO_ERR_INVALID_ARG;
  if (B == 0 || Kt == 0 || max_k == 0) return DODO_OK;
  if (!grad_scores || !cu_q || !cu_nuggets) return DODO_ERR_INVALID_ARG;
  if (!dtype_ok(dtype) || d_h % 8 != 0 || H > 4096) return DODO_ERR_UNSUPPORTED;  // (the last kernel keeps 8 values per head in LDS)
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (Sq == 0 || max_q == 0) {  // no query rows: the gradient of this layer is zero
    if (!accumulate) {
      hipLaunchKernelGGL(fill_zero_kernel, dim3(static_cast<unsigned>((Kt + 255) / 256)), dim3(256), 0, s, grad_scores, Kt);
      return launch_status();
    }
    return DODO_OK;
  }
  if (!Q || !Kn || !Vn || !dO || !O || !lse) return DODO_ERR_INVALID_ARG;
  if (!aligned16(Q) || !aligned16(Kn) || !aligned16(Vn) || !aligned16(dO) || !aligned16(O)) return DODO_ERR_UNSUPPORTED;
  if (Sq * H > 0x7fffffffLL || Kt > 0x7fffffffLL) return DODO_ERR_UNSUPPORTED;
  const size_t need = dodo_ste_score_grad_workspace_bytes(Sq, H, Kt);
  if (!ws || ws_bytes < need) return DODO_ERR_WORKSPACE_TOO_SMALL;
  float* aux_lse2 = static_cast<float*>(ws);
  float* aux_D = aux_lse2 + Sq * H;
  float* partial = aux_D + Sq * H;
  int64_t tok_stride, head_stride;
  if (layout == DODO_LAYOUT_TOKEN_MAJOR) {
    tok_stride = static_cast<int64_t>(H_kv) * d_h;
    head_stride = d_h;
  } else {
    tok_stride = d_h;
    head_stride = Kt * d_h;
  }
  const float scale_log2e = softmax_scale * kLog2e;
  const bool mfma = dtype == DODO_DTYPE_BF16 && (d_h == 128 || d_h == 64) &&
                    static_cast<int64_t>(max_q) * H * d_h * 2 < 0x7fffffffLL;  // row offsets of a sequence in 32 bits
  const auto row_dots = [&]() {
    const unsigned blocks = static_cast<unsigned>((Sq * H * 16 + 255) / 256);
    if (dtype == DODO_DTYPE_BF16)
      hipLaunchKernelGGL(ste_rowdot_kernel<DODO_DTYPE_BF16>, dim3(blocks), dim3(256), 0, s, dO, O, lse, Sq, H, d_h, aux_lse2,
                         aux_D);
    else
      hipLaunchKernelGGL(ste_rowdot_kernel<DODO_DTYPE_F32>, dim3(blocks), dim3(256), 0, s, dO, O, lse, Sq, H, d_h, aux_lse2,
                         aux_D);
    return launch_status();
  };
  int rc;
  if (mfma) {
    const int64_t bh8 = (static_cast<int64_t>(B) * H + 7) / 8 * 8;
    // One block of 32 nuggets per wavefront instead of two (the same bits) where two would leave wavefronts or compute units without
    // any: a row tile's chain is half as long then.  32 heads of 128, two / one: 7 x 980 rows, 82 nuggets 49.1 / 39.0 us, 512 rows, 410
    // nuggets 28.2 / 22.1, 1000 rows, 800 nuggets 44.1 / 33.9, 4 x 400 rows, 128 nuggets 24.2 / 20.2.  With more workgroups than compute
    // units every one of which reads the rows and forms D again: 5 x 800 rows, 250 nuggets 40.6 / 46.2, 4 x 300 rows, 400 nuggets 22.9 /
    // 24.4; heads of 64, 8 x 300 rows, 400 nuggets, 16 heads 17.5 / 16.3.
    const int narrow = (max_k + nuggets_per_workgroup(1) - 1) / nuggets_per_workgroup(1);
    const bool one_block = narrow == 1 || bh8 * narrow <= (d_h == 64 ? 2 : 1) * compute_units();
    const int n_nug_tiles = one_block ? narrow : (max_k + nuggets_per_workgroup(2) - 1) / nuggets_per_workgroup(2);
    const int64_t grid = bh8 * n_nug_tiles;
    if (grid > 0x7fffffffLL) return DODO_ERR_UNSUPPORTED;
    // D in the kernel costs about 0.3 us for every query tile that a compute unit's workgroups walk over, a kernel of
    // its own 2 us and the reading of dO and O (5 TB/s; both in tenths of a us below).  Measured, 32 heads, in the kernel /
    // before it: 8 x 512 rows, 410 nuggets 48.9 / 58.5 us, 1280 nuggets 113 / 109 us, 1638 nuggets 148 / 139 us; 1 x 1024
    // rows, 1000 nuggets 49.0 / 45.6 us; 2 x 1024 rows, 3277 nuggets 135 / 130 us; 1 x 128 rows, 1280 nuggets 14.3 / 15.8 us; 64
    // heads over 8, 5 x 777 rows, 155 nuggets 54.9 / 71.6 us.  (Heads of 64: level.)
    const int64_t steps = (grid + compute_units() - 1) / compute_units() * ((max_q + kQTile - 1) / kQTile);
    const bool pre = d_h == 128 && 3 * steps > 20 + Sq * H / 1000;
    if (pre) {
      rc = row_dots();
      if (rc != DODO_OK) return rc;
    }
    const auto launch = [&](auto kern, int lds_bytes) {
      const int rc_lds = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds_bytes);
      if (rc_lds != DODO_OK) return rc_lds;
      hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(grid)), dim3(kGradThreads), lds_bytes, s,
                         static_cast<const uint16_t*>(Q), static_cast<const uint16_t*>(Kn),
                         static_cast<const uint16_t*>(Vn), static_cast<const uint16_t*>(dO),
                         static_cast<const uint16_t*>(O), lse, aux_lse2, aux_D, cu_q, cu_nuggets, B, H, H_kv, n_nug_tiles,
                         Sq, Kt, tok_stride, head_stride, scale_log2e, partial);
      return DODO_OK;
    };
    const auto launch_blocks = [&](auto blocks_tag) {
      constexpr int NB = decltype(blocks_tag)::value;
      return pre          ? launch(ste_grad_mfma_kernel<128, true, NB>, SteDims<128, true>::kLds)
             : d_h == 128 ? launch(ste_grad_mfma_kernel<128, false, NB>, SteDims<128, false>::kLds)
                          : launch(ste_grad_mfma_kernel<64, false, NB>, SteDims<64, false>::kLds);
    };
    rc = one_block ? launch_blocks(std::integral_constant<int, 1>{}) : launch_blocks(std::integral_constant<int, 2>{});
    if (rc != DODO_OK) return rc;
  } else {
    if (H > 65535) return DODO_ERR_UNSUPPORTED;
    const dim3 grid(static_cast<unsigned>(Kt), static_cast<unsigned>(H));
    rc = row_dots();
    if (rc != DODO_OK) return rc;
    if (dtype == DODO_DTYPE_BF16) {
      hipLaunchKernelGGL(ste_grad_plain_kernel<DODO_DTYPE_BF16>, grid, dim3(kWave), 0, s, Q, Kn, Vn, dO, aux_lse2, aux_D,
                         cu_q, cu_nuggets, B, H, H_kv, d_h, Sq, Kt, tok_stride, head_stride, scale_log2e, partial);
    } else {
      hipLaunchKernelGGL(ste_grad_plain_kernel<DODO_DTYPE_F32>, grid, dim3(kWave), 0, s, Q, Kn, Vn, dO, aux_lse2, aux_D,
                         cu_q, cu_nuggets, B, H, H_kv, d_h, Sq, Kt, tok_stride, head_stride, scale_log2e, partial);
    }
  }
  rc = launch_status();
  if (rc != DODO_OK) return rc;
  hipLaunchKernelGGL(ste_reduce_heads_kernel, dim3(static_cast<unsigned>((Kt + 7) / 8)), dim3(256),
                     static_cast<size_t>(H) * 8 * sizeof(float), s, partial, H, Kt, cu_nuggets, B, grad_scale, accumulate,
                     grad_scores);
  return launch_status();
}
