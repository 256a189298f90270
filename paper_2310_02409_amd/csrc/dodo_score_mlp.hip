// dodo_score_mlp: the scorer as the 2-layer feedforward network of the Dodo
// paper's appendix (Sec. 2.1, App. B: d -> d_hid -> 1, 16.8 M parameters for
// d = d_hid = 4096):
//     s[t] = sum_j w2[j] * act( sum_c W1[j,c] x[t,c] + b1[j] ) + b2.
// The paper does not name the activation; ReLU, GELU (erf form) and tanh are
// offered.  2 N d d_hid flop: a dense contraction, so it runs on the matrix cores.
//
// Up to 20 or 28 tokens (bf16, d % 64 == 0, d_hid % 256 == 0; up to 64 where d % 128 != 0):
// a kernel that streams W1 once over all compute units (score_mlp_few_kernel).  Up to a
// few hundred: tiles of 64 tokens, several steps in flight (score_mlp_some_kernel).
//
// MFMA kernel (the same shapes, more tokens): a workgroup of 8 wavefronts
// owns 256 tokens and walks over 256-wide tiles of hidden units (or 4 wavefronts
// 128 of each, for the tokens that do not fill the chip that way: plan_mlp);
// for each it accumulates H^T = W1_tile X^T over d in steps of 64 channels with
// v_mfma_f32_32x32x16_bf16 (A = W1 rows, B = token rows, so that a token is a lane
// of the accumulators and the reduction over hidden units stays inside a lane),
// then applies bias, activation and w2 to the accumulators and adds them to the
// tokens' partial scores.  The N x d_hid intermediate never leaves the registers.
// X and W1 tiles stream global -> LDS with 16-byte direct loads of whole 128-byte
// rows into two stages of 64 (32) KiB; the 16-byte pieces of a row are XOR-swizzled so
// that the fragment reads are conflict-free (measured: no bank-conflict cycles).
// One barrier per step, after the third of its four 16-channel parts: by then a
// wavefront holds the last part's fragments in registers, so the stage can be
// refilled (for the step after next) right after the barrier, and the next
// step's first fragments are fetched under the last part's matrix instructions.
// Where there is at most one small tile per compute unit, two groups of 4 wavefronts
// share its channels; all of a step's fragments go to registers then, and a step has
// two barriers: it has landed, and it has been read.
// The hidden tiles are split over workgroups, and the workgroups
// resident on one XCD form a patch of token tiles x splits that share their
// panels through that XCD's L2; a second kernel adds the partial scores in split
// order.  All sums have a fixed order (no atomics): run-to-run deterministic.
//
// Everything else (fp32 inputs, other shapes) takes a plain kernel that keeps a
// few token rows in LDS and gives one wavefront a hidden unit at a time: correct
// for any shape, slow for large ones (W1 is re-read for every group of tokens).
#include <algorithm>

#include "dodo_common.h"

namespace dodo {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kBK = 64;  // channels per step
constexpr int kStagesG = 2;
constexpr int kLoadsPerStep = 8;  // direct loads per wavefront per step (4 of X, 4 of W1)
// TG x HG wavefronts, each with 64 tokens and 32 HB hidden units of a square tile; KS such groups of wavefronts share the
// channels.
template <int HB, int TG, int HG, int KS>
struct MlpTile {
  static constexpr int kWaves = TG * HG;
  static constexpr int kThreads = KS * kWaves * kWave;
  static constexpr int kTok = 64 * TG;       // tokens per workgroup
  static constexpr int kHid = 32 * HB * HG;  // hidden units per tile
  static constexpr int kOperandBytes = kTok * kBK * 2;  // one operand tile of a stage
  static constexpr int kStageBytes = 2 * kOperandBytes;
  static constexpr int kChannels = KS * kBK;  // per step
  static constexpr int kLds = KS * kStagesG * kStageBytes;
  static constexpr int kGroupsPerCu = kLds > 80 * 1024 ? 1 : 2;
  static_assert(kTok == kHid && kTok / kWaves == 32, "every wavefront brings 32 rows of either operand per step");
};
using MlpBig = MlpTile<4, 4, 2, 1>;    // 256 x 256, 128 KiB of LDS, 8 wavefronts
using MlpSmall = MlpTile<2, 2, 2, 1>;  // 128 x 128, 64 KiB, 4 wavefronts, two workgroups per compute unit
using MlpHalves = MlpTile<2, 2, 2, 2>;  // the same tile, 8 wavefronts, 128 KiB
constexpr int kTokTile = MlpBig::kTok, kHidTile = MlpBig::kHid;

__device__ __forceinline__ float activation(float h, int act) {
  if (act == DODO_ACT_RELU) return fmaxf(h, 0.f);
  if (act == DODO_ACT_GELU) return 0.5f * h * (1.f + erff(h * 0.70710678118654752440f));
  return tanhf(h);
}

// KS = 2: one hidden tile per workgroup (hsplit = d_hid / kHid), d a multiple of 2 kBK.
// `spread`: consecutive (token tile, split) pairs go to the XCDs in turn; otherwise a token tile stays on one XCD.
template <int HB, int TG, int HG, int KS>
__global__ __launch_bounds__((MlpTile<HB, TG, HG, KS>::kThreads), (MlpTile<HB, TG, HG, KS>::kGroupsPerCu)) void score_mlp_mfma_kernel(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ W1, const float* __restrict__ b1,
    const uint16_t* __restrict__ w2, float b2, int act, int64_t N, int d, int d_hid, int64_t row_stride, int hsplit,
    int spread, float* __restrict__ out) {
  using Tile = MlpTile<HB, TG, HG, KS>;
  constexpr int kOperandBytes = Tile::kOperandBytes, kStageBytesG = Tile::kStageBytes;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void*)lds));
  const int tid = threadIdx.x;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int kg = wave_all / Tile::kWaves, wave = wave_all % Tile::kWaves;  // share of the channels; wavefront of its group
  const int lane = tid % kWave;
  const int j32 = lane & 31, g = lane >> 5;
  const int tg = wave / HG, hg = wave % HG;  // token group (64 tokens) and hidden group (32 HB units) of this wavefront

  // Workgroup -> (token tile, split).  Block i runs on XCD i % 8, and the workgroups resident on one XCD at a time
  // are consecutive slots i / 8: these cover a few token tiles times all the splits, so that their X panels and
  // W1 panels are shared through that XCD's L2 instead of every workgroup streaming panels of its own.  With few
  // token tiles that would leave XCDs idle: there the pairs are dealt out one by one, so that an XCD keeps to its
  // share of W1 (the number of splits being a multiple of 8 in most cases) and works on all tokens.
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int split = static_cast<int>(spread ? blockIdx.x % hsplit : slot % hsplit);
  const int64_t tok_tile = spread ? blockIdx.x / hsplit : static_cast<int64_t>(slot / hsplit) * 8 + xcd;
  const int64_t tok0 = tok_tile * Tile::kTok;
  if (tok0 >= N) return;  // the grid is rounded up to whole groups of 8 token tiles
  const int tiles_total = d_hid / Tile::kHid;
  const int tiles_per_split = (tiles_total + hsplit - 1) / hsplit;
  const int tile0 = split * tiles_per_split;
  const int n_tiles = max(0, min(tiles_per_split, tiles_total - tile0));
  const int ksteps = d / (kBK * KS);
  const int n_steps = n_tiles * ksteps;

  // ---- loader: per step, wavefront w brings rows 32w .. 32w+31 of the X tile and of the W1 tile, 8 rows of 128
  // bytes (1 KiB, whole cache lines) per instruction; lane i sits at (row i/8, position i%8) and fetches the piece
  // that the swizzle stores there: piece = pos ^ ((row >> 1) & 7)
  const int l_row = lane >> 3, l_pos = lane & 7;
  uint32_t x_off[4], w_off[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int r = 32 * wave + 8 * u + l_row;
    const uint32_t piece_bytes = static_cast<uint32_t>((l_pos ^ ((r >> 1) & 7)) * 16);
    const int64_t tok = min(tok0 + r, N - 1);  // rows past the end re-read the last token; nothing of them is stored
    x_off[u] = static_cast<uint32_t>((tok - tok0) * row_stride * 2) + piece_bytes;
    w_off[u] = static_cast<uint32_t>(r) * static_cast<uint32_t>(d) * 2u + piece_bytes;
  }
  const uint16_t* x_base = X + tok0 * row_stride;
  auto issue_part = [&](int step, int q) {  // eighth q of a step's loads: (u = q / 2, operand = q % 2)
    const int st = min(step, n_steps - 1);  // past the end: re-read the last step into a stage nobody reads any more
    const int ht = tile0 + st / ksteps, ks = st % ksteps;
    const uint32_t stage = lds_base + (kg * kStagesG + step % kStagesG) * kStageBytesG;
    const int c0 = (kg * ksteps + ks) * kBK;
    const int u = q >> 1;
    if ((q & 1) == 0) {
      dma16_uniform(x_base + c0, x_off[u], __builtin_amdgcn_readfirstlane(stage + (32 * wave + 8 * u) * 128));
    } else {
      dma16_uniform(W1 + static_cast<int64_t>(ht) * Tile::kHid * d + c0, w_off[u],
            __builtin_amdgcn_readfirstlane(stage + kOperandBytes + (32 * wave + 8 * u) * 128));
    }
  };
  auto issue_step = [&](int step) {
#pragma unroll
    for (int q = 0; q < 8; ++q) issue_part(step, q);
  };

  // ---- fragment addresses: row r of a tile at r*128, piece p at (p ^ ((r >> 1) & 7)) * 16
  const int f_sw = (j32 >> 1) & 7;
  const int x_row_off = (64 * tg + j32) * 128;                    // token blocks tb = 0, 1: + 32*128*tb
  const int w_row_off = kOperandBytes + (32 * HB * hg + j32) * 128;  // hidden blocks hb = 0 .. HB - 1: + 32*128*hb

  floatx16 acc[HB][2];
  float part[2] = {0.f, 0.f};  // partial scores of tokens 64 tg + 32 tb + j32 (this lane's half of the hidden units)
  auto zero_acc = [&]() {
#pragma unroll
    for (int hb = 0; hb < HB; ++hb)
#pragma unroll
      for (int tb = 0; tb < 2; ++tb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[hb][tb][v] = 0.f;
  };
  zero_acc();

  bf16x8 xf[2][2], wf[2][HB];  // two fragment sets, used alternately by the four 16-channel parts of a step
  auto read_frags = [&](int step, int ks, bf16x8* xo, bf16x8* wo) {
    const char* stg = lds + (kg * kStagesG + step % kStagesG) * kStageBytesG;
    const int piece = ((2 * ks + g) ^ f_sw) << 4;
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) xo[tb] = *reinterpret_cast<const bf16x8*>(stg + x_row_off + tb * 4096 + piece);
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) wo[hb] = *reinterpret_cast<const bf16x8*>(stg + w_row_off + hb * 4096 + piece);
  };
  auto mfma_set = [&](int set) {
#pragma unroll
    for (int hb = 0; hb < HB; ++hb)
#pragma unroll
      for (int tb = 0; tb < 2; ++tb)
        acc[hb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[set][hb], xf[set][tb], acc[hb][tb], 0, 0, 0);
  };
  // A hidden tile is complete: accumulator v of block hb is hidden unit 32 hb + 8 (v/4) + 4 g + v%4.  Token blocks
  // tb0 .. tb1 - 1 of this wavefront.
  auto second_layer = [&](int ht, int tb0, int tb1) {
    const int jbase = ht * Tile::kHid + 32 * HB * hg + 4 * g;
#pragma unroll
    for (int hb = 0; hb < HB; ++hb)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        const int jj = jbase + 32 * hb + 8 * vq;
        const float4 bb = *reinterpret_cast<const float4*>(b1 + jj);
        const uint2 ww = *reinterpret_cast<const uint2*>(w2 + jj);
        const float wv[4] = {bf16_lo(ww.x), bf16_hi(ww.x), bf16_lo(ww.y), bf16_hi(ww.y)};
        const float bv[4] = {bb.x, bb.y, bb.z, bb.w};
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
          if (tb >= tb0 && tb < tb1) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              part[tb] = fmaf(wv[e], activation(acc[hb][tb][4 * vq + e] + bv[e], act), part[tb]);
          }
      }
  };
  if (n_steps > 0) {
    issue_step(0);
    issue_step(1);
  }
  if constexpr (KS == 2) {
    // One workgroup per compute unit and 64 KiB per step: what limits it is the time from a stage's refill to its next use.
    // All of a step's fragments go to registers at its start, so the stage is refilled after a quarter of its matrix
    // instructions instead of three (39.3 -> 35.6 us for 128 to 547 tokens at d = d_hid = 4096; 51 us before there were
    // two groups).  With two workgroups per compute unit, which fill each other's waits, that costs (68.5 -> 70.9 us for
    // 2048 tokens).
    bf16x8 xa[4][2], wa[4][HB];
    for (int step = 0; step < n_steps; ++step) {
      __builtin_amdgcn_s_waitcnt(0x0f70 | kLoadsPerStep);  // this step has landed, the next may be on its way
      __syncthreads();
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) read_frags(step, ks, xa[ks], wa[ks]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        if (ks == 1) {
          __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): every fragment of the step is in registers
          __syncthreads();                      // in every wavefront: the stage is free
        }
#pragma unroll
        for (int hb = 0; hb < HB; ++hb)
#pragma unroll
          for (int tb = 0; tb < 2; ++tb) {
            acc[hb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[ks][hb], xa[ks][tb], acc[hb][tb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            const int q = (ks - 1) * 2 * HB + hb * 2 + tb;
            if (q >= 0 && q < kLoadsPerStep) issue_part(step + kStagesG, q);
            __builtin_amdgcn_sched_barrier(0);
          }
      }
    }
  } else {
    if (n_steps > 0) {
      __builtin_amdgcn_s_waitcnt(0x0f70 | kLoadsPerStep);  // step 0 has landed
      __syncthreads();
      read_frags(0, 0, xf[0], wf[0]);
    }
    for (int step = 0; step < n_steps; ++step) {
      // parts 0..2: the next part's fragments are requested, then the matrix cores work on the current part's
      read_frags(step, 1, xf[1], wf[1]);
      mfma_set(0);
      read_frags(step, 2, xf[0], wf[0]);
      mfma_set(1);
      read_frags(step, 3, xf[1], wf[1]);
      mfma_set(0);
      // this wavefront has read everything it needs of this step's stage, and its part of the next step has landed;
      // after the barrier that holds for every wavefront
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
      __syncthreads();
      read_frags(step + 1, 0, xf[0], wf[0]);  // (after the last step: a stage that holds old data; not used)
#pragma unroll
      for (int hb = 0; hb < HB; ++hb) {
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
          acc[hb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[1][hb], xf[1][tb], acc[hb][tb], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int q = 0; q < 4 / HB; ++q) issue_part(step + kStagesG, (2 * hb + tb) * (4 / HB) + q);  // refill this step's stage
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if ((step + 1) % ksteps == 0) {
        second_layer(tile0 + step / ksteps, 0, 2);
        zero_acc();
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);  // drain the look-ahead loads
  __syncthreads();                     // (the stages are about to be reused as a reduction buffer)

  if (KS == 2) {
    // (one hidden tile per workgroup) each group hands the other its sums of the token block that the other finishes
    float* mine = reinterpret_cast<float*>(lds) + (kg * Tile::kWaves + wave) * (HB * 16 * kWave) + lane;
    const float* theirs = reinterpret_cast<const float*>(lds) + ((1 - kg) * Tile::kWaves + wave) * (HB * 16 * kWave) + lane;
#pragma unroll
    for (int hb = 0; hb < HB; ++hb)
#pragma unroll
      for (int v = 0; v < 16; ++v) mine[(hb * 16 + v) * kWave] = kg == 0 ? acc[hb][1][v] : acc[hb][0][v];
    __syncthreads();
#pragma unroll
    for (int hb = 0; hb < HB; ++hb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float other = theirs[(hb * 16 + v) * kWave];
        if (kg == 0) acc[hb][0][v] += other; else acc[hb][1][v] += other;
      }
    if (n_steps > 0) {
      if (kg == 0) second_layer(tile0, 0, 1); else second_layer(tile0, 1, 2);
    }
    __syncthreads();
  }

  // ---- the two halves of a token's hidden units sit in lanes j32 and j32 + 32; the two hidden groups in two
  // wavefronts: added in a fixed order through LDS
  float* red = reinterpret_cast<float*>(lds);  // [HG hidden groups][tokens]
#pragma unroll
  for (int tb = 0; tb < 2; ++tb) {
    const float both = part[tb] + __shfl_xor(part[tb], 32, kWave);
    if (g == 0 && (KS == 1 || tb == kg)) red[hg * Tile::kTok + 64 * tg + 32 * tb + j32] = both;
  }
  __syncthreads();
  if (tid < Tile::kTok) {
    const int64_t tok = tok0 + tid;
    if (tok < N) {
      float s = red[tid] + red[Tile::kTok + tid];
      if (hsplit == 1) {
        s += b2;
        out[tok] = (s == 0.f) ? 0.f : s;
      } else {
        out[static_cast<int64_t>(split) * N + tok] = s;
      }
    }
  }
}

// partial scores of the splits, added in split order, plus the output bias: the first n_big tokens have hs_big splits, the next
// n_small hs_small.  The n_some tokens after them have many splits: a wavefront per token, in the workgroups after thread_blocks,
// every lane adding the splits of its own in order.
constexpr int kCombineThreads = 256;
__global__ __launch_bounds__(kCombineThreads) void score_mlp_combine_kernel(
    const float* __restrict__ partial, int hs_big, int64_t n_big, int hs_small, int64_t n_small, int hs_some, int n_some,
    int thread_blocks, float b2, float* __restrict__ scores) {
  if (static_cast<int>(blockIdx.x) >= thread_blocks) {
    const int t = (blockIdx.x - thread_blocks) * (kCombineThreads / kWave) + threadIdx.x / kWave;
    if (t >= n_some) return;
    const float* p0 = partial + hs_big * n_big + hs_small * n_small + t;
    float s = 0.f;
#pragma unroll 4
    for (int p = lane_id(); p < hs_some; p += kWave) s += p0[static_cast<int64_t>(p) * n_some];
    s = wave_sum64(s) + b2;
    if (lane_id() == 0) scores[n_big + n_small + t] = (s == 0.f) ? 0.f : s;
    return;
  }
  const int64_t t = static_cast<int64_t>(blockIdx.x) * kCombineThreads + threadIdx.x;
  if (t >= n_big + n_small) return;
  const bool big = t < n_big;
  const int splits = big ? hs_big : hs_small;
  const int64_t stride = big ? n_big : n_small;
  const float* p0 = partial + (big ? t : hs_big * n_big + (t - n_big));
  float s = 0.f;
#pragma unroll 8
  for (int p = 0; p < splits; ++p) s += p0[p * stride];
  s += b2;
  scores[t] = (s == 0.f) ? 0.f : s;
}

// ---- few tokens (the streaming mode scores one token per sequence and step) ----
// Bound by reading W1 once (33.5 MB at d = d_hid = 4096: 5 us at the read rate), so the work is spread by bytes of W1:
// every compute unit gets a workgroup with an equal number of hidden units (16 of 4096, 20 of 5120; an incomplete
// block of 16 costs idle lanes of the matrix cores, which have time to spare, and no traffic).  Its 8 wavefronts share
// the channels in runs of 64 (a cache line of a row each), and a wavefront requests up to 16 runs before its first
// matrix instruction; nothing is staged in LDS because no W1 row is used twice.
// v_mfma_f32_16x16x32_bf16 with A = W1 rows, B = token rows (from L2): lane (n, q) holds token n and hidden units
// 4 q .. 4 q + 3.  The wavefronts' sums meet in LDS and are added in wavefront order.
// Measured, d = d_hid = 4096: 13 us for 16 tokens, 24 us for 64 (there the token rows, read from L2 by every workgroup,
// cost more than W1), against 84 us in the tile kernel, whose 16 workgroups walk over the channels one 64-wide step
// after the other; d = d_hid = 5120: 17 and 31 against 190 us.
constexpr int kFewTokens = 64;    // most tokens: four blocks of 16 (beyond, a workgroup re-reads too much of X from L2)
constexpr int kFewWaves = 8;
constexpr int kFewRun = 64;       // channels per run

int few_hid(int32_t d_hid) {  // hidden units per workgroup: at most two blocks of 16
  const int even = (d_hid + compute_units() - 1) / compute_units();
  return even < 32 ? even : 32;
}
int few_splits(int32_t d_hid) { return (d_hid + few_hid(d_hid) - 1) / few_hid(d_hid); }

template <int NB, int RT>  // token blocks of 16, hidden blocks of 16
__global__ __launch_bounds__(kFewWaves * kWave, 2) void score_mlp_few_kernel(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ W1, const float* __restrict__ b1,
    const uint16_t* __restrict__ w2, int act, int N, int d, int d_hid, int hid_per_wg, uint32_t x_stride, uint32_t x_bytes,
    float* __restrict__ partial) {
  // runs of W1 (8 registers each per hidden block) and of X (8 per token block) in flight; 256 registers in all
  constexpr int kXDepth = NB == 1 ? 8 : NB == 2 ? 4 : 3;
  constexpr int kDepth = (RT == 1 ? (NB == 4 ? 12 : 16) : (NB == 4 ? 6 : 8));
  static_assert(kDepth % kXDepth == 0, "one unrolled pass over both rings");
  __shared__ __attribute__((aligned(16))) float red[kFewWaves][NB * 16][RT * 16];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave, n = lane & 15, q = lane >> 4;
  const int h0 = blockIdx.x * hid_per_wg;
  const int n_hid = min(hid_per_wg, d_hid - h0);
  const int runs = d / kFewRun;
  // All loads are unconditional, so that a wait leaves the younger ones in flight; what lies past the last run, hidden
  // unit or token falls outside of the buffers' ranges: it fetches nothing and reads as zeros.
  constexpr uint32_t kOutside = 0x7ffffff0u;
  const auto wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(W1 + static_cast<int64_t>(h0) * d), 0, n_hid * d * 2, 0x00027000);
  const auto xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(X), 0, x_bytes, 0x00027000);
  uint32_t w_off[RT], x_off[NB];
#pragma unroll
  for (int i = 0; i < RT; ++i) w_off[i] = (static_cast<uint32_t>(16 * i + n) * d + 8 * q) * 2;
#pragma unroll
  for (int t = 0; t < NB; ++t) x_off[t] = 16 * t + n < N ? (static_cast<uint32_t>(16 * t + n) * x_stride + 8 * q) * 2 : kOutside;
  floatx4 acc[NB][RT];
#pragma unroll
  for (int t = 0; t < NB; ++t)
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[t][i] = floatx4{0.f, 0.f, 0.f, 0.f};
  u32x4_t wv[kDepth][RT][2], xf[kXDepth][NB][2];
  auto load_w = [&](u32x4_t (&v)[RT][2], int r) {
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const uint32_t off = r < runs ? w_off[i] + static_cast<uint32_t>(r) * (kFewRun * 2) : kOutside;
      v[i][0] = __builtin_amdgcn_raw_buffer_load_b128(wbuf, off, 0, 0);
      v[i][1] = __builtin_amdgcn_raw_buffer_load_b128(wbuf, off, 64, 0);
    }
  };
  auto load_x = [&](u32x4_t (&v)[NB][2], int r) {  // (the halves of a cache line next to each other: the second hits)
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const uint32_t off = r < runs ? x_off[t] + static_cast<uint32_t>(r) * (kFewRun * 2) : kOutside;
      v[t][0] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, off, 0, 0);
      v[t][1] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, off, 64, 0);
    }
  };
  // this wavefront's runs: wave, wave + 8, ...
#pragma unroll
  for (int u = 0; u < kDepth; ++u) {
    load_w(wv[u], wave + u * kFewWaves);
    if (u < kXDepth) load_x(xf[u], wave + u * kFewWaves);
  }
  for (int r0 = wave; r0 < runs; r0 += kFewWaves * kDepth) {
#pragma unroll
    for (int u = 0; u < kDepth; ++u) {
      const int r = r0 + u * kFewWaves;
      if (r >= runs) break;  // uniform over the wavefront
#pragma unroll
      for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int t = 0; t < NB; ++t)
#pragma unroll
          for (int i = 0; i < RT; ++i)
            acc[t][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wv[u][i][half]),
                                                                __builtin_bit_cast(bf16x8, xf[u % kXDepth][t][half]), acc[t][i], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      load_w(wv[u], r + kDepth * kFewWaves);
      load_x(xf[u % kXDepth], r + kXDepth * kFewWaves);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int t = 0; t < NB; ++t)
#pragma unroll
    for (int i = 0; i < RT; ++i) *reinterpret_cast<floatx4*>(&red[wave][16 * t + n][16 * i + 4 * q]) = acc[t][i];
  __syncthreads();
  // 16 lanes per token, one hidden unit of each block per lane
  const int hid = tid & 15;
  float bias[RT], wt[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int h = h0 + min(16 * i + hid, n_hid - 1);
    bias[i] = b1[h];
    wt[i] = load_elem<DODO_DTYPE_BF16>(w2, h);
  }
  for (int tok = tid >> 4; tok < NB * 16; tok += kFewWaves * kWave / 16) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      float h = 0.f;
#pragma unroll
      for (int w = 0; w < kFewWaves; ++w) h += red[w][tok][16 * i + hid];
      // (past the last hidden unit: zeros times a token, NaN where that holds an infinity)
      s = 16 * i + hid < n_hid ? fmaf(wt[i], activation(h + bias[i], act), s) : s;
    }
    s = lanes_sum<16>(s);
    if (hid == 0 && tok < N) partial[static_cast<int64_t>(blockIdx.x) * N + tok] = s;
  }
}

// partial scores of many splits for few tokens: a wavefront per token, every lane adds the splits of its own in order
__global__ __launch_bounds__(kWave) void score_mlp_combine_few_kernel(const float* __restrict__ partial, int splits, int N,
                                                                      float b2, float* __restrict__ scores) {
  const int t = blockIdx.x;
  float s = 0.f;
#pragma unroll 4
  for (int p = lane_id(); p < splits; p += kWave) s += partial[static_cast<int64_t>(p) * N + t];
  s = wave_sum64(s) + b2;
  if (threadIdx.x == 0) scores[t] = (s == 0.f) ? 0.f : s;
}

// ---- some tokens: tiles of 64 tokens and 32 HB hidden units, so that a few hundred tokens fill the chip ----
// Bound by what a compute unit takes from L2 (a step of 128 channels is 24 KiB at HB = 1, 32 KiB at HB = 2, against 128 or 256
// cycles of matrix instructions), so the tile is as large as still gives every compute unit work, and kStages steps are in flight.
// The tile kernel above gives 128 tokens to 32 of 256 compute units at d_hid = 4096 and has one step in flight.
// Wavefronts: 2 groups of 32 tokens times 2 halves of a step's channels (HB = 1) or 2 blocks of 32 hidden units (HB = 2).
constexpr int kSomeTok = 64, kSomeChannels = 128, kSomeRowBytes = kSomeChannels * 2;
template <int HB, int STAGES>
struct SomeTile {
  static constexpr int kHid = 32 * HB;
  static constexpr int kXBytes = kSomeTok * kSomeRowBytes;
  static constexpr int kStageBytes = kXBytes + kHid * kSomeRowBytes;
  static constexpr int kLds = STAGES * kStageBytes;
  static constexpr int kXLoads = 4, kWLoads = 2 * HB, kLoads = kXLoads + kWLoads;  // per wavefront and step, 4 rows each
  static constexpr int kParts = HB == 1 ? 4 : 8;                                    // 16-channel parts of a step per wavefront
};
template <int HB, int STAGES>
__global__ __launch_bounds__(256, 2) void score_mlp_some_kernel(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ W1, const float* __restrict__ b1,
    const uint16_t* __restrict__ w2, int act, int N, int d, int splits, int64_t row_stride, float* __restrict__ partial) {
  using Tile = SomeTile<HB, STAGES>;
  extern __shared__ __attribute__((aligned(1024))) char lds[];  // stages of (64 token rows | 32 HB rows of W1)
  const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void*)lds));
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave, j32 = lane & 31, g = lane >> 5;
  const int tg = wave & 1, part_of = wave >> 1;  // token group; half of the channels or hidden block
  const int split = static_cast<int>(blockIdx.x % splits);  // (the token tiles of a split on one XCD, where 8 divides their number)
  const int tok0 = static_cast<int>(blockIdx.x / splits) * kSomeTok, h0 = split * Tile::kHid;
  const int n_steps = d / kSomeChannels;

  // loader: an instruction brings 4 rows; piece p (16 bytes) of row r sits at position p ^ (r & 15)
  uint32_t x_off[Tile::kXLoads], w_off[Tile::kWLoads];
  const int l_row = lane >> 4, l_pos = lane & 15;
#pragma unroll
  for (int u = 0; u < Tile::kXLoads; ++u) {
    const int r = 4 * (Tile::kXLoads * wave + u) + l_row;
    const int tok = min(tok0 + r, N - 1) - tok0;  // rows past the end re-read the last token; nothing of them is stored
    x_off[u] = static_cast<uint32_t>(tok) * static_cast<uint32_t>(row_stride * 2) + ((l_pos ^ (r & 15)) << 4);
  }
#pragma unroll
  for (int u = 0; u < Tile::kWLoads; ++u) {
    const int r = 4 * (Tile::kWLoads * wave + u) + l_row;
    w_off[u] = static_cast<uint32_t>(r) * static_cast<uint32_t>(d) * 2u + ((l_pos ^ (r & 15)) << 4);
  }
  const uint16_t* x_base = X + static_cast<int64_t>(tok0) * row_stride;
  const uint16_t* w_base = W1 + static_cast<int64_t>(h0) * d;
  auto issue = [&](int step) {  // (past the last step nothing is fetched)
    const uint32_t range = step < n_steps ? 0x7fffffffu : 0u;
    const int c0 = step < n_steps ? step * kSomeChannels : 0;
    const u32x4_t xb = buffer_of(x_base + c0, range), wb = buffer_of(w_base + c0, range);
    const uint32_t stage = lds_base + (step % STAGES) * Tile::kStageBytes;
#pragma unroll
    for (int u = 0; u < Tile::kXLoads; ++u)
      dma16_buffer(xb, x_off[u], __builtin_amdgcn_readfirstlane(stage + (Tile::kXLoads * wave + u) * 1024));
#pragma unroll
    for (int u = 0; u < Tile::kWLoads; ++u)
      dma16_buffer(wb, w_off[u], __builtin_amdgcn_readfirstlane(stage + Tile::kXBytes + (Tile::kWLoads * wave + u) * 1024));
  };
  // Four sums, each of every fourth part, added up every 1024 channels: short chains of rounded additions (against 64 bits, 2-norm,
  // d = 4096: one sum 4e-7, this way 1.3e-7 to 1.6e-7, the kernel for few tokens 1.7e-7 to 2e-7, the tile kernel 3e-7), and no
  // matrix instruction waits for the one before.
  constexpr int kFold = 1024 / kSomeChannels;
  floatx16 acc, acc4[4];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    acc[v] = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc4[i][v] = 0.f;
  }
  auto fold = [&]() {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      acc[v] += (acc4[0][v] + acc4[1][v]) + (acc4[2][v] + acc4[3][v]);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc4[i][v] = 0.f;
    }
  };
#pragma unroll
  for (int t = 0; t < STAGES - 1; ++t) issue(t);
  const int x_row = (32 * tg + j32) * kSomeRowBytes;
  const int w_row = Tile::kXBytes + ((HB == 2 ? 32 * part_of : 0) + j32) * kSomeRowBytes;
  const int first_part = HB == 2 ? 0 : Tile::kParts * part_of;
  constexpr int kYounger = (STAGES - 2) * Tile::kLoads;
  static_assert(kYounger < 64, "vmcnt has six bits");
  for (int step = 0; step < n_steps; ++step) {
    __builtin_amdgcn_s_waitcnt(0x0f70 | (kYounger & 15) | (kYounger >> 4 << 14));  // this wavefront's part of the step has landed
    __syncthreads();  // everyone's has, and everyone has read the step before
    issue(step + STAGES - 1);
    const char* stg = lds + (step % STAGES) * Tile::kStageBytes;
    bf16x8 xf[Tile::kParts], wf[Tile::kParts];
#pragma unroll
    for (int p = 0; p < Tile::kParts; ++p) {
      const int at = ((2 * (first_part + p) + g) ^ (j32 & 15)) << 4;
      xf[p] = *reinterpret_cast<const bf16x8*>(stg + x_row + at);
      wf[p] = *reinterpret_cast<const bf16x8*>(stg + w_row + at);
    }
#pragma unroll
    for (int p = 0; p < Tile::kParts; ++p)
      acc4[p & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[p], xf[p], acc4[p & 3], 0, 0, 0);
    if (step % kFold == kFold - 1) fold();
  }
  fold();
  __builtin_amdgcn_s_waitcnt(0x0f70);
  __syncthreads();  // (the stages become a reduction buffer)
  float* red = reinterpret_cast<float*>(lds);
  if (HB == 1) {  // the halves of the channels, added before the activation
    if (part_of == 1) {
#pragma unroll
      for (int v = 0; v < 16; ++v) red[(tg * 16 + v) * kWave + lane] = acc[v];
    }
    __syncthreads();
    if (part_of == 1) return;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] += red[(tg * 16 + v) * kWave + lane];
  }
  // accumulator v is hidden unit 8 (v / 4) + 4 g + v % 4 of the block, for this lane's token
  float s = 0.f;
  const int hb = h0 + (HB == 2 ? 32 * part_of : 0) + 4 * g;
#pragma unroll
  for (int vq = 0; vq < 4; ++vq) {
    const float4 bb = *reinterpret_cast<const float4*>(b1 + hb + 8 * vq);
    const uint2 ww = *reinterpret_cast<const uint2*>(w2 + hb + 8 * vq);
    const float wv[4] = {bf16_lo(ww.x), bf16_hi(ww.x), bf16_lo(ww.y), bf16_hi(ww.y)}, bv[4] = {bb.x, bb.y, bb.z, bb.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) s = fmaf(wv[e], activation(acc[4 * vq + e] + bv[e], act), s);
  }
  s += __shfl_xor(s, 32, kWave);
  if (HB == 2) {
    if (part_of == 1 && g == 0) red[32 * tg + j32] = s;
    __syncthreads();
    if (part_of == 1) return;
    s += red[32 * tg + j32];
  }
  const int tok = tok0 + 32 * tg + j32;
  if (g == 0 && tok < N) partial[static_cast<int64_t>(split) * N + tok] = s;
}

// ---- plain kernel: `kTok` token rows in LDS, one hidden unit per wavefront at a time
constexpr int kPlainThreads = 256;
template <int DTYPE>
__global__ __launch_bounds__(kPlainThreads) void score_mlp_plain_kernel(
    const void* __restrict__ X, const void* __restrict__ W1, const float* __restrict__ b1, const void* __restrict__ w2,
    float b2, int act, int64_t N, int d, int d_hid, int64_t row_stride, int tok_per_wg, float* __restrict__ scores) {
  extern __shared__ float xs[];  // [tok_per_wg][d] as fp32, then [waves][tok_per_wg] partial sums
  constexpr int kWaves = kPlainThreads / kWave;
  const int64_t tok0 = static_cast<int64_t>(blockIdx.x) * tok_per_wg;
  const int nt = static_cast<int>(min<int64_t>(tok_per_wg, N - tok0));
  for (int i = threadIdx.x; i < nt * d; i += kPlainThreads)
    xs[i] = load_elem<DTYPE>(X, (tok0 + i / d) * row_stride + i % d);
  __syncthreads();
  const int wave = threadIdx.x / kWave, lane = lane_id();
  float* red = xs + static_cast<size_t>(tok_per_wg) * d;
  for (int t = 0; t < nt; ++t) {
    float a = 0.f;
    for (int j = wave; j < d_hid; j += kWaves) {
      float h = 0.f;
      for (int c = lane; c < d; c += kWave) h = fmaf(load_elem<DTYPE>(W1, static_cast<int64_t>(j) * d + c), xs[t * d + c], h);
#pragma unroll
      for (int off = kWave / 2; off >= 1; off >>= 1) h += __shfl_xor(h, off, kWave);
      a = fmaf(load_elem<DTYPE>(w2, j), activation(h + b1[j], act), a);
    }
    if (lane == 0) red[wave * tok_per_wg + t] = a;
  }
  __syncthreads();
  if (threadIdx.x < nt) {
    float s = 0.f;
    for (int w = 0; w < kWaves; ++w) s += red[w * tok_per_wg + threadIdx.x];
    s += b2;
    scores[tok0 + threadIdx.x] = (s == 0.f) ? 0.f : s;
  }
}

bool mfma_path(int dtype, int64_t N, int32_t d, int32_t d_hid, int64_t row_stride, const void* X, const void* W1,
               const void* b1, const void* w2) {
  return dtype == DODO_DTYPE_BF16 && d % kBK == 0 && d_hid % kHidTile == 0 && row_stride % 8 == 0 && aligned16(X) &&
         aligned16(W1) && aligned16(b1) && (reinterpret_cast<uintptr_t>(w2) % 8 == 0) &&
         static_cast<int64_t>(kHidTile) * d * 2 < 0x7fffffffLL && static_cast<int64_t>(kTokTile) * row_stride * 2 < 0x7fffffffLL;
}

// Splits of big tiles throughout, for a workspace that was sized for another number of tokens and is too small for the
// plan below: what the chip needs to be filled, at least four.  A call without room for these is refused.
int hidden_splits(int64_t N, int32_t d_hid) {
  const int64_t blocks = (N + kTokTile - 1) / kTokTile;
  const int tiles = d_hid / kHidTile;
  int hs = 1;
  while (hs * 2 <= tiles && (hs < 4 || blocks * hs < compute_units())) hs *= 2;
  return hs;
}

// The most that this form takes for any number of tokens up to N.  Its need is not even in N (twice the splits as soon as
// half of them leave the chip idle), so a buffer that a caller keeps for falling N has to hold the largest: for every
// number of splits, the need of the most tokens that get it.
size_t hidden_splits_most_bytes(int64_t N, int32_t d_hid) {
  int64_t most = 0;
  for (int hs = 2; hs <= d_hid / kHidTile; hs *= 2) {
    const int64_t last_block = hs <= 4 ? N : (compute_units() + hs / 2 - 1) / (hs / 2) - 1;  // of those with hs splits or more
    const int64_t n = last_block <= N / kTokTile ? last_block * kTokTile : N;
    if (n > 0) most = std::max(most, hidden_splits(n, d_hid) * n);
  }
  return static_cast<size_t>(most) * sizeof(float);
}

// How N tokens are shared out: the first n_big in big tiles (hs_big splits of the hidden units), the rest in small ones.
// A big tile keeps a compute unit for 110 us at d = 4096, so a grid that does not come out in whole rounds of them pays
// for idle units: big tiles take the groups of 8 token tiles (one per XCD) that fill rounds, small ones what is left, and
// everything where there is not one round of big tiles.  The cost of a round, in hundredths of a round of big tiles, was
// measured at d = 1024 to 5120: 60 for small tiles with two workgroups per compute unit (65 of 112 us at d = 4096), which is
// why small tiles do not take it all (2.4 times their share of the work); 45 with at most one, or 32 (35.6 us) where these
// are all there is and have two groups of wavefronts share the channels (which needs an even number of steps).  A second
// round of those would take longer than two workgroups per unit (1500 tokens 69.6 against 58.5 us).
// d = d_hid = 4096, big tiles with four splits at least -> now: 128 tokens 85 -> 36 us, 2048 104 -> 70 us, 4096 the
// same 116 us, 25123 (with their selection) 853 -> 716 us; 5120: 512 tokens 111 -> 44 us.
//
// Up to a few hundred tokens -- all there are, or what whole rounds of the other tiles leave -- take tiles of 64 tokens instead, in one
// round, of 32 hidden units where that is at most one tile per compute unit, of 64 beyond.  d = d_hid = 4096, before -> now: 64 tokens
// 25.2 -> 17.0 us, 128 35.8 -> 17.5, 256 36.3 -> 22.5, 512 36.8 -> 27.5, 2322 109 -> 95 (whole rounds before them); 5120: 128 tokens
// 44.1 -> 26.5, 256 44.3 -> 31.5; 8192: 64 tokens 52.8 -> 37, 128 80 -> 42; 1024: 64 to 2048 tokens 11.2 to 16.2 -> 8.2 to 11.8.
// (32 units with two tiles per compute unit: 256 tokens 24.4 us; more than a round of either: 547 tokens 46 us against 36.)
struct MlpPlan {
  int64_t n_big;
  int hs_big;
  int64_t n_small;
  int hs_small;
  bool halves;  // small tiles: two groups of wavefronts share the channels
  int n_some;
  int hs_some;
  bool direct() const { return n_small == 0 && n_some == 0 && hs_big == 1; }  // the only split writes the scores itself
  size_t bytes() const {
    return direct() ? 0 : (static_cast<size_t>(hs_big) * n_big + static_cast<size_t>(hs_small) * n_small +
                           static_cast<size_t>(hs_some) * n_some) * sizeof(float);
  }
};
constexpr int kBigRound = 100, kSmallHalves = 32, kSmallOne = 45, kSmallTwo = 60;
// Tiles of 64 tokens: 1 (32 hidden units, at most one workgroup per compute unit), 2 (64, one) or 3 (64, two); 0: more than one round of them.
constexpr int kSomeCost[4] = {0, 12, 16, 20};
int some_tiles(int64_t n, int32_t d, int32_t d_hid) {
  const int64_t cus = compute_units(), tiles = (n + kSomeTok - 1) / kSomeTok;
  if (n <= 0 || d % kSomeChannels != 0 || tiles > 2 * cus) return 0;
  if (tiles * (d_hid / 32) <= cus) return 1;
  return tiles * (d_hid / 64) <= cus ? 2 : tiles * (d_hid / 64) <= 2 * cus ? 3 : 0;
}
int some_splits(int64_t n, int32_t d, int32_t d_hid) { return d_hid / (some_tiles(n, d, d_hid) == 1 ? 32 : 64); }
size_t some_bytes(int64_t n, int32_t d, int32_t d_hid) {
  return some_tiles(n, d, d_hid) == 0 ? 0 : static_cast<size_t>(some_splits(n, d, d_hid)) * n * sizeof(float);
}
// Most tokens for which the kernel for few tokens is the faster one where both fit: 28 where these tiles leave half of the compute units
// idle with 2048 channels of W1 or more to bring (d = d_hid = 2048, 21 / 28 tokens: 10.6 / 11.2 us there, 11.3 in tiles; 4096: 15.6 /
// 17.0, 17.3), else 20 (1024, 24 tokens 8.7 against 8.5; 5120, 21 tokens 20.9 against 20.6; 8192 38.4 against 35.9).
int few_best(int32_t d, int32_t d_hid) { return d >= 2048 && d_hid / 32 * 2 <= compute_units() ? 28 : 20; }
// the most that these tiles take for any number of tokens up to N
size_t some_most_bytes(int64_t N, int32_t d, int32_t d_hid) {
  const int64_t cus = compute_units();
  size_t most = 0;
  for (const int64_t tiles : {cus / (d_hid / 32), cus / (d_hid / 64), 2 * cus / (d_hid / 64)})
    most = std::max(most, some_bytes(std::min(N, tiles * kSomeTok), d, d_hid));
  return most;
}
// (some: with tiles of 64 tokens)
MlpPlan plan_mlp(int64_t N, int32_t d, int32_t d_hid, bool some = true) {
  const int cus = compute_units(), cus_xcd = cus >= 8 ? cus / 8 : 1;
  const int tiles = d_hid / MlpBig::kHid, small_tiles = d_hid / MlpSmall::kHid;
  auto small_units = [&](int64_t n) -> int64_t { return (n + MlpSmall::kTok - 1) / MlpSmall::kTok * small_tiles; };
  auto in_halves = [&](int64_t n) { return d % MlpHalves::kChannels == 0 && small_units(n) <= cus; };
  auto small_cost = [&](int64_t n) -> int64_t {
    const int64_t units = small_units(n);
    if (units > 0 && in_halves(n)) return kSmallHalves;
    const int64_t rest = units % (2 * cus);
    return units / (2 * cus) * kSmallTwo + (rest == 0 ? 0 : rest <= cus ? kSmallOne : kSmallTwo);
  };
  // (beyond 32 groups the rounds repeat: 32 groups are as many whole rounds as there are hidden tiles)
  const int64_t groups_all = (N + 8 * MlpBig::kTok - 1) / (8 * MlpBig::kTok);
  int64_t best_groups = 0, best = -1, best_some = 0;
  const int64_t small_round = 2 * cus / small_tiles * MlpSmall::kTok;  // tokens of one (0: more than one round for any)
  for (int64_t t = groups_all; t >= 0 && t > groups_all - 33; --t) {
    const int64_t n_big = t * 8 * MlpBig::kTok < N ? t * 8 * MlpBig::kTok : N, rest = N - n_big;
    const int64_t rounds = (t * tiles + cus_xcd - 1) / cus_xcd * kBigRound;
    const auto consider = [&](int64_t n_some) {
      // (a launch of their own after another one's tail: 8 us, 7 hundredths of a round at d = 4096; at d = 1024 25123 tokens with
      // their last 547 this way 84 us, without 71.5)
      const int64_t more = n_some > 0 && n_some < N ? 30000 / d : 0;
      const int64_t cost = rounds + small_cost(rest - n_some) + kSomeCost[some_tiles(n_some, d, d_hid)] + more;
      if (best >= 0 && cost >= best) return;
      best = cost;
      best_groups = t;
      best_some = n_some;
    };
    consider(0);
    if (!some) continue;
    if (some_tiles(rest, d, d_hid) > 0) consider(rest);
    if (small_round > 0 && rest > small_round && some_tiles(rest % small_round, d, d_hid) > 0) consider(rest % small_round);
  }
  MlpPlan p;
  p.n_big = best_groups * 8 * MlpBig::kTok < N ? best_groups * 8 * MlpBig::kTok : N;
  p.n_some = static_cast<int>(best_some);
  p.hs_some = best_some > 0 ? some_splits(best_some, d, d_hid) : 0;
  p.n_small = N - p.n_big - best_some;
  p.hs_small = small_tiles;
  p.halves = in_halves(p.n_small);
  // as many tiles per workgroup as leave the number of rounds alone (fewer starts and partial scores)
  const int64_t rounds = (best_groups * tiles + cus_xcd - 1) / cus_xcd;
  p.hs_big = tiles;
  for (int per = tiles; per > 1; --per)
    if (tiles % per == 0 && (best_groups * (tiles / per) + cus_xcd - 1) / cus_xcd * per <= rounds) {
      p.hs_big = tiles / per;
      break;
    }
  return p;
}

template <class Tile, class Kernel>
int launch_mfma(Kernel kern, const uint16_t* X, const uint16_t* W1, const float* b1, const uint16_t* w2, float b2, int act,
                int64_t N, int d, int d_hid, int64_t row_stride, int hs, int spread, float* out, hipStream_t s) {
  const int64_t tok_tiles = (N + Tile::kTok - 1) / Tile::kTok;
  const int64_t blocks = (spread ? tok_tiles : (tok_tiles + 7) / 8 * 8) * hs;
  if (blocks > 0x7fffffffLL) return DODO_ERR_UNSUPPORTED;
  const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(kern), Tile::kLds);
  if (rc != DODO_OK) return rc;
  hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(blocks)), dim3(Tile::kThreads), Tile::kLds, s, X, W1, b1, w2, b2, act, N, d,
                     d_hid, row_stride, hs, spread, out);
  return launch_status();
}

template <int HB, int STAGES>
int launch_some(const uint16_t* X, const uint16_t* W1, const float* b1, const uint16_t* w2, int act, int n, int d, int splits,
                int64_t row_stride, float* out, hipStream_t s) {
  const int lds = SomeTile<HB, STAGES>::kLds;
  const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(score_mlp_some_kernel<HB, STAGES>), lds);
  if (rc != DODO_OK) return rc;
  hipLaunchKernelGGL((score_mlp_some_kernel<HB, STAGES>), dim3((n + kSomeTok - 1) / kSomeTok * splits), dim3(256), lds, s, X, W1, b1, w2,
                     act, n, d, splits, row_stride, out);
  return launch_status();
}

}  // namespace
}  // namespace dodo

extern "C" size_t dodo_score_mlp_workspace_bytes(int dtype, int64_t N, int32_t d, int32_t d_hid) {
  using namespace dodo;
  if (N <= 0 || d <= 0 || d_hid <= 0) return 0;
  if (dtype != DODO_DTYPE_BF16 || d % kBK != 0 || d_hid % kHidTile != 0) return 0;
  // room for this N, and for every smaller one as well: a caller may keep the buffer
  const size_t few = static_cast<size_t>(few_splits(d_hid)) * (N < kFewTokens ? N : kFewTokens) * sizeof(float);
  const size_t least = hidden_splits_most_bytes(N, d_hid);
  const size_t plan = N <= kFewTokens ? 0 : std::max(plan_mlp(N, d, d_hid).bytes(), plan_mlp(N, d, d_hid, false).bytes());
  return std::max({plan, few, least, some_most_bytes(N, d, d_hid)});
}

extern "C" int dodo_score_mlp(const void* hidden, const void* W1, const float* b1, const void* w2, float b2, int act,
                              int dtype, int64_t N, int32_t d, int32_t d_hid, int64_t row_stride, float* scores,
                              void* ws, size_t ws_bytes, void* stream) {
  using namespace dodo;
  if (N < 0 || d <= 0 || d_hid <= 0 || row_stride < d) return DODO_ERR_INVALID_ARG;
  if (act != DODO_ACT_RELU && act != DODO_ACT_GELU && act != DODO_ACT_TANH) return DODO_ERR_INVALID_ARG;
  if (N == 0) return DODO_OK;
  if (!hidden || !W1 || !b1 || !w2 || !scores) return DODO_ERR_INVALID_ARG;
  if (!dtype_ok(dtype)) return DODO_ERR_UNSUPPORTED;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (mfma_path(dtype, N, d, d_hid, row_stride, hidden, W1, b1, w2)) {
    float* partial = static_cast<float*>(ws);
    const size_t room = ws != nullptr ? ws_bytes : 0;
    const bool some = N > few_best(d, d_hid) && some_tiles(N, d, d_hid) > 0 && room >= some_bytes(N, d, d_hid);  // (then that is the plan)
    if (N <= kFewTokens && !some && room >= static_cast<size_t>(few_splits(d_hid)) * N * sizeof(float)) {
      const int splits = few_splits(d_hid), hid = few_hid(d_hid), n = static_cast<int>(N);
      const uint32_t x_bytes = static_cast<uint32_t>(((N - 1) * row_stride + d) * 2);
#define DODO_LAUNCH_FEW(NB, RT)                                                                                          \
  hipLaunchKernelGGL((score_mlp_few_kernel<NB, RT>), dim3(splits), dim3(kFewWaves* kWave), 0, s,                         \
                     static_cast<const uint16_t*>(hidden), static_cast<const uint16_t*>(W1), b1,                        \
                     static_cast<const uint16_t*>(w2), act, n, d, d_hid, hid, static_cast<uint32_t>(row_stride), x_bytes, partial)
      if (hid <= 16) {
        if (n <= 16) DODO_LAUNCH_FEW(1, 1); else if (n <= 32) DODO_LAUNCH_FEW(2, 1); else DODO_LAUNCH_FEW(4, 1);
      } else {
        if (n <= 16) DODO_LAUNCH_FEW(1, 2); else if (n <= 32) DODO_LAUNCH_FEW(2, 2); else DODO_LAUNCH_FEW(4, 2);
      }
#undef DODO_LAUNCH_FEW
      const int rc = launch_status();
      if (rc != DODO_OK) return rc;
      hipLaunchKernelGGL(score_mlp_combine_few_kernel, dim3(n), dim3(kWave), 0, s, partial, splits, n, b2, scores);
      return launch_status();
    }
    MlpPlan p = plan_mlp(N, d, d_hid);
    // a buffer that was sized for another number of tokens may hold the plan without tiles of 64 tokens though not this one (d = 4096,
    // 6348 tokens in the buffer of 6793 228 us in the last form, 224 so; d = 2048, 6165 in that of 6987 127 / 123), or neither
    if (room < p.bytes()) p = plan_mlp(N, d, d_hid, false);
    if (room < p.bytes()) {
      p = MlpPlan{N, hidden_splits(N, d_hid), 0, 0, false, 0, 0};
      if (room < p.bytes()) return DODO_ERR_WORKSPACE_TOO_SMALL;
    }
    const uint16_t* x = static_cast<const uint16_t*>(hidden);
    const uint16_t* w = static_cast<const uint16_t*>(W1);
    const uint16_t* wo = static_cast<const uint16_t*>(w2);
    if (p.n_big > 0) {  // (a single split adds the output bias itself; where the sums are combined, that comes later)
      const int rc = launch_mfma<MlpBig>(score_mlp_mfma_kernel<4, 4, 2, 1>, x, w, b1, wo, p.direct() ? b2 : 0.f, act, p.n_big, d, d_hid, row_stride,
                                         p.hs_big, 0, p.direct() ? scores : partial, s);
      if (rc != DODO_OK || p.direct()) return rc;
    }
    if (p.n_small > 0) {
      const int rc = p.halves
          ? launch_mfma<MlpHalves>(score_mlp_mfma_kernel<2, 2, 2, 2>, x + p.n_big * row_stride, w, b1, wo, b2, act, p.n_small,
                                   d, d_hid, row_stride, p.hs_small, 1, partial + p.hs_big * p.n_big, s)
          : launch_mfma<MlpSmall>(score_mlp_mfma_kernel<2, 2, 2, 1>, x + p.n_big * row_stride, w, b1, wo, b2, act, p.n_small,
                                  d, d_hid, row_stride, p.hs_small, 1, partial + p.hs_big * p.n_big, s);
      if (rc != DODO_OK) return rc;
    }
    if (p.n_some > 0) {
      const uint16_t* xs = x + (p.n_big + p.n_small) * row_stride;
      float* out = partial + p.hs_big * p.n_big + p.hs_small * p.n_small;
      const int form = some_tiles(p.n_some, d, d_hid);
      const int rc = form == 1   ? launch_some<1, 3>(xs, w, b1, wo, act, p.n_some, d, p.hs_some, row_stride, out, s)
                     : form == 2 ? launch_some<2, 4>(xs, w, b1, wo, act, p.n_some, d, p.hs_some, row_stride, out, s)
                                 : launch_some<2, 2>(xs, w, b1, wo, act, p.n_some, d, p.hs_some, row_stride, out, s);
      if (rc != DODO_OK) return rc;
    }
    const int64_t thread_blocks = (p.n_big + p.n_small + kCombineThreads - 1) / kCombineThreads;
    const int64_t blocks = thread_blocks + (p.n_some + kCombineThreads / kWave - 1) / (kCombineThreads / kWave);
    hipLaunchKernelGGL(score_mlp_combine_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kCombineThreads), 0, s, partial, p.hs_big,
                       p.n_big, p.hs_small, p.n_small, p.hs_some, p.n_some, static_cast<int>(thread_blocks), b2, scores);
    return launch_status();
  }
  // plain kernel: as many token rows per workgroup as fit in 128 KiB of LDS (at most 8)
  const int64_t row_bytes = static_cast<int64_t>(d) * 4;
  int tok = static_cast<int>(128 * 1024 / row_bytes);
  if (tok < 1) return DODO_ERR_UNSUPPORTED;  // d > 32768
  if (tok > 8) tok = 8;
  const size_t lds = static_cast<size_t>(tok) * d * 4 + (kPlainThreads / kWave) * tok * 4;
  const int64_t blocks = (N + tok - 1) / tok;
  if (blocks > 0x7fffffffLL) return DODO_ERR_UNSUPPORTED;
  if (dtype == DODO_DTYPE_BF16) {
    {
      const int rc_lds = allow_dynamic_lds(reinterpret_cast<const void*>(score_mlp_plain_kernel<DODO_DTYPE_BF16>), static_cast<int>(lds));
      if (rc_lds != DODO_OK) return rc_lds;
    }
    hipLaunchKernelGGL(score_mlp_plain_kernel<DODO_DTYPE_BF16>, dim3(static_cast<unsigned>(blocks)), dim3(kPlainThreads),
                       lds, s, hidden, W1, b1, w2, b2, act, N, d, d_hid, row_stride, tok, scores);
  } else {
    {
      const int rc_lds = allow_dynamic_lds(reinterpret_cast<const void*>(score_mlp_plain_kernel<DODO_DTYPE_F32>), static_cast<int>(lds));
      if (rc_lds != DODO_OK) return rc_lds;
    }
    hipLaunchKernelGGL(score_mlp_plain_kernel<DODO_DTYPE_F32>, dim3(static_cast<unsigned>(blocks)), dim3(kPlainThreads),
                       lds, s, hidden, W1, b1, w2, b2, act, N, d, d_hid, row_stride, tok, scores);
  }
  return launch_status();
}
