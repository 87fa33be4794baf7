// GEMM over the recomputed rows with fused epilogues, for up to a few thousand rows: the
// projections of a vision block, of a decoder layer with few rows and of the patch merger.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "gemm_dev.h"

namespace fc {
namespace {

// RoPE position of rotary frequency pair k for the token at sequence position seqpos
// (its index in the current step's prompt, which also decides causality).  1-D RoPE:
// seqpos itself.  Multimodal RoPE (Qwen2.5-VL): pairs [0, s1) rotate by the temporal,
// [s1, s2) by the row and [s2, hd/2) by the column position; a text token has all three
// equal to its index, the token (I, J) of the frame with logical index l has
// (st, st + I, st + J) with st = T + l span, span = max(grid rows, grid columns), each
// frame taking span positions after the one before it.
// Text after the frames continues from the last frame's span: its three positions are
// T + W span + (its index past the frames).
struct MRope {
  int on, T, N, W, gw, span, s1, s2;
};
__device__ __forceinline__ int rope_pos(const MRope &m, int seqpos, int k) {
  if (!m.on || seqpos < m.T) return seqpos;
  if (seqpos >= m.T + m.W * m.N) return seqpos - m.W * m.N + m.W * m.span;
  const int r = seqpos - m.T, l = r / m.N, tok = r - l * m.N;
  const int st = m.T + l * m.span;
  if (k < m.s1) return st;
  const int I = tok / m.gw;
  return k < m.s2 ? st + I : st + (tok - I * m.gw);
}

// Patch geometry of a vision block's rows.
struct VitGeo {
  int N, m, mm, Np, gh, gw, d, H, hd, win;
};

// slot j of an item -> patch row (idx: the item's token ids)
__device__ __forceinline__ int slot_patch(const int32_t *idx, const VitGeo &g, int b, int j) {
  const int t = min(max(idx[(long)b * g.N + j / g.mm], 0), g.N - 1);
  return t * g.mm + j % g.mm;
}
__device__ __forceinline__ void patch_pos(const VitGeo &g, int p, int &pr, int &pc) {
  const int t = p / g.mm, sub = p - t * g.mm;
  pr = (t / g.gw) * g.m + sub / g.m;
  pc = (t % g.gw) * g.m + sub % g.m;
}
__device__ __forceinline__ float4 bf4(const uint16_t *p) {
  const uint2 u = *reinterpret_cast<const uint2 *>(p);
  return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u),
                     __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xFFFF0000u));
}
__device__ __forceinline__ void st_bf4(uint16_t *p, float a, float b, float c, float d) {
  *reinterpret_cast<uint2 *>(p) = make_uint2(f2bf(a) | ((uint32_t)f2bf(b) << 16),
                                             f2bf(c) | ((uint32_t)f2bf(d) << 16));
}
// Rotary pair (a, b) turned by (cos, sin) = cs, with the same two roundings wherever it is done:
// a cached key and one just written then have the same rotated bits.
__device__ __forceinline__ float2 rot_pair(float a, float b, float2 cs) {
  return make_float2(fmaf(a, cs.x, -(b * cs.y)), fmaf(b, cs.x, a * cs.y));
}
__device__ __forceinline__ float gelu_erf(float v) {
  return 0.5f * v * (1.f + erff(v * 0.70710678118654752f));
}

// ------------------------------------------------------------------------------ GEMMs
// C[rows][cols] = A[rows][K] W[cols][K]^T over the recomputed rows packed across items, with
// the epilogue of a vision block's, a decoder layer's or the merger's projection: one workgroup
// per TM x TN tile (TN staged weight rows), the whole K range, no partial sums.  A projection
// of a frame has a few hundred to a few thousand rows, so what bounds a tile is the load path
// of its CU (TM + TN rows of 128 B a K step), not its MFMAs: the tile is chosen on the device,
// where the row count is known, as the one whose CUs load least (row_tile).
//   * NST stages of (TM + TN) rows rotate in LDS, 64 K values (a 128-B line) a row, 16-B
//     chunks XOR-swizzled by (row >> 1) & 7.  Waves 4-7 only issue the DMAs (a DMA holds its
//     wave at issue): after barrier k those of step k + NST - 1, into the stage of step k - 1.
//     Waves 0-3 multiply, a quarter of the tile each, and read the fragments of the next half
//     step while they multiply this one, across the barrier too.  (All eight waves loading and
//     multiplying, with or without the halves of the workgroup in alternating phases, was up
//     to 30 % slower: the DMAs keep the MFMAs waiting.)
//   * The accumulators go through LDS as whole rows, so that every global access of the
//     epilogue is a piece of a row: the QKV modes (L_QKV: times 1/rms) add the bias, rotate q
//     and scatter raw k and v into the cache; the O modes add the residual (V_O: and the bias) and write h1, the MLP
//     operand bf16(h1 g2) and the row's sums of squares per 64 columns; V_GU applies 1/rms,
//     adds the biases and writes SiLU(g) u; the DOWN modes add h1 (V_DOWN: and the bias) and
//     scatter the output rows; M_GELU adds the bias and writes GELU; M_OUT adds the bias and
//     scatters the output rows.
//   * A QKV mode stages a column beside its rotary partner half a head away (V_GU: a gate beside
//     its up row): staged rows [0, TN / 2) are columns, [TN / 2, TN) their partners.
//   * M tiles of one column tile are consecutive, so each XCD reads its own share of the
//     weights once.
// Measured on the Qwen2.5-VL block (d 1280, MLP 3456), us, against 256 x 256 tiles in up to 8
// K-range parts with a reduction kernel each: QKV 23 + 15 -> 18.5, O 15 + 9 -> 14, gate/up
// 28 + 14 -> 28, down 21 + 9 -> 21 at 1024 rows; the whole windowed block 154 -> 92 at 1024
// rows, 136 -> 81 at 645 and 88 -> 55 at 104 rows (there against the weight-streaming GEMM
// and its reductions).  The DMA pattern alone takes 7.3 us for QKV (37 B a clock and CU); LDS
// traffic (operands written once and read twice), about 3 us before the first step is staged
// and 2 us of epilogue make up the rest.  Decoder layer (d 3584, 162 rows), against the
// weight-streaming GEMM with its K parts and their reductions: QKV 24 + 10 -> 20 (and 5 for
// the rows' norm, which that GEMM did itself), O 23 + 7 -> 20; the toy layer (d 256) 59 -> 40
// in all.  Where K is long and the rows few the weight-streaming GEMM is faster: row_streams.
enum { V_QKV, V_O, V_GU, V_DOWN, L_QKV, L_O, L_DOWN, M_GELU, M_OUT };
constexpr int kRowLds = 150 * 1024;
constexpr int kRowSsqCols = 64;         // columns per partial sum of squares of h1

struct RowGemm {
  const uint16_t *A, *W, *bias;
  int K, cols;                          // cols: weight rows staged in all (V_GU: 2 f)
  int B, cus;
  const int32_t *idx;                   // token ids (null: every token in order)
  // geometry; a decoder layer's or the merger's rows are its tokens: N = Np = slots per item
  // and m = mm = 1 there, d the output width, hd the head dim
  VitGeo g;
  const float2 *rope;                   // V_QKV: [position][32]; L_QKV: [position][hd / 2]
  int qw, kw;                           // QKV: columns of q and of k (and v)
  uint16_t *q, *kc, *vc, *krot;         // QKV (krot: V_QKV)
  const int32_t *smap;                  // L_QKV: slot map of the cache rows
  const float *rinv;                    // L_QKV: 1/rms of each slot's row
  int S, cur_row0, qpos0;               // L_QKV: cache rows, the region's first row and position
  MRope mr;                             // L_QKV
  const uint16_t *x, *g2;               // O
  float *h1, *ssq;                      // O (V_GU reads ssq, DOWN h1)
  uint16_t *hb;                         // O
  uint16_t *act;                        // V_GU, M_GELU
  uint16_t *y;                          // DOWN, M_OUT
  int parts;                            // sums of squares per row
  float eps;
};

// Streams of the weights (one per 256 recomputed rows of an item, and one for the rest) from
// which a projection over K is faster here than in the weight-streaming GEMM, which deals K over
// the chip and reduces its partial sums.  Measured with weights from memory, 3584 columns, a
// whole layer, here / there in us:
//   1 stream, 162 / 256 rows: K 4096 129 / 136, 156 / 165; K 4864 133 / 139, 162 / 168; K 6144
//     140 / 139, 170 / 171; K 9728 155 / 137, 187 / 176; K 18944 200 / 162, 237 / 191; 26 rows:
//     K 2048 94 / 95, K 4864 105 / 98, K 6144 110 / 99
//   2 streams, one item of 300 / 512 rows: K 7168 235 / 239, 282 / 297; K 9728 257 / 243,
//     304 / 310; K 18944 341 / 291, 381 / 348; two items of 162: K 7168 224 / 232, K 9728 242 / 240
//   3 streams, one item of 600 / three of 162 rows: K 9728 373 / 390, 320 / 335; K 12288
//     407 / 405, 348 / 354; K 18944 482 / 459, 415 / 409; one item of 655: K 18944 471 / 481
//   4 streams, one item of 1024 / four of 162 rows: K 18944 630 / 660, 494 / 527
// and the merger (K 5120 twice): 26 / 128 / 256 rows 55 / 39, 57 / 54, 75 / 68; two items of 162
// 78 / 96; one of 400 86 / 103.
constexpr int row_streams(int K) { return K < 5120 ? 1 : K < 9216 ? 2 : 3; }
// Which of the two a call takes.  Every item has at least one recomputed row as a rule, so the
// number of items decides alone where it reaches row_streams (an item without rows then costs
// time, not its result).  Where the slots could hold that many streams but the items need not,
// the rows decide, on the device, which costs a launch some 0.7 us, and an empty reduction where
// the row tiles are taken (nrec null: every slot is a row).
enum Route { kStream, kRowTiles, kOnDevice };
inline Route row_route(int K, int B, int N, const int32_t *nrec) {
  const int need = row_streams(K);
  if (B >= need) return kRowTiles;
  if (B * ((N + 255L) / 256) < need) return kStream;
  return nrec ? kOnDevice : kRowTiles;
}
__device__ __forceinline__ int weight_streams(const int32_t *nrec, int B, int N) {
  int n = 0;
  for (int b = 0; b < B; ++b) n += (n_valid(nrec, b, N) + 255) >> 8;
  return n;
}

struct RowTile {
  int v, tiles;                         // variant, tiles of all rows
};
constexpr int kRowTM[4] = {128, 64, 64, 32}, kRowTN[4] = {128, 128, 64, 64};
constexpr int kRowGuTM[4] = {128, 128, 64, 32}, kRowGuTN[4] = {256, 128, 128, 64};
// The tile for `rows` rows: least rows loaded per CU, (TM + TN) times the rounds of one
// workgroup per CU (a K step of a 64 x 64 tile takes 0.2 us, of a 128 x 128 tile 0.5 us).  Host
// and device take the same decision.
__host__ __device__ inline RowTile row_tile(bool gu, int rows, int cols, int cus) {
  RowTile best{0, 0};
  int least = 0;
  for (int v = 0; v < 4; ++v) {
    const int tm = gu ? kRowGuTM[v] : kRowTM[v], tn = gu ? kRowGuTN[v] : kRowTN[v];
    const int tiles = ((rows + tm - 1) / tm) * ((cols + tn - 1) / tn);
    const int cost = (tiles + cus - 1) / cus * (tm + tn);
    if (v == 0 || cost < least) {
      best = RowTile{v, tiles};
      least = cost;
    }
  }
  return best;
}

__device__ __forceinline__ long row_slot(const int *pre, int B, int N, int p, int &b) {
  if (B > 1) return packed_slot(pre, B, N, p, b);
  b = 0;
  return p;
}

template <int MODE, int TM, int TN>
__device__ __forceinline__ void row_gemm_tile(const RowGemm &a, unsigned char *lds, const int *pre,
                                              int *rslot, int *rpatch, int *rpos, float *rinv,
                                              int row0, int nvalid, int nt) {
  constexpr int STAGE = (TM + TN) * RB;
  constexpr int NST = kRowLds / STAGE > 8 ? 8 : kRowLds / STAGE;
  constexpr int NI = (TM + TN) / 8;               // DMA instructions per step
  constexpr int L = NI / 4;                       // of each loader wave
  constexpr int MBW = TM / 32, NBW = TN / 32;     // 16-row blocks of a wave's quarter
  constexpr bool QKV = MODE == V_QKV || MODE == L_QKV, PAIR = QKV || MODE == V_GU;
  constexpr bool O = MODE == V_O || MODE == L_O, DOWN = MODE == V_DOWN || MODE == L_DOWN;
  constexpr bool BIAS = MODE != L_O && MODE != L_DOWN;
  static_assert(NST >= 3 && NI % 4 == 0 && (NST - 1) * L < 64, "stages");
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const VitGeo &g = a.g;
  const int nk = a.K / KS;
  // column of staged row r (clamped: past the last column nothing is stored)
  auto column = [&](int r) {
    if (QKV) {
      const int half = g.hd / 2, p = min(nt * (TN / 2) + r % (TN / 2), a.cols / 2 - 1);
      const int h = p / half;
      return h * g.hd + (p - h * half) + (r >= TN / 2 ? half : 0);
    }
    if (MODE == V_GU)
      return min(nt * (TN / 2) + r % (TN / 2), a.cols / 2 - 1) + (r >= TN / 2 ? a.cols / 2 : 0);
    return min(nt * TN + r, a.cols - 1);
  };
  constexpr int TP = TN + 4;                      // floats per row of the epilogue tile
  static_assert(TM * TP * 4 <= kRowLds, "the tile fits");
  float *T = reinterpret_cast<float *>(lds);
  if (w >= 4) {
    // ------------------------------------------------------------------ loader waves
    const uint16_t *gp[L];
    const int rsub = lane >> 3, ch = lane & 7;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const int r = (w - 4 + 4 * i) * 8 + rsub;   // row of the stage
      const int cs = (ch ^ swz8(r)) * 8;
      if (r < TM) {
        int ib;
        gp[i] = a.A + row_slot(pre, a.B, g.Np, row0 + min(r, nvalid - 1), ib) * a.K + cs;
      } else {
        gp[i] = a.W + (long)column(r - TM) * a.K + cs;
      }
    }
    const uint32_t lbase = lds_addr(lds) + (w - 4) * 1024;
    auto issue = [&](int k) {
      const uint32_t st = lbase + (k % NST) * STAGE;
#pragma unroll
      for (int i = 0; i < L; ++i) dma16(gp[i] + k * KS, st + i * 4096);
    };
    loads_done();
    for (int k = 0; k < NST - 1 && k < nk; ++k) issue(k);
    for (int k = 0; k < nk; ++k) {
      if (k + NST - 1 <= nk) wait_vm<(NST - 2) * L>();     // this wave's share of step k
      else wait_vm_rt((nk - 1 - k) * L);
      lds_barrier();                                       // barrier k: step k staged, k - 1 read
      if (k + NST - 1 < nk) issue(k + NST - 1);
    }
    lds_barrier();                                         // barrier nk: the stages are free
  } else {
    // -------------------------------------------------------------------- MFMA waves
    // the tile's rows: slot, patch row (b Np + patch) and 1/rms of x (L_QKV) or h1 (V_GU)
    if (t < TM) {
      int b = 0;
      const long sl = row_slot(pre, a.B, g.Np, row0 + min(t, nvalid - 1), b);
      rslot[t] = (int)sl;
      if (MODE <= V_DOWN && MODE != V_GU) {
        const int p = slot_patch(a.idx, g, b, (int)(sl - (long)b * g.Np));
        rpatch[t] = b * g.Np + p;
        if (MODE == V_QKV) {
          int pr, pc;
          patch_pos(g, p, pr, pc);
          rpos[t] = pr << 16 | pc;
        }
      }
      if (MODE > V_DOWN && MODE != M_GELU) {
        const int tok = tok_of(a.idx, sl, g.N);
        if (MODE == L_QKV) {
          rpatch[t] = b * a.S + pool_row(a.smap, b, a.S, a.cur_row0 + tok);   // cache row
          rpos[t] = a.qpos0 + tok;
          rinv[t] = a.rinv[sl];
        } else {
          rpatch[t] = b * g.N + tok;
        }
      }
      if (MODE == V_GU) {
        float v = 0.f;
        for (int c = 0; c < a.parts; ++c) v += a.ssq[sl * a.parts + c];
        rinv[t] = 1.f / sqrtf(v / (float)g.d + a.eps);
      }
    }
    f32x4 acc[MBW][NBW];
#pragma unroll
    for (int i = 0; i < MBW; ++i)
#pragma unroll
      for (int j = 0; j < NBW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int l16 = lane & 15, gq = lane >> 4, wm = w & 1, wn = w >> 1;
    const int sw = swz8(l16);
    const uint32_t aoff = (uint32_t)((wm * (TM / 2) + l16) * RB);
    const uint32_t boff = (uint32_t)((TM + wn * (TN / 2) + l16) * RB);
    auto rd = [&](int k, int s, bf16x8 (&fa)[MBW], bf16x8 (&fb)[NBW]) __attribute__((always_inline)) {
      const unsigned char *st = lds + (k % NST) * STAGE + (((4 * s + gq) ^ sw) << 4);
#pragma unroll
      for (int i = 0; i < MBW; ++i) fa[i] = *reinterpret_cast<const bf16x8 *>(st + aoff + i * 16 * RB);
#pragma unroll
      for (int j = 0; j < NBW; ++j) fb[j] = *reinterpret_cast<const bf16x8 *>(st + boff + j * 16 * RB);
    };
    auto mul = [&](const bf16x8 (&fa)[MBW], const bf16x8 (&fb)[NBW]) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < MBW; ++i)
#pragma unroll
        for (int j = 0; j < NBW; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    };
    // the fragments of the next half step are read while this one's are multiplied, across
    // the barrier too
    bf16x8 fa0[MBW], fb0[NBW], fa1[MBW], fb1[NBW];
    lds_barrier();                                         // barrier 0
    rd(0, 0, fa0, fb0);
    for (int k = 0; k < nk; ++k) {
      rd(k, 1, fa1, fb1);
      mul(fa0, fb0);
      lds_barrier();                                       // barrier k + 1
      if (k + 1 < nk) rd(k + 1, 0, fa0, fb0);
      mul(fa1, fb1);
    }
    // lane holds column l16 and rows 4 gq + e of each 16-row block
#pragma unroll
    for (int i = 0; i < MBW; ++i)
#pragma unroll
      for (int j = 0; j < NBW; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          T[(wm * (TM / 2) + i * 16 + 4 * gq + e) * TP + wn * (TN / 2) + j * 16 + l16] = acc[i][j][e];
  }
  lds_barrier();
  // A thread has 4 columns (PAIR: and their 4 partners) of every (512 / QPR)-th row, so what
  // depends on the columns is found once, and a turn's loads go out for all rows first.
  constexpr int QPR = (PAIR ? TN / 2 : TN) / 4, RSTEP = 512 / QPR, IT = (TM + RSTEP - 1) / RSTEP;
  static_assert(512 % QPR == 0, "fixed columns");
  const int r0 = t / QPR, c4 = (t % QPR) * 4;
  if (PAIR) {
    const int p = nt * (TN / 2) + c4;
    if (p >= a.cols / 2) return;
    const int c0 = column(c4), c1 = column(TN / 2 + c4);
    const float4 b0 = bf4(a.bias + c0), b1 = bf4(a.bias + c1);
    const float bb0[4] = {b0.x, b0.y, b0.z, b0.w}, bb1[4] = {b1.x, b1.y, b1.z, b1.w};
    const bool isq = c0 < a.qw;
    const bool rot = QKV && (isq || (MODE == V_QKV && a.krot && c0 < a.qw + a.kw));
    // rotary pairs c0 % hd .. + 3, of one frequency section (the sections of M-RoPE are multiples
    // of 8; a vision head's first quarter turns by the patch row, the second by its column, and
    // a quarter is a multiple of 4)
    const int quarter = g.hd / 4, pair = QKV ? c0 % g.hd : 0;
    float2 cs[IT][4];
    if (rot) {
#pragma unroll
      for (int n = 0; n < IT; ++n) {
        const int pos = rpos[min(r0 + n * RSTEP, TM - 1)];
        const float2 *rp = MODE == V_QKV
                               ? a.rope + (pair < quarter ? (pos >> 16) * 32 + pair
                                                          : (pos & 0xFFFF) * 32 + pair - quarter)
                               : a.rope + (long)rope_pos(a.mr, pos, pair) * (g.hd / 2) + pair;
#pragma unroll
        for (int i = 0; i < 4; ++i) cs[n][i] = rp[i];
      }
    }
    uint16_t *kv = c0 < a.qw + a.kw ? a.kc - a.qw : a.vc - a.qw - a.kw;
#pragma unroll
    for (int n = 0; n < IT; ++n) {
      const int r = r0 + n * RSTEP;
      if (r >= nvalid) break;
      const float4 v = *reinterpret_cast<const float4 *>(T + r * TP + c4);
      const float4 u = *reinterpret_cast<const float4 *>(T + r * TP + TN / 2 + c4);
      const float v4[4] = {v.x, v.y, v.z, v.w}, u4[4] = {u.x, u.y, u.z, u.w};
      float x0[4], x1[4];
      if (MODE == V_GU) {
        const float inv = rinv[r];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float gv = v4[i] * inv + bb0[i], uv = u4[i] * inv + bb1[i];
          // expf and a division: __expf (some 80 ulp off at -80) and v_rcp_f32 would save 2 of a
          // block's 81 us
          x0[i] = gv / (1.f + expf(-gv)) * uv;
        }
        st_bf4(a.act + (long)rslot[r] * (a.cols / 2) + p, x0[0], x0[1], x0[2], x0[3]);
      } else {
        // raw keys and values go to the cache, rotated queries and keys to the attention
        float y0[4], y1[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          x0[i] = MODE == L_QKV ? fmaf(v4[i], rinv[r], bb0[i]) : v4[i] + bb0[i];
          x1[i] = MODE == L_QKV ? fmaf(u4[i], rinv[r], bb1[i]) : u4[i] + bb1[i];
          if (rot) {
            // a key is rotated as the cache holds it, rounded: the step that computes it and
            // those that reuse it attend to the same bits
            const float2 y = isq ? rot_pair(x0[i], x1[i], cs[n][i])
                                 : rot_pair(bf2f(f2bf(x0[i])), bf2f(f2bf(x1[i])), cs[n][i]);
            y0[i] = y.x;
            y1[i] = y.y;
          }
        }
        if (!isq) {
          uint16_t *dst = kv + (long)rpatch[r] * a.kw;
          st_bf4(dst + c0, x0[0], x0[1], x0[2], x0[3]);
          st_bf4(dst + c1, x1[0], x1[1], x1[2], x1[3]);
        }
        if (rot) {
          uint16_t *dst = isq ? a.q + (long)rslot[r] * a.qw : a.krot - a.qw + (long)rpatch[r] * a.kw;
          st_bf4(dst + c0, y0[0], y0[1], y0[2], y0[3]);
          st_bf4(dst + c1, y1[0], y1[1], y1[2], y1[3]);
        }
      }
    }
  } else {
    const int c = nt * TN + c4;
    const bool cv = c < a.cols;
    const int cc = cv ? c : 0;
    const float4 bb = BIAS ? bf4(a.bias + cc) : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 gn = O ? bf4(a.g2 + cc) : make_float4(0.f, 0.f, 0.f, 0.f);
    uint2 xr[O ? IT : 1];
    float4 hr[DOWN ? IT : 1];
#pragma unroll
    for (int n = 0; n < IT; ++n) {
      const int r = min(r0 + n * RSTEP, nvalid - 1);
      if (O) xr[n] = *reinterpret_cast<const uint2 *>(a.x + (long)rpatch[r] * g.d + cc);
      if (DOWN) hr[n] = *reinterpret_cast<const float4 *>(a.h1 + (long)rslot[r] * g.d + cc);
    }
#pragma unroll
    for (int n = 0; n < IT; ++n) {
      const int r = r0 + n * RSTEP;
      const bool rv = r < nvalid;
      float ss = 0.f;
      if (rv && cv) {
        const long slot = rslot[r];
        const float4 v = *reinterpret_cast<const float4 *>(T + r * TP + c4);
        if (O) {
          const float4 xv = unpack_bf16x4(xr[n]);
          const float4 h = make_float4(xv.x + (v.x + bb.x), xv.y + (v.y + bb.y), xv.z + (v.z + bb.z),
                                       xv.w + (v.w + bb.w));
          *reinterpret_cast<float4 *>(a.h1 + slot * g.d + c) = h;
          st_bf4(a.hb + slot * g.d + c, h.x * gn.x, h.y * gn.y, h.z * gn.z, h.w * gn.w);
          ss = h.x * h.x + h.y * h.y + h.z * h.z + h.w * h.w;
        } else if (DOWN) {
          const float4 h = hr[n];
          st_bf4(a.y + (long)rpatch[r] * g.d + c, h.x + (v.x + bb.x), h.y + (v.y + bb.y),
                 h.z + (v.z + bb.z), h.w + (v.w + bb.w));
        } else if (MODE == M_GELU) {
          st_bf4(a.act + slot * g.d + c, gelu_erf(bb.x + v.x), gelu_erf(bb.y + v.y),
                 gelu_erf(bb.z + v.z), gelu_erf(bb.w + v.w));
        } else {
          st_bf4(a.y + (long)rpatch[r] * g.d + c, bb.x + v.x, bb.y + v.y, bb.z + v.z, bb.w + v.w);
        }
      }
      if (O) {
        // 64 columns of a row are 16 consecutive lanes
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
        if (rv && cv && (lane & 15) == 0) a.ssq[(long)rslot[r] * a.parts + c / kRowSsqCols] = ss;
      }
    }
  }
}

// What a workgroup knows of its tile's rows, beside the stages in LDS.
struct RowLds {
  int pre[kMMaxItems + 4];
  int slot[128], patch[128], pos[128];
  float inv[128];
};

template <int MODE>
__device__ __forceinline__ void row_gemm(const RowGemm &a, const int32_t *rows, unsigned char *lds,
                                         RowLds &s) {
  int M;
  if (a.B == 1) {                                // one item: its rows are the packed rows
    M = n_valid(rows, 0, a.g.Np);
  } else {
    if (threadIdx.x < 64) row_prefix(rows, a.B, a.g.Np, s.pre);
    __syncthreads();
    M = s.pre[a.B];
  }
  const RowTile vt = row_tile(MODE == V_GU, M, a.cols, a.cus);
  if ((int)blockIdx.x >= vt.tiles) return;
  const int tm = MODE == V_GU ? kRowGuTM[vt.v] : kRowTM[vt.v];
  const int mt = (M + tm - 1) / tm;
  const int l = xcd_tile(blockIdx.x, vt.tiles), nt = l / mt, row0 = (l - nt * mt) * tm;
  const int nvalid = min(tm, M - row0);
#define FC_VT(i)                                                                               \
  row_gemm_tile<MODE, MODE == V_GU ? kRowGuTM[i] : kRowTM[i], MODE == V_GU ? kRowGuTN[i] : kRowTN[i]>( \
      a, lds, s.pre, s.slot, s.patch, s.pos, s.inv, row0, nvalid, nt)
  switch (vt.v) {
    case 0: FC_VT(0); break;
    case 1: FC_VT(1); break;
    case 2: FC_VT(2); break;
    default: FC_VT(3); break;
  }
#undef FC_VT
}

template <int MODE>
__global__ __launch_bounds__(512) void k_row_gemm(RowGemm a, const int32_t *__restrict__ rows) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[kRowLds];
  __shared__ RowLds s;
  row_gemm<MODE>(a, rows, lds, s);
}

// The most tiles any row count up to `rows` takes (the grid; surplus workgroups exit).
int row_grid(bool gu, int rows, int cols, int cus) {
  int most = 1;
  for (int r = 1; r <= rows; r += 32)
    most = std::max(most, row_tile(gu, std::min(r + 31, rows), cols, cus).tiles);
  return most;
}

template <int MODE>
fc_status run_row_gemm(fc_ctx *ctx, hipStream_t st, const char *name, const RowGemm &a,
                       const int32_t *rows) {
  const int grid = row_grid(MODE == V_GU, a.B * a.g.Np, a.cols, a.cus);
  ProfScope ps(ctx, st, name);
  hipLaunchKernelGGL(k_row_gemm<MODE>, dim3((unsigned)grid), dim3(512), 0, st, a,
                     rows);
  FC_LAUNCH_OK(st, "k_row_gemm");
  return FC_OK;
}

}  // namespace
}  // namespace fc
