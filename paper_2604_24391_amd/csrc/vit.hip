// Vision-encoder side of the partial recompute on gfx950: one Qwen2.5-VL-style vision
// block over the patches of the recomputed merged tokens (Sec. 4.1: a token that is not
// reused goes through the vision encoder again), with the reused patches' keys and values
// taken from the encoder's per-layer cache.
//
// Rows: the recomputed patches of item b are slots b Np + j, j < n_recompute[b] m^2,
// slot j being patch sub-position j mod m^2 of merged token recompute_idx[j / m^2]
// (patch rows token-major).  Kernels per call:
//
//   k_vit_gather_norm  one workgroup per slot: the patch row of x, RMSNorm (g1) as the
//                      bf16 operand of the QKV GEMM; the item's row count; the rotary table;
//                      the cached keys rotated, where a window has more than 64 keys.
//   k_row_gemm<V_QKV>  + bias; q rotated at the patch position (bf16, compact), raw k and v
//                      into the cache at the patch row.
//   k_vit_attn         one workgroup per (window, query chunk, head) or, with full
//                      attention, per (query chunk, head): the chunk's queries against the
//                      window's (the frame's) keys in blocks, S^T = K Q^T and O^T = V^T P^T
//                      on bf16 MFMAs, online softmax in fp32.
//   k_row_gemm<V_O>    + bias + residual -> h1 (fp32), bf16(h1 g2) and the row's sums of
//                      squares by 64 columns.
//   k_row_gemm<V_GU>   times 1/rms(h1), + biases, SiLU(g) u -> bf16.
//   k_row_gemm<V_DOWN> + bias + h1 -> the slot's output row of y (bf16).
//
// The 2-D rotary angle of dim pair i (i < hd/2) of a patch at (row, col) is
// row * f_i for i < hd/4 and col * f_(i - hd/4) otherwise, f_k = theta^(-2k / (hd/2));
// cos and sin are formed in fp64 and rounded to fp32, once per call, into a table by
// position and frequency (filled by the gather kernel's first workgroups).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "fc_internal.h"
#include "gemm_dev.h"
#include "rowgemm.h"

namespace fc {
namespace {

constexpr int kVitThreads = 256;
constexpr int kVitQ = 64;            // queries per attention workgroup

__device__ __forceinline__ int n_rows(const int32_t *nrec, const VitGeo &g, int b) {
  return min(max(nrec[b], 0), g.N) * g.mm;
}
__device__ float block_sum(float v, float *red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float s = 0.f;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += red[i];
  __syncthreads();
  return s;
}

// Sum over the splits of the float4 at p0 + sp stride, in split order, loads issued in
// groups of up to 4 (a group past the last split is skipped; `splits` is uniform).
template <int SPL>
__device__ __forceinline__ float4 sum_splits4(const float *__restrict__ p0, long stride, int splits) {
  constexpr int G = SPL < 4 ? SPL : 4;
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int g0 = 0; g0 < SPL; g0 += G) {
    if (g0 > 0 && g0 >= splits) break;
    float4 u[G];
#pragma unroll
    for (int i = 0; i < G; ++i)
      u[i] = *reinterpret_cast<const float4 *>(p0 + (long)min(g0 + i, splits - 1) * stride);
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const bool in = g0 + i < splits;
      a.x += in ? u[i].x : 0.f;
      a.y += in ? u[i].y : 0.f;
      a.z += in ? u[i].z : 0.f;
      a.w += in ? u[i].w : 0.f;
    }
  }
  return a;
}
// Split-K sums of columns c .. c + 3 of row s (partials [split][rows][nc]).
template <int SPL>
__device__ __forceinline__ float4 sum_parts4(const float *__restrict__ part, int splits, long rows,
                                             long s, int nc, int c) {
  return sum_splits4<SPL>(part + s * nc + c, rows * nc, splits);
}
__device__ __forceinline__ void ld_bf8(const uint16_t *p, float *v) {
  const uint4 u = *reinterpret_cast<const uint4 *>(p);
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
  }
}
__device__ __forceinline__ void st_bf8(uint16_t *p, const float *v) {
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = f2bf(v[2 * i]) | ((uint32_t)f2bf(v[2 * i + 1]) << 16);
  *reinterpret_cast<uint4 *>(p) = make_uint4(w[0], w[1], w[2], w[3]);
}

// RMSNorm of one bf16 row of d <= 2048 (a multiple of 8) times a gain, by a whole
// workgroup in one pass: thread t holds columns 8 t .. 8 t + 7.
__device__ __forceinline__ void norm_row(const uint16_t *xr, const uint16_t *gain, int d, float eps,
                                         uint16_t *dst, float *red) {
  const int c = 8 * threadIdx.x;
  float v[8];
  float ss = 0.f;
  if (c < d) {
    ld_bf8(xr + c, v);
#pragma unroll
    for (int i = 0; i < 8; ++i) ss = fmaf(v[i], v[i], ss);
  }
  const float inv = 1.f / sqrtf(block_sum(ss, red) / (float)d + eps);
  if (c < d) {
    float gn[8];
    ld_bf8(gain + c, gn);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = v[i] * inv * gn[i];
    st_bf8(dst + c, v);
  }
}

// --------------------------------------------------------------------- gather + norm
// One workgroup per slot: the patch row of x, RMSNorm (g1) as the bf16 GEMM operand; the
// item's row count; and, with krot, the cached key row of patch s rotated at its position (rows
// that are recomputed are written again by the QKV epilogue).  Angles: position ps times
// frequency theta^(-2 fk / (hd / 2)), formed in fp64, cos and sin rounded to fp32; the first
// workgroups also leave them as a table at [ps][fk] for the kernels that follow.
__global__ __launch_bounds__(kVitThreads) void k_vit_gather_norm(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ g1,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ nrec, VitGeo g, float eps,
    double theta, uint16_t *__restrict__ hb, int32_t *__restrict__ rows_out,
    float2 *__restrict__ rope, const uint16_t *__restrict__ kc, uint16_t *__restrict__ krot) {
  __shared__ float red[kVitThreads / 64];
  __shared__ float2 cs[64];
  const long s = blockIdx.x;
  const int t = threadIdx.x;
  const int b = (int)(s / g.Np), j = (int)(s - (long)b * g.Np);
  const int half = g.hd / 2, quarter = g.hd / 4;
  const long e = s * kVitThreads + t;      // past 2^31 for the last of many items' slots
  const int npos = max(g.gh, g.gw) * g.m;
  if (e < npos * 32) {
    const int ps = (int)e / 32, fk = (int)e - ps * 32;
    if (fk < quarter) {
      const double ang = (double)ps * pow(theta, -2.0 * fk / (double)half);
      rope[e] = make_float2((float)cos(ang), (float)sin(ang));
    }
  }
  if (krot) {
    // this patch's angles: pair i < quarter by its row, the others by its column
    int pr, pc;
    patch_pos(g, j, pr, pc);
    if (t < half) {
      const int fk = t < quarter ? t : t - quarter;
      const double ang = (double)(t < quarter ? pr : pc) * pow(theta, -2.0 * fk / (double)half);
      cs[t] = make_float2((float)cos(ang), (float)sin(ang));
    }
    __syncthreads();
    const uint16_t *kr = kc + s * g.d;
    for (int p = 4 * t; p < g.d / 2; p += 4 * kVitThreads) {   // 4 pairs of one head
      const int h = p / half, c = h * g.hd + (p - h * half);
      const float4 x0 = bf4(kr + c), x1 = bf4(kr + c + half);
      const float2 *w = cs + (p - h * half);
      const float2 y0 = rot_pair(x0.x, x1.x, w[0]), y1 = rot_pair(x0.y, x1.y, w[1]),
                   y2 = rot_pair(x0.z, x1.z, w[2]), y3 = rot_pair(x0.w, x1.w, w[3]);
      st_bf4(krot + s * g.d + c, y0.x, y1.x, y2.x, y3.x);
      st_bf4(krot + s * g.d + c + half, y0.y, y1.y, y2.y, y3.y);
    }
  }
  if (j == 0 && t == 0) rows_out[b] = n_rows(nrec, g, b);
  if (j >= n_rows(nrec, g, b)) return;
  norm_row(x + ((long)b * g.Np + slot_patch(idx, g, b, j)) * g.d, g1, g.d, eps, hb + s * g.d, red);
}

// ------------------------------------------------------------------------ attention
// Key k of a workgroup's key set: the window's patches (token-major within the window)
// or, with full attention, patch k of the frame.
__device__ __forceinline__ int key_patch(const VitGeo &g, int w, int k) {
  if (g.win <= 0) return k;
  const int wpr = (g.gw + g.win - 1) / g.win;
  const int wi = w / wpr, wj = w - wi * wpr;
  const int I0 = wi * g.win, J0 = wj * g.win;
  const int wcols = min(g.win, g.gw - J0);
  const int tk = k / g.mm, sub = k - tk * g.mm;
  const int I = I0 + tk / wcols, J = J0 + tk % wcols;
  return (I * g.gw + J) * g.mm + sub;
}
__device__ __forceinline__ int window_keys(const VitGeo &g, int w) {
  if (g.win <= 0) return g.Np;
  const int wpr = (g.gw + g.win - 1) / g.win;
  const int wi = w / wpr, wj = w - wi * wpr;
  return min(g.win, g.gh - wi * g.win) * min(g.win, g.gw - wj * g.win) * g.mm;
}
__device__ __forceinline__ int window_of(const VitGeo &g, int p) {
  if (g.win <= 0) return 0;
  const int t = p / g.mm;
  const int wpr = (g.gw + g.win - 1) / g.win;
  return (t / g.gw) / g.win * wpr + (t % g.gw) / g.win;
}

// The chunk-th group of up to 64 recomputed slots of window w (slot order), found by all
// threads in rounds of 256 slots with a ballot prefix count; returns how many there are.
__device__ int window_queries(const int32_t *idx, const VitGeo &g, int b, int w, int chunk,
                              int nrow, int *qslot, int *wcnt, int *nq_s) {
  const int t = threadIdx.x;
  const int lo = chunk * kVitQ, hi = lo + kVitQ;
  int seen = 0;
  for (int j0 = 0; j0 < nrow && seen < hi; j0 += blockDim.x) {
    const int j = j0 + t;
    const bool in = j < nrow && window_of(g, slot_patch(idx, g, b, j)) == w;
    const unsigned long long bal = __ballot(in);
    const int lane = t & 63, wv = t >> 6;
    if (lane == 0) wcnt[wv] = __popcll(bal);
    __syncthreads();
    int before = 0, total = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
      if (i < wv) before += wcnt[i];
      total += wcnt[i];
    }
    const int pos = seen + before + __popcll(bal & ((1ull << lane) - 1ull));
    if (in && pos >= lo && pos < hi) qslot[pos - lo] = j;
    seen += total;
    __syncthreads();
  }
  if (t == 0) *nq_s = min(max(seen - lo, 0), kVitQ);
  __syncthreads();
  return *nq_s;
}

// Grid: x = head, y = window * chunks_per_window + chunk, z = item (the chunks of one head,
// which read the same keys, share an XCD's L2).  64 queries a workgroup, eight waves: two groups
// of four, 16 queries a wave, both groups with all the queries and each with KPG keys of its own
// of every block of 2 KPG, merged at the end; a SIMD then has two independent chains of QK,
// softmax and PV.
//   * Keys are staged row-major, values as 8-B words of one dim of 4 keys (byte permutes of 4
//     rows).  The loads of the next block are in registers while a block is multiplied.
//   * KPG = 64 (more than 64 keys a window): the keys come rotated (k_vit_gather_norm rotates
//     the cached rows, the QKV epilogue the new ones), as every key is staged by all query
//     chunks of its window.  KPG = 32 (a window is one block, staged about once): raw keys are
//     rotated on their way to LDS; the pass over all cached keys costs more there.
//   * S^T = K Q^T with 16x16x32 bf16 MFMAs, so a lane's accumulators all belong to one query
//     (keys 4 (lane / 16) + e of each 16-key tile) and the online softmax needs two cross-lane
//     steps; P then feeds O^T = V^T P^T straight from the registers, the values being read
//     from LDS in the same key order.
// Full attention over 1024 patches (16 heads x 80): 65 -> 24.5 us (four waves, every chunk
// rotating all keys again and transposing the values by 2-B LDS writes); about 9 us of it are
// launch, first block and merge, and per block the loads and the multiplication overlap only
// partly.  More keys in flight or two query tiles a wave gained nothing.
template <int HDP, int KPG>
__global__ __launch_bounds__(512) void k_vit_attn(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ kr,
    const uint16_t *__restrict__ vc, const int32_t *__restrict__ idx,
    const int32_t *__restrict__ nrec, VitGeo g, const float2 *__restrict__ rope, int chunks,
    uint16_t *__restrict__ out) {
  constexpr bool ROT = KPG == 32;      // raw keys, rotated on load
  constexpr int KP = HDP + 8;          // key row pitch (bf16)
  constexpr int BK = 2 * KPG;          // keys per block
  constexpr int KT = (BK * (HDP / (ROT ? 16 : 8)) + 511) / 512, VT = ((BK / 4) * (HDP / 4) + 511) / 512;
  constexpr int kKs = BK * KP * 2, kVq = (BK / 4) * HDP * 8;
  __shared__ __attribute__((aligned(16))) unsigned char lds[2 * (kKs + kVq)];
  __shared__ int qslot[kVitQ];
  __shared__ int wcnt[8];
  __shared__ int nq_s;
  __shared__ float ml[2][kVitQ];
  auto Ks = [&](int buf) { return reinterpret_cast<uint16_t *>(lds + buf * kKs); };
  auto Vq = [&](int buf) { return reinterpret_cast<u32x2 *>(lds + 2 * kKs + buf * kVq); };
  const int h = blockIdx.x, b = blockIdx.z;
  const int w = blockIdx.y / chunks, chunk = blockIdx.y - w * chunks;
  const int t = threadIdx.x, lane = t & 63, l16 = lane & 15, gq = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int gr = wv >> 2;                                  // key group
  const int hd = g.hd;
  const int nrow = n_rows(nrec, g, b);
  const int nk = window_keys(g, w);
  const int nblk = (nk + BK - 1) / BK;
  const int half = hd / 2;
  // Staging tasks: 8 dims of a key (rotated on load: 8 dims and their partners half a head
  // away); values of 4 keys, 4 dims.  Keys past the last are read as the last: their
  // probability is 0.
  const int cpr = ROT ? hd / 16 : hd / 8, qpr = hd / 4;
  const uint16_t *kbase = kr + (long)b * g.Np * g.d + h * hd, *vbase = vc + (long)b * g.Np * g.d + h * hd;
  int ki[KT], kc0[KT], kg[VT], vc0[VT];
  uint32_t ko[KT], vo[VT];
#pragma unroll
  for (int i = 0; i < KT; ++i) {
    const int e = min(t + i * 512, BK * cpr - 1);
    ki[i] = e / cpr;
    kc0[i] = (e - ki[i] * cpr) * 8;
    ko[i] = (uint32_t)(ki[i] * g.d + kc0[i]) * 2;
  }
#pragma unroll
  for (int i = 0; i < VT; ++i) {
    const int e = min(t + i * 512, (BK / 4) * qpr - 1);
    kg[i] = e / qpr;
    vc0[i] = (e - kg[i] * qpr) * 4;
    vo[i] = (uint32_t)(4 * kg[i] * g.d + vc0[i]) * 2;
  }
  u32x4 rk[KT], rp[ROT ? KT : 1];
  u32x2 rv[VT][4];
  auto load_block = [&](int k0) __attribute__((always_inline)) {
    if (g.win <= 0 && k0 + BK <= nk) {
      // a whole block of the frame's patches, in order
      const unsigned char *kb = reinterpret_cast<const unsigned char *>(kbase + (long)k0 * g.d);
      const unsigned char *vb = reinterpret_cast<const unsigned char *>(vbase + (long)k0 * g.d);
#pragma unroll
      for (int i = 0; i < KT; ++i) {
        rk[i] = *reinterpret_cast<const u32x4 *>(kb + ko[i]);
        if (ROT) rp[i] = *reinterpret_cast<const u32x4 *>(kb + ko[i] + hd);
      }
#pragma unroll
      for (int i = 0; i < VT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          rv[i][r] = *reinterpret_cast<const u32x2 *>(vb + (size_t)r * 2 * g.d + vo[i]);
      return;
    }
#pragma unroll
    for (int i = 0; i < KT; ++i) {
      const uint16_t *src = kbase + (long)key_patch(g, w, min(k0 + ki[i], nk - 1)) * g.d + kc0[i];
      rk[i] = *reinterpret_cast<const u32x4 *>(src);
      if (ROT) rp[i] = *reinterpret_cast<const u32x4 *>(src + half);
    }
#pragma unroll
    for (int i = 0; i < VT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        rv[i][r] = *reinterpret_cast<const u32x2 *>(
            vbase + (long)key_patch(g, w, min(k0 + 4 * kg[i] + r, nk - 1)) * g.d + vc0[i]);
  };
  auto store_block = [&](int k0, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < KT; ++i) {
      if (t + i * 512 >= BK * cpr) continue;
      uint16_t *dst = Ks(buf) + ki[i] * KP + kc0[i];
      if (ROT) {
        const int quarter = hd / 4;
        int pr, pc;
        patch_pos(g, key_patch(g, w, min(k0 + ki[i], nk - 1)), pr, pc);
        float rx[8], ry[8];
#pragma unroll
        for (int q2 = 0; q2 < 8; ++q2) {
          const uint32_t kw = rk[i][q2 >> 1], pw = rp[i][q2 >> 1];
          const float x = __uint_as_float((q2 & 1) ? kw & 0xFFFF0000u : kw << 16);
          const float y = __uint_as_float((q2 & 1) ? pw & 0xFFFF0000u : pw << 16);
          const int pair = kc0[i] + q2;
          const bool lo = pair < quarter;
          const float2 cs = rope[(lo ? pr : pc) * 32 + (lo ? pair : pair - quarter)];
          const float2 z = rot_pair(x, y, cs);
          rx[q2] = z.x;
          ry[q2] = z.y;
        }
        st_bf8(dst, rx);
        st_bf8(dst + half, ry);
      } else {
        *reinterpret_cast<u32x4 *>(dst) = rk[i];
      }
    }
#pragma unroll
    for (int i = 0; i < VT; ++i) {
      if (t + i * 512 >= (BK / 4) * qpr) continue;
      uint32_t u[8];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        // low (c even) or high (c odd) halves of word c / 2 of the 4 rows
        const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;
        u[2 * c] = __builtin_amdgcn_perm(rv[i][1][c >> 1], rv[i][0][c >> 1], sel);
        u[2 * c + 1] = __builtin_amdgcn_perm(rv[i][3][c >> 1], rv[i][2][c >> 1], sel);
      }
      u32x4 *d = reinterpret_cast<u32x4 *>(Vq(buf) + kg[i] * HDP + vc0[i]);
      d[0] = u32x4{u[0], u[1], u[2], u[3]};
      d[1] = u32x4{u[4], u[5], u[6], u[7]};
    }
  };
  load_block(0);
  int nq;
  if (g.win <= 0) {                                        // every slot is of the one window
    nq = min(max(nrow - chunk * kVitQ, 0), kVitQ);
    if (nq == 0) return;
    if (t < kVitQ) qslot[t] = chunk * kVitQ + t;
    __syncthreads();
  } else {
    nq = window_queries(idx, g, b, w, chunk, nrow, qslot, wcnt, &nq_s);
    if (nq == 0) return;
  }
  // padded head dims stay zero for the whole kernel
  for (int e = t; e < BK * (HDP - hd); e += 512) {
    const int r = e / (HDP - hd);
    Ks(0)[r * KP + hd + (e - r * (HDP - hd))] = 0;
    Ks(1)[r * KP + hd + (e - r * (HDP - hd))] = 0;
  }
  for (int e = t; e < (BK / 4) * (HDP - hd); e += 512) {
    const int r = e / (HDP - hd);
    Vq(0)[r * HDP + hd + (e - r * (HDP - hd))] = u32x2{0, 0};
    Vq(1)[r * HDP + hd + (e - r * (HDP - hd))] = u32x2{0, 0};
  }
  // this lane's query (column l16 of the wave's 16) as the B operand, dims 32 s + 8 gq ..
  const int qi = (wv & 3) * 16 + l16;
  const bool wact = (wv & 3) * 16 < nq;
  bf16x8 qf[HDP / 32];
#pragma unroll
  for (int s = 0; s < HDP / 32; ++s) {
    const int c0 = 32 * s + 8 * gq;
    uint4 raw = make_uint4(0, 0, 0, 0);
    if (qi < nq && c0 < hd)
      raw = *reinterpret_cast<const uint4 *>(q + ((long)b * g.Np + qslot[qi]) * g.d + h * hd + c0);
    qf[s] = __builtin_bit_cast(bf16x8, raw);
  }
  f32x4 o[HDP / 16];
#pragma unroll
  for (int i = 0; i < HDP / 16; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float mrun = -INFINITY, lpart = 0.f;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)hd);
  // this group's KPG keys of the block in LDS buffer buf, kn of them valid
  constexpr int NT = KPG / 16;
  auto compute = [&](int buf, int kn) __attribute__((always_inline)) {
    const uint16_t *K = Ks(buf) + gr * KPG * KP;
    const u32x2 *V = Vq(buf) + gr * (KPG / 4) * HDP;
    f32x4 sa[NT];
#pragma unroll
    for (int kt = 0; kt < NT; ++kt) sa[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < HDP / 32; ++s)
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) {
        const bf16x8 ka = *reinterpret_cast<const bf16x8 *>(K + (16 * kt + l16) * KP + 32 * s + 8 * gq);
        sa[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qf[s], sa[kt], 0, 0, 0);
      }
    if (kn < KPG) {
#pragma unroll
      for (int kt = 0; kt < NT; ++kt)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (16 * kt + 4 * gq + e >= kn) sa[kt][e] = -INFINITY;
    }
    float bm[NT];
#pragma unroll
    for (int kt = 0; kt < NT; ++kt) bm[kt] = fmaxf(fmaxf(sa[kt][0], sa[kt][1]), fmaxf(sa[kt][2], sa[kt][3]));
    float bmax = bm[0];
#pragma unroll
    for (int kt = 1; kt < NT; ++kt) bmax = fmaxf(bmax, bm[kt]);
    bmax = fmaxf(bmax, __shfl_xor(bmax, 16));
    bmax = fmaxf(bmax, __shfl_xor(bmax, 32)) * scale_log2;   // log2 units; finite: kn >= 1
    // the reference maximum moves only when a score exceeds it by more than 2^8: below that
    // the probabilities keep their relative precision, and the rescale is skipped
    const bool grow = bmax > mrun + 8.f;
    if (__ballot(grow)) {
      const float corr = grow ? __builtin_amdgcn_exp2f(mrun - bmax) : 1.f;
      lpart *= corr;
#pragma unroll
      for (int i = 0; i < HDP / 16; ++i) o[i] *= corr;
      if (grow) mrun = bmax;
    }
    float ps[NT];
#pragma unroll
    for (int kt = 0; kt < NT; ++kt) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        sa[kt][e] = __builtin_amdgcn_exp2f(fmaf(sa[kt][e], scale_log2, -mrun));
      ps[kt] = (sa[kt][0] + sa[kt][1]) + (sa[kt][2] + sa[kt][3]);
    }
#pragma unroll
    for (int kt = 0; kt < NT; ++kt) lpart += ps[kt];
#pragma unroll
    for (int ks = 0; ks < NT / 2; ++ks) {
      bf16x8 pb;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        pb[e] = (__bf16)sa[2 * ks][e];
        pb[4 + e] = (__bf16)sa[2 * ks + 1][e];
      }
#pragma unroll
      for (int dt = 0; dt < HDP / 16; ++dt) {
        const u32x2 lo = V[(8 * ks + gq) * HDP + 16 * dt + l16], hi = V[(8 * ks + 4 + gq) * HDP + 16 * dt + l16];
        const bf16x8 va = __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pb, o[dt], 0, 0, 0);
      }
    }
  };
  store_block(0, 0);
  for (int kb = 0; kb < nblk; ++kb) {
    // block kb is in buffer kb & 1, and every reader of the other one (block kb - 1) is done
    __syncthreads();
    if (kb + 1 < nblk) load_block((kb + 1) * BK);
    const int kn = min(nk - kb * BK - gr * KPG, KPG);
    if (wact && kn > 0) compute(kb & 1, kn);
    if (kb + 1 < nblk) store_block((kb + 1) * BK, (kb & 1) ^ 1);
  }
  // merge the second group's sums into the first's
  float ltot = lpart + __shfl_xor(lpart, 16);
  ltot += __shfl_xor(ltot, 32);
  __syncthreads();
  constexpr int MP = HDP + 4;
  float *mo = reinterpret_cast<float *>(lds);               // [query][MP]
  static_assert(kVitQ * MP * 4 <= (int)sizeof(lds), "the sums fit");
  if (gr > 0 && wact) {
    if (gq == 0) {
      ml[0][qi] = mrun;
      ml[1][qi] = ltot;
    }
#pragma unroll
    for (int dt = 0; dt < HDP / 16; ++dt) *reinterpret_cast<f32x4 *>(mo + qi * MP + 16 * dt + 4 * gq) = o[dt];
  }
  __syncthreads();
  if (gr > 0 || qi >= nq) return;
  const float m1 = ml[0][qi], mm = fmaxf(mrun, m1);         // finite: the first group has keys
  const float f0 = __builtin_amdgcn_exp2f(mrun - mm), f1 = __builtin_amdgcn_exp2f(m1 - mm);
  const float inv = 1.f / (ltot * f0 + ml[1][qi] * f1);
  uint16_t *orow = out + ((long)b * g.Np + qslot[qi]) * g.d + h * hd;
#pragma unroll
  for (int dt = 0; dt < HDP / 16; ++dt) {
    const int c0 = 16 * dt + 4 * gq;
    if (c0 >= hd) continue;
    const f32x4 v = (o[dt] * f0 + *reinterpret_cast<const f32x4 *>(mo + qi * MP + c0) * f1) * inv;
    st_bf4(orow + c0, v[0], v[1], v[2], v[3]);
  }
}

// --------------------------------------------------------------------- patch merger
// Grid (item x recomputed token, patch): the patch row RMS-normalised, written at its
// place in the token's concatenated row (hidden = merge^2 d).
__global__ __launch_bounds__(kVitThreads) void k_merge_norm(
    const uint16_t *__restrict__ y, const uint16_t *__restrict__ gain,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ nrec, int N, int mm, int d,
    float eps, uint16_t *__restrict__ hb) {
  __shared__ float red[kVitThreads / 64];
  const long s = blockIdx.x;
  const int a = blockIdx.y;
  const int b = (int)(s / N), j = (int)(s - (long)b * N);
  if (j >= min(max(nrec[b], 0), N)) return;
  const int t = min(max(idx[s], 0), N - 1);
  norm_row(y + (((long)b * N + t) * mm + a) * d, gain, d, eps, hb + (s * mm + a) * d, red);
}

// Grid (slot, 1024-column chunk): split-K sums + bias, exact GELU (x Phi(x)), bf16
template <int SPL>
__global__ __launch_bounds__(kVitThreads) void k_merge_red_gelu(
    const float *__restrict__ part, int splits, int need, int B, const uint16_t *__restrict__ bias,
    const int32_t *__restrict__ nrec, int N, int hidden, uint16_t *__restrict__ act) {
  const long s = blockIdx.x;
  const int b = (int)(s / N), j = (int)(s - (long)b * N);
  if (j >= min(max(nrec[b], 0), N)) return;
  if (need && weight_streams(nrec, B, N) >= need) return;
  const int c = 4 * (blockIdx.y * kVitThreads + threadIdx.x);
  if (c >= hidden) return;
  const float4 v = sum_parts4<SPL>(part, splits, (long)gridDim.x, s, hidden, c);
  const float4 bb = bf4(bias + c);
  st_bf4(act + s * hidden + c, gelu_erf(bb.x + v.x), gelu_erf(bb.y + v.y), gelu_erf(bb.z + v.z),
         gelu_erf(bb.w + v.w));
}

// Grid (slot, 1024-column chunk): split-K sums + bias into the token's output row
template <int SPL>
__global__ __launch_bounds__(kVitThreads) void k_merge_red_out(
    const float *__restrict__ part, int splits, int need, int B, const uint16_t *__restrict__ bias,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ nrec, int N, int d_out,
    uint16_t *__restrict__ x_out) {
  const long s = blockIdx.x;
  const int b = (int)(s / N), j = (int)(s - (long)b * N);
  if (j >= min(max(nrec[b], 0), N)) return;
  if (need && weight_streams(nrec, B, N) >= need) return;
  const int c = 4 * (blockIdx.y * kVitThreads + threadIdx.x);
  if (c >= d_out) return;
  const int t = min(max(idx[s], 0), N - 1);
  const float4 v = sum_parts4<SPL>(part, splits, (long)gridDim.x, s, d_out, c);
  const float4 bb = bf4(bias + c);
  st_bf4(x_out + ((long)b * N + t) * d_out + c, bb.x + v.x, bb.y + v.y, bb.z + v.z, bb.w + v.w);
}

}  // namespace

// A reduction kernel instantiated for the smallest power of two >= the split count
#define FC_VIT_RED(kern, grid, splits, ...)                                             \
  do {                                                                                  \
    if (splits <= 1) hipLaunchKernelGGL(kern<1>, grid, dim3(kVitThreads), 0, st, __VA_ARGS__);      \
    else if (splits <= 2) hipLaunchKernelGGL(kern<2>, grid, dim3(kVitThreads), 0, st, __VA_ARGS__); \
    else if (splits <= 4) hipLaunchKernelGGL(kern<4>, grid, dim3(kVitThreads), 0, st, __VA_ARGS__); \
    else if (splits <= 8) hipLaunchKernelGGL(kern<8>, grid, dim3(kVitThreads), 0, st, __VA_ARGS__); \
    else hipLaunchKernelGGL(kern<16>, grid, dim3(kVitThreads), 0, st, __VA_ARGS__);                 \
  } while (0)

static fc_status vit_block(fc_ctx *ctx, const fc_vit_desc &L, const fc_vit_cache &c,
                           const uint16_t *x, const int32_t *idx, const int32_t *nrec,
                           uint16_t *y, int B, hipStream_t st) {
  VitGeo g;
  g.N = c.grid_h * c.grid_w;
  g.m = c.merge;
  g.mm = c.merge * c.merge;
  g.Np = g.N * g.mm;
  g.gh = c.grid_h;
  g.gw = c.grid_w;
  g.d = L.d_model;
  g.H = L.n_heads;
  g.hd = L.head_dim;
  g.win = c.window;
  const long slots = (long)B * g.Np;
  const int f = L.d_ffn;
  // rotated keys and, past a value a slot and column, the sums of squares: the partial-sum buffer
  // is free on this path and holds at least as many 32-bit values as the QKV columns of every slot
  const int nwin = c.window > 0 ? ((g.gh + c.window - 1) / c.window) * ((g.gw + c.window - 1) / c.window) : 1;
  const int wkeys = c.window > 0 ? std::min(c.window, g.gh) * std::min(c.window, g.gw) * g.mm : g.Np;
  uint16_t *krot = wkeys > 64 ? reinterpret_cast<uint16_t *>(ctx->part) : nullptr;
  fc_status rc;
  RowGemm a{};
  a.krot = krot;
  a.qw = a.kw = g.d;
  const int32_t *rows = ctx->vit_rows;
  a.B = B;
  a.cus = std::max(ctx->num_cus, 1);
  a.idx = idx;
  a.g = g;
  a.rope = ctx->vit_rope;
  a.h1 = ctx->h1;
  a.ssq = ctx->part + slots * g.d;
  a.parts = (g.d + kRowSsqCols - 1) / kRowSsqCols;
  a.eps = L.rms_eps;
  {
    ProfScope ps(ctx, st, "fc_vit_gather_norm");
    hipLaunchKernelGGL(k_vit_gather_norm, dim3((unsigned)slots), dim3(kVitThreads), 0, st, x, L.g1,
                       idx, nrec, g, L.rms_eps, L.rope_theta, ctx->hb, ctx->vit_rows,
                       ctx->vit_rope, (const uint16_t *)c.k, krot);
    FC_LAUNCH_OK(st, "k_vit_gather_norm");
  }
  a.A = ctx->hb; a.W = L.w_qkv; a.bias = L.b_qkv;
  a.K = g.d; a.cols = 3 * g.d;
  a.q = ctx->qbuf; a.kc = c.k; a.vc = c.v;
  if ((rc = run_row_gemm<V_QKV>(ctx, st, "fc_vit_gemm_qkv", a, rows)) != FC_OK) return rc;
  {
    // query chunks of 64 per window (full attention: one window of every patch)
    const int chunks = (wkeys + kVitQ - 1) / kVitQ;
    const dim3 grid((unsigned)g.H, (unsigned)(nwin * chunks), (unsigned)B);
    const uint16_t *qb = ctx->qbuf, *vb = c.v;
    const float2 *rp = ctx->vit_rope;
    ProfScope ps(ctx, st, "fc_vit_attn");
    // a window of at most 64 keys is one block of two groups' keys
#define FC_VIT_ATTN(HDP)                                                                       \
  do {                                                                                         \
    if (!krot)                                                                                 \
      hipLaunchKernelGGL((k_vit_attn<HDP, 32>), grid, dim3(512), 0, st, qb,                    \
                         (const uint16_t *)c.k, vb, idx, nrec, g, rp, chunks, ctx->attn);      \
    else                                                                                       \
      hipLaunchKernelGGL((k_vit_attn<HDP, 64>), grid, dim3(512), 0, st, qb,                    \
                         (const uint16_t *)krot, vb, idx, nrec, g, rp, chunks, ctx->attn);     \
  } while (0)
    if (g.hd <= 32) FC_VIT_ATTN(32);
    else if (g.hd <= 64) FC_VIT_ATTN(64);
    else if (g.hd <= 96) FC_VIT_ATTN(96);
    else FC_VIT_ATTN(128);
#undef FC_VIT_ATTN
    FC_LAUNCH_OK(st, "k_vit_attn");
  }
  a.A = ctx->attn; a.W = L.w_o; a.bias = L.b_o;
  a.cols = g.d;
  a.x = x; a.g2 = L.g2; a.hb = ctx->hb;
  if ((rc = run_row_gemm<V_O>(ctx, st, "fc_vit_gemm_o", a, rows)) != FC_OK) return rc;
  a.A = ctx->hb; a.W = L.w_gate_up; a.bias = L.b_gate_up;
  a.cols = 2 * f; a.act = ctx->act;
  if ((rc = run_row_gemm<V_GU>(ctx, st, "fc_vit_gemm_gateup", a, rows)) != FC_OK) return rc;
  a.A = ctx->act; a.W = L.w_down; a.bias = L.b_down;
  a.K = f; a.cols = g.d; a.y = y;
  return run_row_gemm<V_DOWN>(ctx, st, "fc_vit_gemm_down", a, rows);
}

fc_status launch_vit_block(fc_ctx *ctx, const fc_vit_desc &L, const fc_vit_cache &c,
                           const uint16_t *x, const int32_t *idx, const int32_t *nrec,
                           uint16_t *y, int B, hipStream_t st) {
  const long N = (long)c.grid_h * c.grid_w, Np = N * c.merge * c.merge;
  // The rotated keys and sums of squares take d / 2 + d / 64 values a row of the partial-sum
  // workspace.  The rows a context takes are those whose projections would fit there, as for
  // the layer's split-K sums, though no projection here writes them.
  if ((size_t)B * Np * std::max(3 * L.d_model, 2 * L.d_ffn) > ctx->part_elems)
    return fail(FC_ERR_CAPACITY, "fc_vit_block_forward: rows x columns of the projections exceed "
                "the partial-sum workspace");
  // the packed row map of a GEMM holds kMMaxItems items
  for (int b0 = 0; b0 < B; b0 += kMMaxItems) {
    fc_vit_cache cb = c;
    cb.k += b0 * Np * L.d_model;
    cb.v += b0 * Np * L.d_model;
    const fc_status s = vit_block(ctx, L, cb, x + b0 * Np * L.d_model, idx + b0 * N, nrec + b0,
                                  y + b0 * Np * L.d_model, std::min(B - b0, kMMaxItems), st);
    if (s != FC_OK) return s;
  }
  return FC_OK;
}

fc_status launch_vit_cache_update(fc_ctx *ctx, const fc_vit_desc &L, const fc_vit_cache &c,
                                  const uint16_t *y_prev, uint16_t *y_cur, const int32_t *shift,
                                  const uint8_t *reuse, int B, hipStream_t st) {
  // a merged token's patch rows are contiguous: the token-level remap with rows of
  // m^2 patches, from a separate previous-frame cache, or in place in the one frame
  // slot (whose overwrite stages the old rows)
  const int mm = c.merge * c.merge;
  if (c.k_prev)
    return launch_remap_copy(ctx, c.k_prev, c.v_prev, c.k, c.v, y_prev, y_cur,
                             c.grid_h * c.grid_w, mm * L.d_model, mm * L.d_model, c.grid_w,
                             shift, reuse, B, st);
  fc_layer_desc ld{};
  ld.d_model = mm * L.d_model;
  ld.n_heads = mm * L.n_heads;
  ld.n_kv_heads = mm * L.n_heads;
  ld.head_dim = L.head_dim;
  fc_kv_cache kv{};
  kv.k = c.k;
  kv.v = c.v;
  kv.text_tokens = 0;
  kv.frame_tokens = c.grid_h * c.grid_w;
  kv.window = 1;
  kv.head = 0;
  return launch_cache_update(ctx, ld, kv, y_prev, y_cur, shift, reuse, c.grid_w, B, st);
}

fc_status launch_vit_merger(fc_ctx *ctx, const fc_merger_desc &M, const uint16_t *y,
                            const int32_t *idx, const int32_t *nrec, uint16_t *x_out, int N,
                            int B, hipStream_t st) {
  const int mm = M.merge * M.merge;
  const int hidden = mm * M.d_model;
  const long slots = (long)B * N;
  uint16_t *hb = ctx->act;                                   // normalised token rows
  uint16_t *act = ctx->act + slots * hidden;                 // GELU outputs
  // (the row tiles need no partial sums; what fits does not depend on the GEMM taken)
  if ((size_t)slots * std::max(hidden, M.d_out) > ctx->part_elems)
    return fail(FC_ERR_CAPACITY, "fc_vit_merger_forward: partial sums exceed the workspace");
  fc_status rc;
  {
    ProfScope ps(ctx, st, "fc_merge_norm");
    hipLaunchKernelGGL(k_merge_norm, dim3((unsigned)slots, (unsigned)mm), dim3(kVitThreads), 0, st,
                       y, M.g, idx, nrec, N, mm, M.d_model, M.rms_eps, hb);
    FC_LAUNCH_OK(st, "k_merge_norm");
  }
  MergerRed red;
  if ((rc = run_merger_gemm(ctx, st, "fc_merge_gemm1", true, hb, M.w1, M.b1, hidden, hidden, N, idx,
                            nrec, act, B, red)) != FC_OK)
    return rc;
  if (red.splits) {
    ProfScope ps(ctx, st, "fc_merge_red_gelu");
    const dim3 grid((unsigned)slots, (unsigned)((hidden + 1023) / 1024));
    FC_VIT_RED(k_merge_red_gelu, grid, red.splits, (const float *)ctx->part, red.splits, red.need, B,
               M.b1, nrec, N, hidden, act);
    FC_LAUNCH_OK(st, "k_merge_red_gelu");
  }
  if ((rc = run_merger_gemm(ctx, st, "fc_merge_gemm2", false, act, M.w2, M.b2, hidden, M.d_out, N, idx,
                            nrec, x_out, B, red)) != FC_OK)
    return rc;
  if (red.splits) {
    ProfScope ps(ctx, st, "fc_merge_red_out");
    const dim3 grid((unsigned)slots, (unsigned)((M.d_out + 1023) / 1024));
    FC_VIT_RED(k_merge_red_out, grid, red.splits, (const float *)ctx->part, red.splits, red.need, B,
               M.b2, idx, nrec, N, M.d_out, x_out);
    FC_LAUNCH_OK(st, "k_merge_red_out");
  }
  return FC_OK;
}

}  // namespace fc
