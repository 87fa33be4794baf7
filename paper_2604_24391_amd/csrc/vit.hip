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
//   k_vit_gemm<V_QKV>  + bias; q rotated at the patch position (bf16, compact), raw k and v
//                      into the cache at the patch row.
//   k_vit_attn         one workgroup per (window, query chunk, head) or, with full
//                      attention, per (query chunk, head): the chunk's queries against the
//                      window's (the frame's) keys in blocks, S^T = K Q^T and O^T = V^T P^T
//                      on bf16 MFMAs, online softmax in fp32.
//   k_vit_gemm<V_O>    + bias + residual -> h1 (fp32), bf16(h1 g2) and the row's sums of
//                      squares by 64 columns.
//   k_vit_gemm<V_GU>   times 1/rms(h1), + biases, SiLU(g) u -> bf16.
//   k_vit_gemm<V_DOWN> + bias + h1 -> the slot's output row of y (bf16).
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

namespace fc {
namespace {

constexpr int kVitThreads = 256;
constexpr int kVitQ = 64;            // queries per attention workgroup

__device__ __forceinline__ float bf2f_v(uint16_t u) { return __uint_as_float((uint32_t)u << 16); }
__device__ __forceinline__ uint16_t f2bf_v(float f) {
  const uint32_t u = __float_as_uint(f);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

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

// Split-K sums of columns c .. c + 3 of row s (partials [split][rows][nc]): all SPL
// 16-byte loads issued first (indices past the last split re-read it), then summed in
// split order with the extra ones masked out.
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
template <int SPL>
__device__ __forceinline__ float4 sum_parts4(const float *__restrict__ part, int splits, long rows,
                                             long s, int nc, int c) {
  return sum_splits4<SPL>(part + s * nc + c, rows * nc, splits);
}
__device__ __forceinline__ float4 bf4(const uint16_t *p) {
  const uint2 u = *reinterpret_cast<const uint2 *>(p);
  return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u),
                     __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xFFFF0000u));
}
__device__ __forceinline__ void st_bf4(uint16_t *p, float a, float b, float c, float d) {
  *reinterpret_cast<uint2 *>(p) = make_uint2(f2bf_v(a) | ((uint32_t)f2bf_v(b) << 16),
                                             f2bf_v(c) | ((uint32_t)f2bf_v(d) << 16));
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
  for (int i = 0; i < 4; ++i) w[i] = f2bf_v(v[2 * i]) | ((uint32_t)f2bf_v(v[2 * i + 1]) << 16);
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
  const int e = (int)s * kVitThreads + t;
  const int npos = max(g.gh, g.gw) * g.m;
  if (e < npos * 32) {
    const int ps = e / 32, fk = e - ps * 32;
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
      st_bf4(krot + s * g.d + c, x0.x * w[0].x - x1.x * w[0].y, x0.y * w[1].x - x1.y * w[1].y,
             x0.z * w[2].x - x1.z * w[2].y, x0.w * w[3].x - x1.w * w[3].y);
      st_bf4(krot + s * g.d + c + half, x1.x * w[0].x + x0.x * w[0].y, x1.y * w[1].x + x0.y * w[1].y,
             x1.z * w[2].x + x0.z * w[2].y, x1.w * w[3].x + x0.w * w[3].y);
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
          rx[q2] = x * cs.x - y * cs.y;
          ry[q2] = y * cs.x + x * cs.y;
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

// ------------------------------------------------------------------------------ GEMMs
// C[rows][cols] = A[rows][K] W[cols][K]^T over the recomputed rows packed across items, with
// the projection's epilogue: one workgroup per TM x TN tile (TN staged weight rows), the whole
// K range, no partial sums.  A projection of a frame has a few hundred to a few thousand rows,
// so what bounds a tile is the load path of its CU (TM + TN rows of 128 B a K step), not its
// MFMAs: the tile is chosen on the device, where the row count is known, as the one whose CUs
// load least (vit_tile).
//   * NST stages of (TM + TN) rows rotate in LDS, 64 K values (a 128-B line) a row, 16-B
//     chunks XOR-swizzled by (row >> 1) & 7.  Waves 4-7 only issue the DMAs (a DMA holds its
//     wave at issue): after barrier k those of step k + NST - 1, into the stage of step k - 1.
//     Waves 0-3 multiply, a quarter of the tile each, and read the fragments of the next half
//     step while they multiply this one, across the barrier too.  (All eight waves loading and
//     multiplying, with or without the halves of the workgroup in alternating phases, was up
//     to 30 % slower: the DMAs keep the MFMAs waiting.)
//   * The accumulators go through LDS as whole rows, so that every global access of the
//     epilogue is a piece of a row: V_QKV adds the bias, rotates q and scatters raw k and v
//     into the cache; V_O adds bias and residual and writes h1, the MLP operand bf16(h1 g2)
//     and the row's sums of squares per 64 columns; V_GU applies 1/rms, adds the biases and
//     writes SiLU(g) u; V_DOWN adds bias and h1 and scatters the output rows.
//   * V_QKV stages a column beside its rotary partner half a head away (V_GU: a gate beside
//     its up row): staged rows [0, TN / 2) are columns, [TN / 2, TN) their partners.
//   * M tiles of one column tile are consecutive, so each XCD reads its own share of the
//     weights once.
// Measured on the Qwen2.5-VL block (d 1280, MLP 3456), us, against 256 x 256 tiles in up to 8
// K-range parts with a reduction kernel each: QKV 23 + 15 -> 18.5, O 15 + 9 -> 14, gate/up
// 28 + 14 -> 26, down 21 + 9 -> 21 at 1024 rows; the whole windowed block 157 -> 91 at 1024
// rows, 129 -> 78 at 512 and 89 -> 54 at 104 rows (there against the weight-streaming GEMM
// and its reductions).  The DMA pattern alone takes 7.3 us for QKV (37 B a clock and CU); LDS
// traffic (operands written once and read twice), about 3 us before the first step is staged
// and 2 us of epilogue make up the rest.
enum { V_QKV = 0, V_O = 1, V_GU = 2, V_DOWN = 3 };
constexpr int kVitLds = 150 * 1024;
constexpr int kVitSsqCols = 64;         // columns per partial sum of squares of h1

struct VitGemm {
  const uint16_t *A, *W, *bias;
  int K, cols;                          // cols: weight rows staged in all (V_GU: 2 f)
  int B, cus;
  const int32_t *idx;
  VitGeo g;
  const float2 *rope;
  uint16_t *q, *kc, *vc, *krot;         // V_QKV
  const uint16_t *x, *g2;               // V_O
  float *h1, *ssq;                      // V_O (V_GU reads ssq, V_DOWN h1)
  uint16_t *hb;                         // V_O
  uint16_t *act;                        // V_GU
  uint16_t *y;                          // V_DOWN
  int parts;                            // sums of squares per row
  float eps;
};

struct VitTile {
  int v, tiles;                         // variant, tiles of all rows
};
constexpr int kVitTM[4] = {128, 64, 64, 32}, kVitTN[4] = {128, 128, 64, 64};
constexpr int kVitGuTM[4] = {128, 128, 64, 32}, kVitGuTN[4] = {256, 128, 128, 64};
// The tile for `rows` rows: least rows loaded per CU, (TM + TN) times the rounds of one
// workgroup per CU (a K step of a 64 x 64 tile takes 0.2 us, of a 128 x 128 tile 0.5 us).  Host
// and device take the same decision.
__host__ __device__ inline VitTile vit_tile(bool gu, int rows, int cols, int cus) {
  VitTile best{0, 0};
  int least = 0;
  for (int v = 0; v < 4; ++v) {
    const int tm = gu ? kVitGuTM[v] : kVitTM[v], tn = gu ? kVitGuTN[v] : kVitTN[v];
    const int tiles = ((rows + tm - 1) / tm) * ((cols + tn - 1) / tn);
    const int cost = (tiles + cus - 1) / cus * (tm + tn);
    if (v == 0 || cost < least) {
      best = VitTile{v, tiles};
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
__device__ __forceinline__ void vit_gemm_tile(const VitGemm &a, unsigned char *lds, const int *pre,
                                              int *rslot, int *rpatch, int *rpos, float *rinv,
                                              int row0, int nvalid, int nt) {
  constexpr int STAGE = (TM + TN) * RB;
  constexpr int NST = kVitLds / STAGE > 8 ? 8 : kVitLds / STAGE;
  constexpr int NI = (TM + TN) / 8;               // DMA instructions per step
  constexpr int L = NI / 4;                       // of each loader wave
  constexpr int MBW = TM / 32, NBW = TN / 32;     // 16-row blocks of a wave's quarter
  constexpr bool PAIR = MODE == V_QKV || MODE == V_GU;
  static_assert(NST >= 3 && NI % 4 == 0 && (NST - 1) * L < 64, "stages");
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const VitGeo &g = a.g;
  const int nk = a.K / KS;
  // column of staged row r (clamped: past the last column nothing is stored)
  auto column = [&](int r) {
    if (MODE == V_QKV) {
      const int half = g.hd / 2, p = min(nt * (TN / 2) + r % (TN / 2), a.cols / 2 - 1);
      const int h = p / half;
      return h * g.hd + (p - h * half) + (r >= TN / 2 ? half : 0);
    }
    if (MODE == V_GU)
      return min(nt * (TN / 2) + r % (TN / 2), a.cols / 2 - 1) + (r >= TN / 2 ? a.cols / 2 : 0);
    return min(nt * TN + r, a.cols - 1);
  };
  constexpr int TP = TN + 4;                      // floats per row of the epilogue tile
  static_assert(TM * TP * 4 <= kVitLds, "the tile fits");
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
    // the tile's rows: slot, patch row (b Np + patch) and, for V_GU, 1/rms of h1
    if (t < TM) {
      int b = 0;
      const long sl = row_slot(pre, a.B, g.Np, row0 + min(t, nvalid - 1), b);
      rslot[t] = (int)sl;
      if (MODE != V_GU) {
        const int p = slot_patch(a.idx, g, b, (int)(sl - (long)b * g.Np));
        rpatch[t] = b * g.Np + p;
        if (MODE == V_QKV) {
          int pr, pc;
          patch_pos(g, p, pr, pc);
          rpos[t] = pr << 16 | pc;
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
    const bool rot = MODE == V_QKV && c0 < (a.krot ? 2 : 1) * g.d;
    // rotary pairs c0 % hd .. + 3: the first quarter of a head turns by the patch row, the
    // second by its column (four pairs may span both)
    const int quarter = g.hd / 4, pair = c0 % g.hd;
    const bool isq = c0 < g.d;
    float2 cs[IT][4];
    if (rot) {
#pragma unroll
      for (int n = 0; n < IT; ++n) {
        const int pos = rpos[min(r0 + n * RSTEP, TM - 1)], pr = pos >> 16, pc = pos & 0xFFFF;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool lo = pair + i < quarter;
          cs[n][i] = a.rope[(lo ? pr : pc) * 32 + pair + i - (lo ? 0 : quarter)];
        }
      }
    }
    uint16_t *kv = c0 < 2 * g.d ? a.kc - g.d : a.vc - 2 * g.d;
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
          x0[i] = gv * __builtin_amdgcn_rcpf(1.f + __expf(-gv)) * uv;
        }
        st_bf4(a.act + (long)rslot[r] * (a.cols / 2) + p, x0[0], x0[1], x0[2], x0[3]);
      } else {
        // raw keys and values go to the cache, rotated queries and keys to the attention
        float y0[4], y1[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          x0[i] = v4[i] + bb0[i];
          x1[i] = u4[i] + bb1[i];
          if (rot) {
            y0[i] = x0[i] * cs[n][i].x - x1[i] * cs[n][i].y;
            y1[i] = x1[i] * cs[n][i].x + x0[i] * cs[n][i].y;
          }
        }
        if (!isq) {
          uint16_t *dst = kv + (long)rpatch[r] * g.d;
          st_bf4(dst + c0, x0[0], x0[1], x0[2], x0[3]);
          st_bf4(dst + c1, x1[0], x1[1], x1[2], x1[3]);
        }
        if (rot) {
          uint16_t *dst = isq ? a.q + (long)rslot[r] * g.d : a.krot - g.d + (long)rpatch[r] * g.d;
          st_bf4(dst + c0, y0[0], y0[1], y0[2], y0[3]);
          st_bf4(dst + c1, y1[0], y1[1], y1[2], y1[3]);
        }
      }
    }
  } else {
    const int c = nt * TN + c4;
    const bool cv = c < a.cols;
    const int cc = cv ? c : 0;
    const float4 bb = bf4(a.bias + cc);
    const float4 gn = MODE == V_O ? bf4(a.g2 + cc) : make_float4(0.f, 0.f, 0.f, 0.f);
    uint2 xr[MODE == V_O ? IT : 1];
    float4 hr[MODE == V_DOWN ? IT : 1];
#pragma unroll
    for (int n = 0; n < IT; ++n) {
      const int r = min(r0 + n * RSTEP, nvalid - 1);
      if (MODE == V_O) xr[n] = *reinterpret_cast<const uint2 *>(a.x + (long)rpatch[r] * g.d + cc);
      if (MODE == V_DOWN) hr[n] = *reinterpret_cast<const float4 *>(a.h1 + (long)rslot[r] * g.d + cc);
    }
#pragma unroll
    for (int n = 0; n < IT; ++n) {
      const int r = r0 + n * RSTEP;
      const bool rv = r < nvalid;
      float ss = 0.f;
      if (rv && cv) {
        const long slot = rslot[r];
        const float4 v = *reinterpret_cast<const float4 *>(T + r * TP + c4);
        if (MODE == V_O) {
          const float4 xv = unpack_bf16x4(xr[n]);
          const float4 h = make_float4(xv.x + (v.x + bb.x), xv.y + (v.y + bb.y), xv.z + (v.z + bb.z),
                                       xv.w + (v.w + bb.w));
          *reinterpret_cast<float4 *>(a.h1 + slot * g.d + c) = h;
          st_bf4(a.hb + slot * g.d + c, h.x * gn.x, h.y * gn.y, h.z * gn.z, h.w * gn.w);
          ss = h.x * h.x + h.y * h.y + h.z * h.z + h.w * h.w;
        } else {
          const float4 h = hr[n];
          st_bf4(a.y + (long)rpatch[r] * g.d + c, h.x + (v.x + bb.x), h.y + (v.y + bb.y),
                 h.z + (v.z + bb.z), h.w + (v.w + bb.w));
        }
      }
      if (MODE == V_O) {
        // 64 columns of a row are 16 consecutive lanes
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
        if (rv && cv && (lane & 15) == 0) a.ssq[(long)rslot[r] * a.parts + c / kVitSsqCols] = ss;
      }
    }
  }
}

template <int MODE>
__global__ __launch_bounds__(512) void k_vit_gemm(VitGemm a, const int32_t *__restrict__ rows) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[kVitLds];
  __shared__ int pre[kMMaxItems + 1];
  __shared__ int rslot[128], rpatch[128], rpos[128];
  __shared__ float rinv[128];
  int M;
  if (a.B == 1) {                                // one item: its rows are the packed rows
    M = n_valid(rows, 0, a.g.Np);
  } else {
    if (threadIdx.x < 64) row_prefix(rows, a.B, a.g.Np, pre);
    __syncthreads();
    M = pre[a.B];
  }
  const VitTile vt = vit_tile(MODE == V_GU, M, a.cols, a.cus);
  if ((int)blockIdx.x >= vt.tiles) return;
  const int tm = MODE == V_GU ? kVitGuTM[vt.v] : kVitTM[vt.v];
  const int mt = (M + tm - 1) / tm;
  const int l = xcd_tile(blockIdx.x, vt.tiles), nt = l / mt, row0 = (l - nt * mt) * tm;
  const int nvalid = min(tm, M - row0);
#define FC_VT(i)                                                                               \
  vit_gemm_tile<MODE, MODE == V_GU ? kVitGuTM[i] : kVitTM[i], MODE == V_GU ? kVitGuTN[i] : kVitTN[i]>( \
      a, lds, pre, rslot, rpatch, rpos, rinv, row0, nvalid, nt)
  switch (vt.v) {
    case 0: FC_VT(0); break;
    case 1: FC_VT(1); break;
    case 2: FC_VT(2); break;
    default: FC_VT(3); break;
  }
#undef FC_VT
}

// The most tiles any row count up to `rows` takes (the grid; surplus workgroups exit).
int vit_grid(bool gu, int rows, int cols, int cus) {
  int most = 1;
  for (int r = 1; r <= rows; r += 32)
    most = std::max(most, vit_tile(gu, std::min(r + 31, rows), cols, cus).tiles);
  return most;
}

template <int MODE>
fc_status run_vit_gemm(fc_ctx *ctx, hipStream_t st, const char *name, const VitGemm &a) {
  const int grid = vit_grid(MODE == V_GU, a.B * a.g.Np, a.cols, a.cus);
  ProfScope ps(ctx, st, name);
  hipLaunchKernelGGL(k_vit_gemm<MODE>, dim3((unsigned)grid), dim3(512), 0, st, a,
                     (const int32_t *)ctx->vit_rows);
  FC_LAUNCH_OK(st, "k_vit_gemm");
  return FC_OK;
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

__device__ __forceinline__ float gelu_erf(float v) {
  return 0.5f * v * (1.f + erff(v * 0.70710678118654752f));
}
// Grid (slot, 1024-column chunk): split-K sums + bias, exact GELU (x Phi(x)), bf16
template <int SPL>
__global__ __launch_bounds__(kVitThreads) void k_merge_red_gelu(
    const float *__restrict__ part, int splits, const uint16_t *__restrict__ bias,
    const int32_t *__restrict__ nrec, int N, int hidden, uint16_t *__restrict__ act) {
  const long s = blockIdx.x;
  const int b = (int)(s / N), j = (int)(s - (long)b * N);
  if (j >= min(max(nrec[b], 0), N)) return;
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
    const float *__restrict__ part, int splits, const uint16_t *__restrict__ bias,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ nrec, int N, int d_out,
    uint16_t *__restrict__ x_out) {
  const long s = blockIdx.x;
  const int b = (int)(s / N), j = (int)(s - (long)b * N);
  if (j >= min(max(nrec[b], 0), N)) return;
  const int c = 4 * (blockIdx.y * kVitThreads + threadIdx.x);
  if (c >= d_out) return;
  const int t = min(max(idx[s], 0), N - 1);
  const float4 v = sum_parts4<SPL>(part, splits, (long)gridDim.x, s, d_out, c);
  const float4 bb = bf4(bias + c);
  st_bf4(x_out + ((long)b * N + t) * d_out + c, bb.x + v.x, bb.y + v.y, bb.z + v.z, bb.w + v.w);
}

}  // namespace

// A reduction kernel instantiated for the smallest power of two >= the split count
#define FC_VIT_RED(kern, grid, ...)                                                     \
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
  // rotated keys and, after them, the sums of squares: the partial-sum buffer is free on this
  // path and holds at least as many 32-bit values as the QKV columns of every slot
  const int nwin = c.window > 0 ? ((g.gh + c.window - 1) / c.window) * ((g.gw + c.window - 1) / c.window) : 1;
  const int wkeys = c.window > 0 ? std::min(c.window, g.gh) * std::min(c.window, g.gw) * g.mm : g.Np;
  uint16_t *krot = wkeys > 64 ? reinterpret_cast<uint16_t *>(ctx->part) : nullptr;
  fc_status rc;
  VitGemm a{};
  a.krot = krot;
  a.B = B;
  a.cus = std::max(ctx->num_cus, 1);
  a.idx = idx;
  a.g = g;
  a.rope = ctx->vit_rope;
  a.h1 = ctx->h1;
  a.ssq = ctx->part + slots * g.d;
  a.parts = (g.d + kVitSsqCols - 1) / kVitSsqCols;
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
  if ((rc = run_vit_gemm<V_QKV>(ctx, st, "fc_vit_gemm_qkv", a)) != FC_OK) return rc;
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
  if ((rc = run_vit_gemm<V_O>(ctx, st, "fc_vit_gemm_o", a)) != FC_OK) return rc;
  a.A = ctx->hb; a.W = L.w_gate_up; a.bias = L.b_gate_up;
  a.cols = 2 * f; a.act = ctx->act;
  if ((rc = run_vit_gemm<V_GU>(ctx, st, "fc_vit_gemm_gateup", a)) != FC_OK) return rc;
  a.A = ctx->act; a.W = L.w_down; a.bias = L.b_down;
  a.K = f; a.cols = g.d; a.y = y;
  return run_vit_gemm<V_DOWN>(ctx, st, "fc_vit_gemm_down", a);
}

fc_status launch_vit_block(fc_ctx *ctx, const fc_vit_desc &L, const fc_vit_cache &c,
                           const uint16_t *x, const int32_t *idx, const int32_t *nrec,
                           uint16_t *y, int B, hipStream_t st) {
  const long N = (long)c.grid_h * c.grid_w, Np = N * c.merge * c.merge;
  // the projections' sums fit the partial-sum workspace of the context
  if ((size_t)B * Np * std::max(3 * L.d_model, 2 * L.d_ffn) > ctx->part_elems)
    return fail(FC_ERR_CAPACITY, "fc_vit_block_forward: partial sums exceed the workspace");
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
  int splits = 1;
  fc_status rc;
  {
    ProfScope ps(ctx, st, "fc_merge_norm");
    hipLaunchKernelGGL(k_merge_norm, dim3((unsigned)slots, (unsigned)mm), dim3(kVitThreads), 0, st,
                       y, M.g, idx, nrec, N, mm, M.d_model, M.rms_eps, hb);
    FC_LAUNCH_OK(st, "k_merge_norm");
  }
  if ((rc = run_plain_gemm(ctx, st, "fc_merge_gemm1", hb, M.w1, hidden, hidden, N, nrec,
                           ctx->part, B, &splits)) != FC_OK)
    return rc;
  {
    ProfScope ps(ctx, st, "fc_merge_red_gelu");
    const dim3 grid((unsigned)slots, (unsigned)((hidden + 1023) / 1024));
    FC_VIT_RED(k_merge_red_gelu, grid, (const float *)ctx->part, splits, M.b1, nrec, N, hidden,
               act);
    FC_LAUNCH_OK(st, "k_merge_red_gelu");
  }
  if ((rc = run_plain_gemm(ctx, st, "fc_merge_gemm2", act, M.w2, hidden, M.d_out, N, nrec,
                           ctx->part, B, &splits)) != FC_OK)
    return rc;
  {
    ProfScope ps(ctx, st, "fc_merge_red_out");
    const dim3 grid((unsigned)slots, (unsigned)((M.d_out + 1023) / 1024));
    FC_VIT_RED(k_merge_red_out, grid, (const float *)ctx->part, splits, M.b2, idx, nrec, N,
               M.d_out, x_out);
    FC_LAUNCH_OK(st, "k_merge_red_out");
  }
  return FC_OK;
}

}  // namespace fc
