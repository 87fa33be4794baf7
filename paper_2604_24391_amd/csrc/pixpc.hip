// Pixel-resolution phase correlation on gfx950: Eq. 4-1 with the feature maps taken as
// the frames' full-resolution BT.601 luma, the integer peak refined per axis by a
// three-point parabola, and (for the selection) the displacement rounded to whole tokens.
// A variant of Module I (Sec. 4.1) for frames whose motion is not a whole number of
// tokens; the token-grid reading stays the default.
//
// The frames are real, so only columns 0..W/2 of each row spectrum are kept (the rest
// is their conjugate mirror).  Five kernels per call, all float64 like the oracle's
// decision:
//
//   k_pc_rows      a wave takes two rows of one frame's luma as the real and imaginary part
//                  of one length-W sequence, transforms it and separates the two half-row
//                  spectra (both rows are of the same frame: packing rows of two frames
//                  would leak one frame's rounding noise into the other's spectrum, which
//                  dominates when a frame is zero).
//   k_pc_cols_fwd  a wave takes one column at a time: column FFTs of both half-spectra,
//                  cross power X = F_{t-1} conj(F_t), the workgroup's largest |X|.
//   k_pc_cols_inv  same columns: X / |X| under the guard |X| > 1e-9 max|X| (else 0),
//                  inverse column FFTs.
//   k_pc_rows_inv  a wave takes two rows: their Hermitian spectra completed from the halves
//                  and packed into one sequence, inverse FFT, real part / (H W) = the
//                  response surface (written only when the caller asks for it) and each
//                  row's first maximum.
//   k_pc_peak      one workgroup per pair: first maximum over the rows, signed wrap,
//                  parabolic refinement with circular neighbours (four values of the
//                  surface, summed from its row spectra), the token shift.
//
// The maximum is the first element, in row order, that reaches it up to kPcTie: frames that
// repeat along an axis (bands, tiles, a wall of one colour) have a surface of equal maxima,
// and the rounding of a packed row's two halves and of the twiddle products would pick one
// of them at random, up to half a frame away.
//
// The FFTs are of length n = 7 2^k, one sequence (several short ones) inside one wave, so
// that their stages need no workgroup barrier: 448 points (896 for n = 896), 7 or 8 (14 or
// 16) a lane, one radix-7 stage and one or two power-of-two stages in registers with an
// exchange through the wave's own LDS between stages.  The forward transform is decimated
// in frequency and leaves its result in a lane order of its own; the inverse is its mirror
// and starts from that order, so the cross power goes to memory and back as the registers
// hold it.  Twiddles come from a table per workgroup (sincospi of the exact rational angle).
// Sizes: H and W of the form 7 2^k with 2 <= 2^k <= 128 (14 ... 896).
//
// What bounds it: memory.  64 pairs of 448 x 448 move 308 MB of frames and 826 MB of
// half-spectra, eight passes over 103 MB (both written once and read by the forward columns,
// the cross power written and read, its inverse columns written and read).  Measured there, against transforms of one sequence
// per workgroup with a barrier after every stage and every twiddle product in LDS:
//   k_pc_rows 421 -> 105 us (4.9 TB/s; a large copy reaches 4.6 TB/s), k_pc_cols_fwd
//   305 -> 58 us (5.4 TB/s), k_pc_cols_inv 129 -> 46 us (4.5 TB/s), k_pc_rows_inv
//   249 -> 33 us (3.2 TB/s; it no longer writes the surface for the selection),
//   k_pc_peak 4.8 -> 5.4 us (it sums the neighbours itself); fc_select 1225 -> 358 us.
//
// Half-spectra lie in strips of 8 columns, [strip][row][8] (the last strip as wide as what
// is left), so that a row's pieces and a strip's rows are whole 128-B lines; the cross power
// lies by columns, [column][n] in lane order, over the same columns' place.
//
// Rotation (Fourier-Mellin, launch_pixel_pc_rot): the forward column pass also writes
// the high-pass weighted magnitude spectra of both frames; k_lp_sample resamples them
// on a log-polar grid (H angles over [0, pi), min(H, W) / 2 radii); the same correlation
// kernels on those maps give the rotation from the peak's angular coordinate;
// k_derotate rotates the current frame's luma back about the centre; a last
// correlation gives the displacement of the image centre.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "fc_internal.h"

namespace fc {
namespace {

constexpr int kPcThreads = 256;
constexpr int kPcMaxN = 896;
constexpr int kPcWaves = kPcThreads / 64;
// Elements of a surface this close to its maximum, relative to it, are equal to it: the
// rounding of the transforms is of some 1e-15, and 2e5 elements without a period leave
// their two largest about 1e-2 apart.
constexpr double kPcTie = 1e-12;

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
// a times w (forward) or conj(w) (inverse)
template <bool INV>
__device__ __forceinline__ double2 ctw(double2 a, double2 w) {
  return INV ? make_double2(a.x * w.x + a.y * w.y, a.y * w.x - a.x * w.y) : cmul(a, w);
}
// a times -i (forward) or i (inverse)
template <bool INV>
__device__ __forceinline__ double2 crot(double2 a) {
  return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

// In-register DFT of R points: v[q] = sum_r v[r] e^{-+2 pi i r q / R} (- forward).
template <int R, bool INV>
struct Dft;
template <bool INV>
struct Dft<2, INV> {
  static __device__ __forceinline__ void run(double2 (&v)[2]) {
    const double2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  }
};
template <bool INV>
__device__ __forceinline__ void dft4(double2 &a, double2 &b, double2 &c, double2 &d) {
  const double2 s02 = cadd(a, c), d02 = csub(a, c);
  const double2 s13 = cadd(b, d), j13 = crot<INV>(csub(b, d));
  a = cadd(s02, s13);
  b = cadd(d02, j13);
  c = csub(s02, s13);
  d = csub(d02, j13);
}
template <bool INV>
struct Dft<4, INV> {
  static __device__ __forceinline__ void run(double2 (&v)[4]) { dft4<INV>(v[0], v[1], v[2], v[3]); }
};
template <bool INV>
struct Dft<8, INV> {
  static __device__ __forceinline__ void run(double2 (&v)[8]) {
    constexpr double h = 0.70710678118654752440;     // cos(pi / 4)
    double2 e[4], o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      e[i] = cadd(v[i], v[i + 4]);
      o[i] = csub(v[i], v[i + 4]);
    }
    const double2 r1 = crot<INV>(o[1]), r3 = crot<INV>(o[3]);
    o[1] = make_double2(h * (o[1].x + r1.x), h * (o[1].y + r1.y));      // e^{-+ i pi / 4}
    o[2] = crot<INV>(o[2]);
    o[3] = make_double2(h * (r3.x - o[3].x), h * (r3.y - o[3].y));      // e^{-+ 3 i pi / 4}
    dft4<INV>(e[0], e[1], e[2], e[3]);
    dft4<INV>(o[0], o[1], o[2], o[3]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = e[i];
      v[2 * i + 1] = o[i];
    }
  }
};
template <bool INV>
struct Dft<16, INV> {
  static __device__ __forceinline__ void run(double2 (&v)[16]) {
    constexpr double h = 0.70710678118654752440, c = 0.92387953251128675613,
                     s = 0.38268343236508977173;     // cos, sin of pi / 8
    // e^{-2 pi i m / 16}, m = i p for i, p in 0..3
    const double2 w[10] = {{1, 0}, {c, -s}, {h, -h}, {s, -c}, {0, -1}, {-s, -c}, {-h, -h}, {-c, -s}, {-1, 0}, {-c, s}};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      dft4<INV>(v[i], v[i + 4], v[i + 8], v[i + 12]);
#pragma unroll
      for (int p = 1; p < 4; ++p)
        if (i > 0) v[i + 4 * p] = ctw<INV>(v[i + 4 * p], w[i * p]);
    }
    double2 o[16];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      dft4<INV>(v[4 * p], v[4 * p + 1], v[4 * p + 2], v[4 * p + 3]);
#pragma unroll
      for (int q = 0; q < 4; ++q) o[p + 4 * q] = v[4 * p + q];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = o[i];
  }
};
// 7 points from their sums and differences of opposite elements: X_q = c_q -+ i d_q and
// X_{7-q} = c_q +- i d_q with c_q = v_0 + sum cos(2 pi i q / 7) (v_i + v_{7-i}),
// d_q = sum sin(2 pi i q / 7) (v_i - v_{7-i}), i = 1..3: 36 multiply-adds instead of the
// 144 of the plain sum.
template <bool INV>
struct Dft<7, INV> {
  static __device__ __forceinline__ void run(double2 (&v)[7]) {
    constexpr double C[3] = {0.62348980185873353053, -0.22252093395631440429, -0.90096886790241912624};
    constexpr double S[3] = {0.78183148246802980871, 0.97492791218182360702, 0.43388373911755812048};
    double2 t[3], u[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      t[i] = cadd(v[i + 1], v[6 - i]);
      u[i] = csub(v[i + 1], v[6 - i]);
    }
    const double2 v0 = v[0];
    v[0] = cadd(cadd(v0, t[0]), cadd(t[1], t[2]));
#pragma unroll
    for (int q = 1; q <= 3; ++q) {
      double2 c = v0, d = make_double2(0.0, 0.0);
#pragma unroll
      for (int i = 1; i <= 3; ++i) {
        const int m = (i * q) % 7;                       // cos is even, sin odd in m -> 7 - m
        const double cs = C[(m <= 3 ? m : 7 - m) - 1];
        const double sn = m <= 3 ? S[m - 1] : -S[6 - m];
        c.x = fma(cs, t[i - 1].x, c.x);
        c.y = fma(cs, t[i - 1].y, c.y);
        d.x = i == 1 ? sn * u[0].x : fma(sn, u[i - 1].x, d.x);
        d.y = i == 1 ? sn * u[0].y : fma(sn, u[i - 1].y, d.y);
      }
      const double2 r = crot<INV>(d);
      v[q] = cadd(c, r);
      v[7 - q] = csub(c, r);
    }
  }
};

// LDS of one wave: order its writes before its later reads (other lanes' elements).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}

// Transforms of length N = 7 L, L = 2^k = R1 R2, S of them side by side in one wave (PTS
// points).  Lane s L + j holds elements j + L r, r < 7, of sequence s (lane j: j and j + 64
// for L = 128).
//   stage 1: DFT over r -> q, times e^{-2 pi i j q / N}; A_q[j]
//   stage 2: j = j0 + R2 j1, DFT over j1 -> p0, times e^{-2 pi i j0 p0 / L}; B_q[p0][j0]
//   stage 3: DFT over j0 -> p1: X[q + 7 (p0 + R1 p1)]       (R2 = 1: stage 2 is the last)
// Butterfly `it` of stages 2 and 3 is lane it % 56's (it = lane + 56 i), so 56 lanes work.
// A forward result is element (i, e) of lane < 56: item it = lane + 56 i, last index e.
template <int L>
struct Fft {
  static constexpr int N = 7 * L;
  static constexpr int S = L < 64 ? 64 / L : 1;
  static constexpr int V = L > 64 ? L / 64 : 1;
  static constexpr int R1 = L >= 128 ? 16 : (L >= 32 ? 8 : (L >= 16 ? 4 : L));
  static constexpr int R2 = L / R1;
  static constexpr int PTS = N * S;
  static constexpr int NI1 = PTS / R1 / 56, NI2 = PTS / R2 / 56;
  static constexpr int RL = R2 > 1 ? R2 : R1, NIL = R2 > 1 ? NI2 : NI1;   // the last stage
  static constexpr int IPS = N / RL;                       // last-stage items per sequence
  static constexpr int TW1 = 6 * L, TW = TW1 + (R2 > 1 ? (R1 - 1) * R2 : 0);
  static_assert(S * L * V >= 64 && NIL * 56 * RL == PTS && NI1 * 56 * R1 == PTS, "whole lanes");

  // tw[(q - 1) L + j] = e^{-2 pi i j q / N}, then [(p0 - 1) R2 + j0] = e^{-2 pi i j0 p0 / L}
  static __device__ void table(double2 *tw) {
    for (int e = threadIdx.x; e < TW; e += blockDim.x) {
      int m;
      if (e < TW1) {
        m = (e % L) * (e / L + 1);
      } else {
        const int x = e - TW1;
        m = 7 * (x % R2) * (x / R2 + 1);
      }
      double s, c;
      sincospi(2.0 * (double)(m % N) / (double)N, &s, &c);
      tw[e] = make_double2(c, -s);
    }
  }
  // place of B_q[p0][j0] in its q block: j0 is exchanged by an XOR of p0 so that both the
  // stage-2 writes (p0 fixed) and the stage-3 reads (j0 fixed) meet eight different 16-B
  // columns of the LDS in eight neighbouring lanes
  static __device__ __forceinline__ int bplace(int p0, int j0) {
    return p0 * R2 + (j0 ^ (R2 == 8 ? (p0 & 7) : (p0 >> 1) & (R2 - 1)));
  }
  // sequence and natural index of a result element
  static __device__ __forceinline__ void where(int it, int e, int &s, int &k) {
    s = it / IPS;
    const int x = it - s * IPS;
    k = R2 > 1 ? x / R1 + 7 * (x % R1 + R1 * e) : x + 7 * e;
  }

  template <bool INV>
  static __device__ __forceinline__ void dif(double2 (&v)[V][7], double2 (&out)[NIL][RL],
                                             double2 *buf, const double2 *tw) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int a = 0; a < V; ++a) {
      const int j = (lane % (L < 64 ? L : 64)) + 64 * a, s = L < 64 ? lane / L : 0;
      Dft<7, INV>::run(v[a]);
      double2 *d = buf + s * N + j;
      d[0] = v[a][0];
#pragma unroll
      for (int q = 1; q < 7; ++q) d[q * L] = ctw<INV>(v[a][q], tw[(q - 1) * L + j]);
    }
    wave_sync();
    double2 x[NI1][R1];
    if (lane < 56) {
#pragma unroll
      for (int i = 0; i < NI1; ++i) {
        const int it = lane + 56 * i, s = it / (7 * R2), q = (it / R2) % 7, j0 = it % R2;
#pragma unroll
        for (int r = 0; r < R1; ++r) x[i][r] = buf[s * N + q * L + j0 + R2 * r];
      }
    }
    wave_sync();
    if (R2 == 1) {
#pragma unroll
      for (int i = 0; i < NI1; ++i) {
        Dft<R1, INV>::run(x[i]);
#pragma unroll
        for (int r = 0; r < R1; ++r) out[i % NIL][r % RL] = x[i][r];
      }
      return;
    }
    if (lane < 56) {
#pragma unroll
      for (int i = 0; i < NI1; ++i) {
        const int it = lane + 56 * i, s = it / (7 * R2), q = (it / R2) % 7, j0 = it % R2;
        Dft<R1, INV>::run(x[i]);
        double2 *d = buf + s * N + q * L;
        d[bplace(0, j0)] = x[i][0];
#pragma unroll
        for (int p = 1; p < R1; ++p)
          d[bplace(p, j0)] = ctw<INV>(x[i][p], tw[TW1 + (p - 1) * R2 + j0]);
      }
    }
    wave_sync();
    if (lane < 56) {
#pragma unroll
      for (int i = 0; i < NIL; ++i) {
        const int it = lane + 56 * i, s = it / IPS, y = it - s * IPS, q = y / R1, p0 = y % R1;
#pragma unroll
        for (int e = 0; e < RL; ++e) out[i][e] = buf[s * N + q * L + bplace(p0, e)];
        Dft<RL, INV>::run(out[i]);
      }
    }
    wave_sync();
  }

  // The mirror of dif: from a result in lane order back to natural order (unnormalised).
  template <bool INV>
  static __device__ __forceinline__ void dit(double2 (&in)[NIL][RL], double2 (&v)[V][7],
                                             double2 *buf, const double2 *tw) {
    const int lane = threadIdx.x & 63;
    if (R2 > 1 && lane < 56) {
#pragma unroll
      for (int i = 0; i < NIL; ++i) {
        const int it = lane + 56 * i, s = it / IPS, y = it - s * IPS, q = y / R1, p0 = y % R1;
        Dft<RL, INV>::run(in[i]);
        double2 *d = buf + s * N + q * L;
        d[bplace(p0, 0)] = in[i][0];
#pragma unroll
        for (int e = 1; e < RL; ++e)
          d[bplace(p0, e)] = p0 > 0 ? ctw<INV>(in[i][e], tw[TW1 + (p0 - 1) * R2 + e]) : in[i][e];
      }
    }
    wave_sync();
    double2 x[NI1][R1];
    if (lane < 56) {
#pragma unroll
      for (int i = 0; i < NI1; ++i) {
        const int it = lane + 56 * i, s = it / (7 * R2), q = (it / R2) % 7, j0 = it % R2;
#pragma unroll
        for (int p = 0; p < R1; ++p)
          x[i][p] = R2 > 1 ? buf[s * N + q * L + bplace(p, j0)] : in[i % NIL][p % RL];
        Dft<R1, INV>::run(x[i]);
      }
    }
    wave_sync();
    if (lane < 56) {
#pragma unroll
      for (int i = 0; i < NI1; ++i) {
        const int it = lane + 56 * i, s = it / (7 * R2), q = (it / R2) % 7, j0 = it % R2;
#pragma unroll
        for (int r = 0; r < R1; ++r) buf[s * N + q * L + j0 + R2 * r] = x[i][r];
      }
    }
    wave_sync();
#pragma unroll
    for (int a = 0; a < V; ++a) {
      const int j = (lane % (L < 64 ? L : 64)) + 64 * a, s = L < 64 ? lane / L : 0;
      const double2 *d = buf + s * N + j;
      v[a][0] = d[0];
#pragma unroll
      for (int q = 1; q < 7; ++q) v[a][q] = ctw<INV>(d[q * L], tw[(q - 1) * L + j]);
      Dft<7, INV>::run(v[a]);
    }
    wave_sync();
  }
};

__device__ __forceinline__ double luma_at(const float *frame, size_t plane, size_t off) {
  return 0.299 * (double)frame[off] + 0.587 * (double)frame[plane + off] +
         0.114 * (double)frame[2 * plane + off];
}

// Element (y, k) of an item's half-spectra of hw columns: strips of 8 columns.
__device__ __forceinline__ size_t strip_at(int H, int hw, int y, int k) {
  const int k0 = k & ~7;
  return (size_t)k0 * H + (size_t)y * min(8, hw - k0) + (k - k0);
}

// ------------------------------------------------------------------------- k_pc_rows
// Each side of a pair is a real map ([B][H][W] float64) or a frame's luma ([B][3][H][W]
// float32 RGB), or all zero when both are null.
struct PcIn {
  const float *rgb_prev, *rgb_cur;
  const double *map_prev, *map_cur;
};

__device__ __forceinline__ double pc_input(const float *rgb, const double *map, int b, size_t plane,
                                           size_t off) {
  if (map) return map[(size_t)b * plane + off];
  if (rgb) return luma_at(rgb + (size_t)b * 3 * plane, plane, off);
  return 0.0;
}

// A wave's unit is S row pairs of one side of one item; waves step over all units.
template <int L>
__global__ __launch_bounds__(kPcThreads) void k_pc_rows(PcIn in, int H, int B, PixWs ws) {
  using F = Fft<L>;
  constexpr int W = F::N, hw = W / 2 + 1;
  __shared__ double2 lds[kPcWaves * F::PTS];
  __shared__ double2 tw[F::TW];
  F::table(tw);
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double2 *buf = lds + w * F::PTS;
  const size_t plane = (size_t)H * W;
  const int groups = (H / 2 + F::S - 1) / F::S;
  const int units = 2 * B * groups;
  const int s = L < 64 ? lane / L : 0, j = lane % (L < 64 ? L : 64);
  for (int u = blockIdx.x * kPcWaves + w; u < units; u += gridDim.x * kPcWaves) {
    const int g = u % groups, f = (u / groups) & 1, b = u / (2 * groups);
    const float *rgb = f ? in.rgb_cur : in.rgb_prev;
    const double *map = f ? in.map_cur : in.map_prev;
    const int y = 2 * (g * F::S + s);
    const bool row = y < H;                    // H is even: both rows or neither
    double2 v[F::V][7];
#pragma unroll
    for (int a = 0; a < F::V; ++a)
#pragma unroll
      for (int r = 0; r < 7; ++r) {
        const size_t off = (size_t)(row ? y : 0) * W + j + 64 * a + L * r;
        v[a][r] = make_double2(pc_input(rgb, map, b, plane, off), pc_input(rgb, map, b, plane, off + W));
      }
    double2 z[F::NIL][F::RL];
    F::template dif<false>(v, z, buf, tw);
    if (lane < 56) {
#pragma unroll
      for (int i = 0; i < F::NIL; ++i)
#pragma unroll
        for (int e = 0; e < F::RL; ++e) {
          int sq, k;
          F::where(lane + 56 * i, e, sq, k);
          buf[sq * W + k] = z[i][e];
        }
    }
    wave_sync();
    // Z = A + i B of the two rows: A = (Z_k + conj Z_{W-k}) / 2, B = -i (Z_k - conj Z_{W-k}) / 2
    double2 *o = (f ? ws.sb : ws.sa) + (size_t)b * H * hw;
    for (int e = lane; e < F::S * hw; e += 64) {
      const int sq = e / hw, k = e - sq * hw;
      const int yo = 2 * (g * F::S + sq);
      if (yo >= H) continue;
      const double2 a = buf[sq * W + k], c = buf[sq * W + (k ? W - k : 0)];
      o[strip_at(H, hw, yo, k)] = make_double2(0.5 * (a.x + c.x), 0.5 * (a.y - c.y));
      o[strip_at(H, hw, yo + 1, k)] = make_double2(0.5 * (a.y + c.y), 0.5 * (c.x - a.x));
    }
    wave_sync();
  }
}

// ------------------------------------------------------------------------- k_pc_cols
// A workgroup takes 8 S columns (S strips), a wave S of them.  Strips come and go through
// LDS, element (y, column c of the strip) at y 8 + (c + y) % 8, which lets a column's
// consecutive rows meet different banks.
constexpr int kPcColThreads = 512;

typedef double vd2 __attribute__((ext_vector_type(2)));
template <int L>
struct ColStage {
  using F = Fft<L>;
  static constexpr int H = F::N;
  static constexpr int LD = 8 * F::PTS / kPcColThreads;          // elements per thread
  // LDS place of element e of the workgroup's strips of ncol columns
  static __device__ __forceinline__ int place(int e, int ncol) {
    const int t8 = e / (8 * H), x = e - t8 * 8 * H;
    const int cw = ncol == 8 * F::S ? 8 : min(8, ncol - 8 * t8);
    const int y = cw == 8 ? x >> 3 : x / cw, c = cw == 8 ? x & 7 : x - y * cw;
    return t8 * 8 * H + y * 8 + ((c + y) & 7);
  }
  // A workgroup whose strips are all there moves them through registers, so that the next
  // ones are in flight while the last are transformed; the one with the item's last columns
  // copies them when it needs them.
  static __device__ __forceinline__ void fetch(const double2 *g, int ncol, vd2 (&r)[LD]) {
    if (ncol < 8 * F::S) return;
#pragma unroll
    for (int i = 0; i < LD; ++i) r[i] = reinterpret_cast<const vd2 *>(g)[threadIdx.x + kPcColThreads * i];
  }
  static __device__ __forceinline__ void put(const double2 *g, const vd2 (&r)[LD], int ncol, double2 *lds) {
    if (ncol < 8 * F::S) {
      // Short columns: the last workgroup of an item is often its only one, so its loads go out
      // four at a time (112 x 112: 21.5 -> 19.8 us in both passes).  Of long ones it has a column
      // or a few, and extra loads would cost more (64 pairs of 448 x 448: 358 -> 362 us).
      constexpr int U = F::S > 1 ? 4 : 1;
      const int n = ncol * H;
      for (int e0 = threadIdx.x; e0 < n; e0 += U * kPcColThreads) {
        vd2 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = reinterpret_cast<const vd2 *>(g)[min(e0 + u * kPcColThreads, n - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (e0 + u * kPcColThreads < n) reinterpret_cast<vd2 *>(lds)[place(e0 + u * kPcColThreads, ncol)] = v[u];
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < LD; ++i)
      reinterpret_cast<vd2 *>(lds)[place(threadIdx.x + kPcColThreads * i, 8 * F::S)] = r[i];
  }
  static __device__ __forceinline__ int column(int c, int y) {
    return (c >> 3) * 8 * H + y * 8 + (((c & 7) + y) & 7);
  }
};

// mag (rotation): also the high-pass weighted magnitudes of both spectra,
// mag[b][side][ky][kx] = (1 - X)(2 - X) |F|, X = cos(pi f_y) cos(pi f_x) (f the signed
// frequency in cycles per sample).
template <int L, bool MAG>
__global__ __launch_bounds__(kPcColThreads) void k_pc_cols_fwd(int W, PixWs ws, double *mag) {
  using F = Fft<L>;
  using C = ColStage<L>;
  constexpr int H = F::N;
  __shared__ double2 lds[8 * F::PTS];
  __shared__ double2 tw[F::TW];
  __shared__ double red[8];
  const int b = blockIdx.y, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int hw = W / 2 + 1;
  const int c0 = blockIdx.x * 8 * F::S, ncol = min(8 * F::S, hw - c0);
  const size_t base = (size_t)b * H * hw + (size_t)c0 * H;
  const double2 *ga = ws.sa + base, *gb = ws.sb + base;
  F::table(tw);
  double2 *buf = lds + w * F::PTS;
  const int s = L < 64 ? lane / L : 0, j = lane % (L < 64 ? L : 64);
  vd2 r[C::LD];                                 // the next strips, in flight
  double2 v[F::V][7], za[F::NIL][F::RL], zb[F::NIL][F::RL];
  C::fetch(ga, ncol, r);
  C::put(ga, r, ncol, lds);
  __syncthreads();
  C::fetch(gb, ncol, r);
#pragma unroll
  for (int a = 0; a < F::V; ++a)
#pragma unroll
    for (int q = 0; q < 7; ++q) v[a][q] = lds[C::column(w * F::S + s, j + 64 * a + L * q)];
  __syncthreads();                              // the strips are in registers
  F::template dif<false>(v, za, buf, tw);
  __syncthreads();                              // every wave is done with its LDS
  C::put(gb, r, ncol, lds);
  __syncthreads();
#pragma unroll
  for (int a = 0; a < F::V; ++a)
#pragma unroll
    for (int q = 0; q < 7; ++q) v[a][q] = lds[C::column(w * F::S + s, j + 64 * a + L * q)];
  __syncthreads();
  F::template dif<false>(v, zb, buf, tw);
  double mx = 0.0;
  if (lane < 56) {
#pragma unroll
    for (int i = 0; i < F::NIL; ++i)
#pragma unroll
      for (int e = 0; e < F::RL; ++e) {
        const int it = lane + 56 * i, c = w * F::S + it / F::IPS;
        if (c >= ncol) continue;
        const double2 f1 = za[i][e], f2 = zb[i][e];
        if (MAG) {
          int sq, ky;
          F::where(it, e, sq, ky);
          const int kx = c0 + c;
          const double fy = (double)(2 * ky < H ? ky : ky - H) / (double)H;
          const double fx = (double)(2 * kx < W ? kx : kx - W) / (double)W;
          const double X = cospi(fy) * cospi(fx);
          const double hp = (1.0 - X) * (2.0 - X);
          const size_t o = ((size_t)b * 2 * H + ky) * hw + kx;
          mag[o] = hp * sqrt(f1.x * f1.x + f1.y * f1.y);
          mag[o + (size_t)H * hw] = hp * sqrt(f2.x * f2.x + f2.y * f2.y);
        }
        const double xr = f1.x * f2.x + f1.y * f2.y;
        const double xi = f1.y * f2.x - f1.x * f2.y;
        ws.sa[base + (size_t)c * H + e * F::IPS + it % F::IPS] = make_double2(xr, xi);
        mx = fmax(mx, sqrt(xr * xr + xi * xi));
      }
  }
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
  if (lane == 0) red[w] = mx;
  __syncthreads();
  if (t == 0) {
    double m = red[0];
    for (int i = 1; i < 8; ++i) m = fmax(m, red[i]);
    ws.bmax[(size_t)b * gridDim.x + blockIdx.x] = m;
  }
}

template <int L>
__global__ __launch_bounds__(kPcColThreads) void k_pc_cols_inv(int W, PixWs ws) {
  using F = Fft<L>;
  using C = ColStage<L>;
  constexpr int H = F::N;
  __shared__ double2 lds[8 * F::PTS];
  __shared__ double2 tw[F::TW];
  const int b = blockIdx.y, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int hw = W / 2 + 1;
  const int c0 = blockIdx.x * 8 * F::S, ncol = min(8 * F::S, hw - c0);
  double2 *sa = ws.sa + (size_t)b * H * hw + (size_t)c0 * H;
  double2 z[F::NIL][F::RL];
#pragma unroll
  for (int i = 0; i < F::NIL; ++i)
#pragma unroll
    for (int e = 0; e < F::RL; ++e) {
      const int it = lane + 56 * i, c = w * F::S + it / F::IPS;
      z[i][e] = lane < 56 && c < ncol ? sa[(size_t)c * H + e * F::IPS + it % F::IPS]
                                      : make_double2(0.0, 0.0);
    }
  // the item's largest |X| (every wave for itself)
  double gmax = 0.0;
  for (int i = lane; i < (int)gridDim.x; i += 64) gmax = fmax(gmax, ws.bmax[(size_t)b * gridDim.x + i]);
  for (int o = 32; o > 0; o >>= 1) gmax = fmax(gmax, __shfl_xor(gmax, o));
  F::table(tw);
#pragma unroll
  for (int i = 0; i < F::NIL; ++i)
#pragma unroll
    for (int e = 0; e < F::RL; ++e) {
      const double2 x = z[i][e];
      const double m = sqrt(x.x * x.x + x.y * x.y);
      z[i][e] = gmax > 0.0 && m > 1e-9 * gmax ? make_double2(x.x / m, x.y / m) : make_double2(0.0, 0.0);
    }
  __syncthreads();
  double2 v[F::V][7];
  F::template dit<true>(z, v, lds + w * F::PTS, tw);
  __syncthreads();                              // every wave is done with its LDS
  const int s = L < 64 ? lane / L : 0, j = lane % (L < 64 ? L : 64);
#pragma unroll
  for (int a = 0; a < F::V; ++a)
#pragma unroll
    for (int r = 0; r < 7; ++r) lds[C::column(w * F::S + s, j + 64 * a + L * r)] = v[a][r];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < C::LD; ++i) {
    const int e = t + kPcColThreads * i;
    if (e < ncol * H) sa[e] = lds[C::place(e, ncol)];
  }
}

// --------------------------------------------------------------------- k_pc_rows_inv
// A wave's unit is S row pairs of one item.  The columns 0 and W/2 of a Hermitian row are
// real: their imaginary parts (rounding noise) are left out, as the real part of the
// inverse would leave them out.
template <int L>
__global__ __launch_bounds__(kPcThreads) void k_pc_rows_inv(int H, int B, PixWs ws,
                                                            double *__restrict__ resp) {
  using F = Fft<L>;
  constexpr int W = F::N, hw = W / 2 + 1;
  __shared__ double2 lds[kPcWaves * F::PTS];
  __shared__ double2 tw[F::TW];
  F::table(tw);
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double2 *buf = lds + w * F::PTS;
  const int groups = (H / 2 + F::S - 1) / F::S;
  const int units = B * groups;
  const int s = L < 64 ? lane / L : 0, j = lane % (L < 64 ? L : 64);
  const double hwn = (double)H * (double)W;
  for (int u = blockIdx.x * kPcWaves + w; u < units; u += gridDim.x * kPcWaves) {
    const int g = u % groups, b = u / groups;
    const double2 *G = ws.sa + (size_t)b * H * hw;
    const int y = min(2 * (g * F::S + s), H - 2);     // rows past the last pair: not stored
    double2 v[F::V][7];
#pragma unroll
    for (int a = 0; a < F::V; ++a)
#pragma unroll
      for (int r = 0; r < 7; ++r) {
        const int n = j + 64 * a + L * r, k = 2 * n <= W ? n : W - n;
        double2 g1 = G[strip_at(H, hw, y, k)], g2 = G[strip_at(H, hw, y + 1, k)];
        if (k == 0 || 2 * k == W) g1.y = g2.y = 0.0;
        if (k != n) {
          g1.y = -g1.y;
          g2.y = -g2.y;
        }
        v[a][r] = make_double2(g1.x - g2.y, g1.y + g2.x);
      }
    double2 z[F::NIL][F::RL];
    F::template dif<true>(v, z, buf, tw);
    if (lane < 56) {
#pragma unroll
      for (int i = 0; i < F::NIL; ++i)
#pragma unroll
        for (int e = 0; e < F::RL; ++e) {
          int sq, k;
          F::where(lane + 56 * i, e, sq, k);
          buf[sq * W + k] = make_double2(z[i][e].x / hwn, z[i][e].y / hwn);
        }
    }
    wave_sync();
    // 64 / S lanes take the two rows of a sequence
    constexpr int GL = 64 / F::S, NX = W / GL;
    const int sq = lane / GL, gl = lane % GL, yo = 2 * (g * F::S + sq);
    double2 r[NX];
    double best[2] = {-INFINITY, -INFINITY};
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      r[i] = buf[sq * W + gl + GL * i];
      if (r[i].x > best[0]) best[0] = r[i].x;
      if (r[i].y > best[1]) best[1] = r[i].y;
    }
    if (resp && yo < H) {
      double *row = resp + ((size_t)b * H + yo) * W;
#pragma unroll
      for (int i = 0; i < NX; ++i) {
        row[gl + GL * i] = r[i].x;
        row[W + gl + GL * i] = r[i].y;
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int o = GL / 2; o > 0; o >>= 1) best[h] = fmax(best[h], __shfl_xor(best[h], o));
    // the first element of each row that reaches its maximum (a row of NaN: element 0)
    int arg[2] = {W, W};
#pragma unroll
    for (int i = NX - 1; i >= 0; --i) {
      if (r[i].x >= best[0] - kPcTie * fabs(best[0])) arg[0] = gl + GL * i;
      if (r[i].y >= best[1] - kPcTie * fabs(best[1])) arg[1] = gl + GL * i;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int o = GL / 2; o > 0; o >>= 1) arg[h] = min(arg[h], __shfl_xor(arg[h], o));
      if (arg[h] >= W) arg[h] = 0;
    }
    if (gl < 2 && yo < H) {
      ws.rowmax[(size_t)b * H + yo + gl] = gl ? best[1] : best[0];
      ws.rowarg[(size_t)b * H + yo + gl] = gl ? arg[1] : arg[0];
    }
    wave_sync();
  }
}

// ------------------------------------------------------------------------- k_pc_peak
__device__ __forceinline__ double parabolic(double a, double c0, double c) {
  const double den = a - 2.0 * c0 + c;
  return den >= 0.0 ? 0.0 : (a - c) / (2.0 * den);
}

__device__ __forceinline__ int token_round(double d, int tp) {
  const double q = fabs(d) / (double)tp;
  const int k = (int)floor(q + 0.5);
  return d >= 0.0 ? k : -k;
}

// The four neighbours of the peak are the surface's values there, summed from the row
// spectra of its row and of the rows above and below:
// r[y][x] = (G[y][0] + (-1)^x G[y][W/2] + 2 Re sum_{0<k<W/2} G[y][k] e^{2 pi i k x / W}) / (H W).
__global__ __launch_bounds__(kPcThreads) void k_pc_peak(int H, int W, PixWs ws,
                                                        double *__restrict__ shift_px,
                                                        int32_t *__restrict__ peak,
                                                        int32_t *__restrict__ tok_shift, int tp,
                                                        int zero_shift) {
  __shared__ double bv[kPcWaves];
  __shared__ int by[kPcWaves];
  __shared__ double n[4];
  const int b = blockIdx.x, t = threadIdx.x;
  constexpr int NR = (kPcMaxN + kPcThreads - 1) / kPcThreads;
  double rm[NR];
  int ra[NR];
  double v = -INFINITY;
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int y = t + kPcThreads * i;
    rm[i] = y < H ? ws.rowmax[(size_t)b * H + y] : -INFINITY;
    ra[i] = y < H ? ws.rowarg[(size_t)b * H + y] : 0;
    v = fmax(v, rm[i]);
  }
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
  if ((t & 63) == 0) bv[t >> 6] = v;
  __syncthreads();
  for (int i = 0; i < kPcWaves; ++i) v = fmax(v, bv[i]);
  // the first row that reaches it, and that row's first element (a surface of NaN: element 0),
  // as row * 1024 + column
  const double least = v - kPcTie * fabs(v);
  int at = 0x7fffffff;
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int y = t + kPcThreads * i;
    if (y < H && rm[i] >= least) at = min(at, y * 1024 + ra[i]);
  }
  for (int o = 32; o > 0; o >>= 1) at = min(at, __shfl_xor(at, o));
  if ((t & 63) == 0) by[t >> 6] = at;
  __syncthreads();
  for (int i = 0; i < kPcWaves; ++i) at = min(at, by[i]);
  static_assert(kPcMaxN <= 1024, "a column in 10 bits");
  if (at >= H * 1024) at = 0;
  const int ki = at / 1024, kj = at % 1024;
  const int hw = W / 2 + 1;
  const double2 *G = ws.sa + (size_t)b * H * hw;
  const int yu = (ki - 1 + H) % H, yd = (ki + 1) % H;
  // each wave sums one of them: up, down, left, right
  static_assert(kPcWaves == 4, "a wave per neighbour");
  const int wv = t >> 6;
  const int yn = wv == 0 ? yu : wv == 1 ? yd : ki;
  const int xn = wv < 2 ? kj : wv == 2 ? (kj - 1 + W) % W : (kj + 1) % W;
  double sum = 0.0;
  for (int k = t & 63; k < hw; k += 64) {
    const double2 g = G[strip_at(H, hw, yn, k)];
    double s, c;
    sincospi(2.0 * (double)((long)k * xn % W) / (double)W, &s, &c);
    sum += k == 0 || 2 * k == W ? g.x * c : 2.0 * (g.x * c - g.y * s);
  }
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if ((t & 63) == 0) n[wv] = sum / ((double)H * (double)W);
  __syncthreads();
  if (t != 0) return;
  const int pi = ki <= H / 2 ? ki : ki - H;
  const int pj = kj <= W / 2 ? kj : kj - W;
  const double di = pi + parabolic(n[0], v, n[1]);
  const double dj = pj + parabolic(n[2], v, n[3]);
  if (shift_px) {
    shift_px[2 * b] = di;
    shift_px[2 * b + 1] = dj;
  }
  if (peak) {
    peak[2 * b] = pi;
    peak[2 * b + 1] = pj;
  }
  if (tok_shift) {
    tok_shift[2 * b] = zero_shift ? 0 : token_round(di, tp);
    tok_shift[2 * b + 1] = zero_shift ? 0 : token_round(dj, tp);
  }
}

// ----------------------------------------------------------------- rotation (log-polar)
// Log-polar samples of both frames' weighted magnitude spectra: angle i pi / NT, radius
// R^(j / NR), R = min(H, W) / 2 - 1, bilinear over the half-plane kx in [0, W/2] (a point
// with kx outside it is read at its mirror -k: the magnitudes of real frames are centrally
// symmetric).  lp[side][b][i][j] (side 0: previous frame), so each side is a batch of
// NT x NR maps.
__device__ __forceinline__ double mag_at(const double *m, int H, int W, int ky, int kx) {
  const int hw = W / 2 + 1;
  kx %= W;
  if (kx < 0) kx += W;
  ky %= H;
  if (ky < 0) ky += H;
  if (kx >= hw) {            // the mirror -k
    kx = W - kx;
    ky = ky == 0 ? 0 : H - ky;
  }
  return m[(size_t)ky * hw + kx];
}

__global__ __launch_bounds__(kPcThreads) void k_lp_sample(const double *__restrict__ mag, int H,
                                                          int W, int NT, int NR,
                                                          double *__restrict__ lp) {
  const int i = blockIdx.x, b = blockIdx.y;
  const int hw = W / 2 + 1;
  const double R = (double)min(H, W) / 2.0 - 1.0;
  double sn, cs;
  sincospi((double)i / (double)NT, &sn, &cs);
  for (int e = threadIdx.x; e < 2 * NR; e += blockDim.x) {
    const int side = e / NR, j = e - side * NR;
    const double r = pow(R, (double)j / (double)NR);
    const double fy = r * sn, fx = r * cs;
    const double y0 = floor(fy), x0 = floor(fx);
    const double wy = fy - y0, wx = fx - x0;
    const int iy = (int)y0, ix = (int)x0;
    const double *m = mag + ((size_t)b * 2 + side) * H * hw;
    const double v = (1.0 - wy) * (1.0 - wx) * mag_at(m, H, W, iy, ix) +
                     (1.0 - wy) * wx * mag_at(m, H, W, iy, ix + 1) +
                     wy * (1.0 - wx) * mag_at(m, H, W, iy + 1, ix) +
                     wy * wx * mag_at(m, H, W, iy + 1, ix + 1);
    lp[(((size_t)side * gridDim.y + b) * NT + i) * NR + j] = v;
  }
}

// The current frame's luma rotated back by the estimated angle, a = -dtheta pi / NT
// (dtheta: the angular coordinate of the log-polar correlation peak):
// yrot(q) = Y(R(a)(q - c) + c), bilinear, 0 outside the frame.
__global__ __launch_bounds__(kPcThreads) void k_derotate(const float *__restrict__ cur, int H,
                                                         int W, const double *__restrict__ dth,
                                                         int NT, double *__restrict__ yrot,
                                                         double *__restrict__ angle) {
  const int y = blockIdx.x, b = blockIdx.y;
  const double a = -dth[2 * b] * M_PI / (double)NT;
  if (angle && y == 0 && threadIdx.x == 0) angle[b] = a;
  double sa, ca;
  sincos(a, &sa, &ca);
  const double cy = (H - 1) / 2.0, cx = (W - 1) / 2.0;
  const size_t plane = (size_t)H * W;
  const float *fr = cur + (size_t)b * 3 * plane;
  for (int x = threadIdx.x; x < W; x += blockDim.x) {
    const double qy = y - cy, qx = x - cx;
    const double sy = qx * sa + qy * ca + cy, sx = qx * ca - qy * sa + cx;
    const double y0 = floor(sy), x0 = floor(sx);
    const double wy = sy - y0, wx = sx - x0;
    const int iy = (int)y0, ix = (int)x0;
    double v = 0.0;
    for (int u = 0; u < 2; ++u)
      for (int w2 = 0; w2 < 2; ++w2) {
        const int yy = iy + u, xx = ix + w2;
        if (yy < 0 || yy >= H || xx < 0 || xx >= W) continue;
        const double wgt = (u ? wy : 1.0 - wy) * (w2 ? wx : 1.0 - wx);
        v += wgt * luma_at(fr, plane, (size_t)yy * W + xx);
      }
    yrot[(size_t)b * plane + (size_t)y * W + x] = v;
  }
}

}  // namespace

bool pix_size_ok(int n) {
  if (n < 14 || n > kPcMaxN || n % 7) return false;
  const int p = n / 7;
  return (p & (p - 1)) == 0;
}

bool pix_rot_size_ok(int H, int W) {
  return pix_size_ok(H) && pix_size_ok(W) && pix_size_ok(std::min(H, W) / 2);
}

namespace {
// Workspace parts in order: sa, sb, rowmax, rowarg, bmax, shift_px, then with rotation
// mag [B][2][H][W/2 + 1], lp [2][B][H][min(H, W) / 2], yrot [B][H][W].
template <typename F>
void pix_parts(long B, long H, long W, bool rot, F &&take) {
  const long hw = W / 2 + 1;
  // bmax: a column workgroup takes 8 columns or more; the part has been one value per 2 columns,
  // and what fits a scratch of fixed size stays what it was
  const long ncb = (hw + 1) / 2;
  take(0, (size_t)B * H * hw * sizeof(double2));
  take(1, (size_t)B * H * hw * sizeof(double2));
  take(2, (size_t)B * H * sizeof(double));
  take(3, (size_t)B * H * sizeof(int));
  take(4, (size_t)B * ncb * sizeof(double));
  take(5, (size_t)B * 2 * sizeof(double));
  if (rot) {
    take(6, (size_t)B * 2 * H * hw * sizeof(double));
    take(7, (size_t)B * 2 * H * (std::min(H, W) / 2) * sizeof(double));
    take(8, (size_t)B * H * W * sizeof(double));
  }
}
size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }
}  // namespace

size_t pix_ws_bytes(long B, long H, long W, bool rot) {
  size_t n = 0;
  pix_parts(B, H, W, rot, [&](int, size_t bytes) { n += al256(bytes); });
  return n;
}

PixWs pix_ws_at(void *base, long B, long H, long W, bool rot) {
  unsigned char *p = static_cast<unsigned char *>(base);
  PixWs ws;
  pix_parts(B, H, W, rot, [&](int part, size_t bytes) {
    switch (part) {
      case 0: ws.sa = reinterpret_cast<double2 *>(p); break;
      case 1: ws.sb = reinterpret_cast<double2 *>(p); break;
      case 2: ws.rowmax = reinterpret_cast<double *>(p); break;
      case 3: ws.rowarg = reinterpret_cast<int *>(p); break;
      case 4: ws.bmax = reinterpret_cast<double *>(p); break;
      case 5: ws.shift_px = reinterpret_cast<double *>(p); break;
      case 6: ws.mag = reinterpret_cast<double *>(p); break;
      case 7: ws.lp = reinterpret_cast<double *>(p); break;
      case 8: ws.yrot = reinterpret_cast<double *>(p); break;
    }
    p += al256(bytes);
  });
  return ws;
}

namespace {
// The row kernels' waves step over the units: enough workgroups for four on every CU, or
// one wave per unit when there are fewer.
constexpr int kPcRowGroups = 1024;
template <int L>
void launch_rows(const PcIn &in, int H, int B, const PixWs &ws, hipStream_t st) {
  const long units = 2L * B * ((H / 2 + Fft<L>::S - 1) / Fft<L>::S);
  const unsigned grid = (unsigned)std::min<long>(kPcRowGroups, (units + kPcWaves - 1) / kPcWaves);
  hipLaunchKernelGGL(k_pc_rows<L>, dim3(grid), dim3(kPcThreads), 0, st, in, H, B, ws);
}
template <int L>
void launch_rows_inv(int H, int B, const PixWs &ws, double *resp, hipStream_t st) {
  const long units = (long)B * ((H / 2 + Fft<L>::S - 1) / Fft<L>::S);
  const unsigned grid = (unsigned)std::min<long>(kPcRowGroups, (units + kPcWaves - 1) / kPcWaves);
  hipLaunchKernelGGL(k_pc_rows_inv<L>, dim3(grid), dim3(kPcThreads), 0, st, H, B, ws, resp);
}
template <int L>
void launch_cols(int W, int B, const PixWs &ws, bool mag_only, hipStream_t st) {
  const int hw = W / 2 + 1, nc = 8 * Fft<L>::S;
  const dim3 grid((unsigned)((hw + nc - 1) / nc), (unsigned)B);
  if (mag_only) {
    hipLaunchKernelGGL((k_pc_cols_fwd<L, true>), grid, dim3(kPcColThreads), 0, st, W, ws, ws.mag);
  } else {
    hipLaunchKernelGGL((k_pc_cols_fwd<L, false>), grid, dim3(kPcColThreads), 0, st, W, ws,
                       (double *)nullptr);
    hipLaunchKernelGGL(k_pc_cols_inv<L>, grid, dim3(kPcColThreads), 0, st, W, ws);
  }
}
// f(std::integral_constant<int, n / 7>) for a transform length n = 7 2^k (pix_size_ok)
template <typename Fn>
void with_length(int n, Fn &&f) {
  switch (n / 7) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 16: f(std::integral_constant<int, 16>{}); break;
    case 32: f(std::integral_constant<int, 32>{}); break;
    case 64: f(std::integral_constant<int, 64>{}); break;
    default: f(std::integral_constant<int, 128>{}); break;
  }
}

// One phase correlation of B pairs of H x W inputs.  mag_only: the row transforms and
// the forward column pass only, with the weighted magnitudes written to ws.mag.
fc_status pc_run(fc_ctx *ctx, const PixWs &ws, PcIn in, int B, int H, int W, bool mag_only,
                 double *shift_px, int32_t *peak, double *resp, int32_t *tok_shift, int tp,
                 bool zero_shift, hipStream_t st) {
  {
    ProfScope ps(ctx, st, "fc_pc_rows");
    with_length(W, [&](auto l) { launch_rows<decltype(l)::value>(in, H, B, ws, st); });
    FC_LAUNCH_OK(st, "k_pc_rows");
  }
  {
    ProfScope ps(ctx, st, "fc_pc_cols");
    with_length(H, [&](auto l) { launch_cols<decltype(l)::value>(W, B, ws, mag_only, st); });
    FC_LAUNCH_OK(st, "k_pc_cols");
  }
  if (mag_only) return FC_OK;
  {
    ProfScope ps(ctx, st, "fc_pc_rows_inv");
    with_length(W, [&](auto l) { launch_rows_inv<decltype(l)::value>(H, B, ws, resp, st); });
    FC_LAUNCH_OK(st, "k_pc_rows_inv");
  }
  {
    ProfScope ps(ctx, st, "fc_pc_peak");
    hipLaunchKernelGGL(k_pc_peak, dim3((unsigned)B), dim3(kPcThreads), 0, st, H, W, ws,
                       shift_px ? shift_px : ws.shift_px, peak, tok_shift, tp, zero_shift ? 1 : 0);
    FC_LAUNCH_OK(st, "k_pc_peak");
  }
  return FC_OK;
}
}  // namespace

fc_status launch_pixel_pc(fc_ctx *ctx, const PixWs &ws, const float *prev, const float *cur,
                          int B, int H, int W, double *shift_px, int32_t *peak, double *resp,
                          int32_t *tok_shift, int tp, bool zero_shift, hipStream_t st) {
  if (!pix_size_ok(H) || !pix_size_ok(W))
    return fail(FC_ERR_UNSUPPORTED, "pixel phase correlation: H=%d, W=%d must be 7 * 2^k, 14..%d",
                H, W, kPcMaxN);
  return pc_run(ctx, ws, PcIn{prev, cur, nullptr, nullptr}, B, H, W, false, shift_px, peak, resp,
                tok_shift, tp, zero_shift, st);
}

fc_status launch_pixel_pc_rot(fc_ctx *ctx, const PixWs &ws, const float *prev, const float *cur,
                              int B, int H, int W, double *angle, double *shift_px,
                              int32_t *tok_shift, int tp, bool zero_shift, hipStream_t st) {
  if (!pix_rot_size_ok(H, W) || !ws.mag)
    return fail(FC_ERR_UNSUPPORTED, "rotation phase correlation: H=%d, W=%d must be 7 * 2^k with "
                "min(H, W) >= 28", H, W);
  const int NT = H, NR = std::min(H, W) / 2;
  fc_status s;
  // 1. weighted magnitude spectra of both frames
  if ((s = pc_run(ctx, ws, PcIn{prev, cur, nullptr, nullptr}, B, H, W, true, nullptr, nullptr,
                  nullptr, nullptr, 1, false, st)) != FC_OK)
    return s;
  // 2. their log-polar samples, correlated: the angular offset of the peak
  {
    ProfScope ps(ctx, st, "fc_lp_sample");
    hipLaunchKernelGGL(k_lp_sample, dim3((unsigned)NT, (unsigned)B), dim3(kPcThreads), 0, st,
                       (const double *)ws.mag, H, W, NT, NR, ws.lp);
    FC_LAUNCH_OK(st, "k_lp_sample");
  }
  if ((s = pc_run(ctx, ws, PcIn{nullptr, nullptr, ws.lp, ws.lp + (size_t)B * NT * NR}, B, NT, NR,
                  false, ws.shift_px, nullptr, nullptr, nullptr, 1, false, st)) != FC_OK)
    return s;
  // 3. the current frame rotated back, then the displacement of the image centre
  {
    ProfScope ps(ctx, st, "fc_derotate");
    hipLaunchKernelGGL(k_derotate, dim3((unsigned)H, (unsigned)B), dim3(kPcThreads), 0, st, cur, H,
                       W, (const double *)ws.shift_px, NT, ws.yrot, angle);
    FC_LAUNCH_OK(st, "k_derotate");
  }
  return pc_run(ctx, ws, PcIn{prev, nullptr, nullptr, ws.yrot}, B, H, W, false, shift_px, nullptr,
                nullptr, tok_shift, tp, zero_shift, st);
}

}  // namespace fc
