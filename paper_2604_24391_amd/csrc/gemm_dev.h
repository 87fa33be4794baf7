// Device code that the GEMM kernels share: LDS DMA loads and their waits, the swizzle of
// staged rows, tile order over the XCDs, and the rows of several items packed into one range.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "fc_internal.h"

namespace fc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int KS = kGemmBK;                 // 64 K values per step
constexpr int RB = KS * 2;                  // bytes per staged operand row
constexpr int kMMaxItems = 1024;            // batch items the packed row map holds

__device__ __forceinline__ float bf2f(uint16_t u) { return __uint_as_float((uint32_t)u << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {
  // round to nearest even (inputs are finite)
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Device-side counts and ids come from fc_select; clamp them so that a caller
// passing anything else can never make a kernel leave its buffers.
// Null counts and ids (the trailing-text rows) mean every token of the region, in order.
__device__ __forceinline__ int n_valid(const int32_t *nrec, int b, int N) {
  return nrec ? min(max(nrec[b], 0), N) : N;
}
__device__ __forceinline__ int tok_of(const int32_t *idx, long slot, int N) {
  return idx ? min(max(idx[slot], 0), N - 1) : (int)(slot % N);
}

// Workgroup id -> tile id so that each XCD (workgroups are dealt round-robin over
// the 8 XCDs) works on a contiguous range of tiles.
__device__ __forceinline__ int xcd_tile(int w, int total) {
  const int per = total / 8;
  if (w >= per * 8) return w;
  return (w & 7) * per + (w >> 3);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t lds_addr(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}
// LDS DMA of 16 B per lane to lds + 16 * lane (lds must be wave-uniform).  M0 is
// reserved to the compiler, so the asm restores it.
__device__ __forceinline__ void dma16(const void *gp, uint32_t lds) {
  const uint32_t l = __builtin_amdgcn_readfirstlane(lds);
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %2\n\t"
      "global_load_lds_dwordx4 %1, off\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "v"(gp), "s"(l)
      : "memory");
}
// The same for data read once (streamed weights): the non-temporal hint keeps such
// lines from displacing the re-read activation rows in L2.
__device__ __forceinline__ void dma16_nt(const void *gp, uint32_t lds) {
  const uint32_t l = __builtin_amdgcn_readfirstlane(lds);
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %2\n\t"
      "global_load_lds_dwordx4 %1, off nt\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "v"(gp), "s"(l)
      : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt holds at most 63 outstanding loads");
  __builtin_amdgcn_s_waitcnt(0x3F70 | (N & 0xF) | ((N >> 4) << 14));
}
// wait until at most n (wave-uniform, < 64) of this wave's loads are outstanding
__device__ __forceinline__ void wait_vm_rt(int n) {
  switch (n) {
#define FC_W1(x) case x: wait_vm<x>(); break;
#define FC_W8(x) FC_W1(x) FC_W1(x + 1) FC_W1(x + 2) FC_W1(x + 3) FC_W1(x + 4) FC_W1(x + 5) FC_W1(x + 6) FC_W1(x + 7)
    FC_W8(0) FC_W8(8) FC_W8(16) FC_W8(24) FC_W8(32) FC_W8(40) FC_W8(48) FC_W8(56)
#undef FC_W8
#undef FC_W1
    default: wait_vm<0>(); break;
  }
}
// Before a loop of DMAs: nothing is outstanding there, and this tells the compiler so.  In a
// kernel of two GEMMs it takes the other one's loads for outstanding and waits for all loads
// before each DMA's address is formed (a down projection of 100 rows, K 18944: 35 -> 53 us).
__device__ __forceinline__ void loads_done() { __builtin_amdgcn_s_waitcnt(0); }
// Workgroup barrier that orders LDS accesses only: global loads in flight stay in
// flight across it (the full fence of __syncthreads would drain them).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
__device__ __forceinline__ int swz8(int row) { return (row >> 1) & 7; }

__device__ __forceinline__ uint2 pack_bf16x4(float a, float b, float c, float d) {
  return make_uint2(f2bf(a) | ((uint32_t)f2bf(b) << 16), f2bf(c) | ((uint32_t)f2bf(d) << 16));
}
__device__ __forceinline__ float4 unpack_bf16x4(uint2 u) {
  return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u),
                     __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xFFFF0000u));
}

// The gathered rows of all items, packed: packed row p is slot b * N + (p - pre[b]) of
// the item b with pre[b] <= p < pre[b + 1] (pre = exclusive prefix sums of the
// recompute counts), so only the last tile of the whole batch is partly empty.
__device__ __forceinline__ long packed_slot(const int *pre, int B, int N, int p, int &b) {
  int lo = 0, hi = B - 1;                       // largest b with pre[b] <= p
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pre[mid] <= p) lo = mid; else hi = mid - 1;
  }
  b = lo;
  return (long)lo * N + (p - pre[lo]);
}

// Exclusive prefix sums of the recompute counts into pre[0..B] (wave 0; the caller
// synchronises): each lane sums a run of items, then the runs are scanned.
__device__ __forceinline__ void row_prefix(const int32_t *nrec, int B, int N, int *pre) {
  const int lane = threadIdx.x & 63;
  const int per = (B + 63) / 64, i0 = lane * per;
  int run = 0;
  for (int i = i0; i < min(i0 + per, B); ++i) run += n_valid(nrec, i, N);
  int inc = run;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(inc, o);
    if (lane >= o) inc += v;
  }
  int acc_run = inc - run;
  for (int i = i0; i < min(i0 + per, B); ++i) {
    pre[i] = acc_run;
    acc_run += n_valid(nrec, i, N);
  }
  if (lane == 63) pre[B] = inc;
}

}  // namespace
}  // namespace fc
