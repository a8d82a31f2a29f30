// Device helpers shared by the PCG kernels (pcg.hip, pcg_fused.hip).
#pragma once

#include <type_traits>

#include "common.h"
#include "wave_ops.h"

namespace bfal {

// A value that no workgroup of the launch writes, loaded through the scalar cache.
template <class T>
__device__ __forceinline__ T uniform_load(const T* p) {
  static_assert(sizeof(T) % 4 == 0 && std::is_trivially_copyable<T>::value, "whole words");
  const auto* w = (const __attribute__((address_space(4))) uint32_t*)(p);
  uint32_t u[sizeof(T) / 4];
#pragma unroll
  for (unsigned m = 0; m < sizeof(T) / 4; ++m) u[m] = w[m];
  T v;
  __builtin_memcpy(&v, u, sizeof(T));
  return v;
}

// Dispatch ids go round-robin over the 8 XCDs: give each XCD one contiguous
// range of logical workgroups.
__device__ inline int xcd_block(int b, int nb) { return (nb % 8 == 0) ? (b % 8) * (nb / 8) + b / 8 : b; }

__device__ inline void load_block(const float* __restrict__ u, int j, float b[9]) {
  const float* s = u + 9LL * j;
#pragma unroll
  for (int m = 0; m < 9; ++m) b[m] = s[m];
}

// BF16 block: 10 half-words in 5 words, element 2i in the low half of word i.
__device__ inline void load_block(const uint32_t* __restrict__ u, int j, float b[9]) {
  const uint32_t* s = u + 5LL * j;
  uint32_t w[5];
#pragma unroll
  for (int m = 0; m < 5; ++m) w[m] = s[m];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    b[2 * m] = __uint_as_float(w[m] << 16);
    b[2 * m + 1] = __uint_as_float(w[m] & 0xffff0000u);
  }
  b[8] = __uint_as_float(w[4] << 16);
}

// (written out: left to the compiler, the order of the three would change from place to place)
__device__ inline double dot3(double b0, double b1, double b2, const double x[3]) {
  return fma(b2, x[2], fma(b0, x[0], __dmul_rn(b1, x[1])));
}

// H_hat x for row `lane` of slice sl, off-diagonal part, the FP32 blocks
// widened to FP64: the upper slots in order, then the lower ones.  The loads of
// kAhead slots are in flight together (a slot past the width reads the last one
// again and is not added): one slot after the other was two round trips per
// slot (k_residual64 on 384 slices of 7 to 18 slots: 14.9 us against 11.9).
__device__ inline void row_product64(const PcgSystem& S, int sl, int lane, const double* __restrict__ xd, double& a0,
                                     double& a1, double& a2) {
  const float* __restrict__ blk = static_cast<const float*>(S.blk);
  const int bu = S.sbu[sl], wu = (S.sbu[sl + 1] - bu) / kSlice;
  const int bl = S.sbl[sl], wl = (S.sbl[sl + 1] - bl) / kSlice;
  a0 = a1 = a2 = 0.0;
  constexpr int kAhead = 4;
  for (int k0 = 0; k0 < wu; k0 += kAhead) {
    int e[kAhead], c[kAhead];
    float b[kAhead][9];
    double x[kAhead][3];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      e[u] = bu + min(k0 + u, wu - 1) * kSlice + lane;
      c[u] = S.scol[e[u]];
      load_block(blk, e[u], b[u]);
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
#pragma unroll
      for (int m = 0; m < 3; ++m) x[u][m] = xd[3LL * c[u] + m];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const bool in = k0 + u < wu;   // (a select: the loads are not to sink behind a branch)
      a0 = in ? __dadd_rn(a0, dot3(b[u][0], b[u][1], b[u][2], x[u])) : a0;
      a1 = in ? __dadd_rn(a1, dot3(b[u][3], b[u][4], b[u][5], x[u])) : a1;
      a2 = in ? __dadd_rn(a2, dot3(b[u][6], b[u][7], b[u][8], x[u])) : a2;
    }
  }
  for (int k0 = 0; k0 < wl; k0 += kAhead) {
    int2 t[kAhead];
    float b[kAhead][9];
    double x[kAhead][3];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) t[u] = S.sent[bl + min(k0 + u, wl - 1) * kSlice + lane];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      load_block(blk, t[u].x, b[u]);
#pragma unroll
      for (int m = 0; m < 3; ++m) x[u][m] = xd[3LL * t[u].y + m];
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const bool in = k0 + u < wl;
      a0 = in ? __dadd_rn(a0, dot3(b[u][0], b[u][3], b[u][6], x[u])) : a0;
      a1 = in ? __dadd_rn(a1, dot3(b[u][1], b[u][4], b[u][7], x[u])) : a1;
      a2 = in ? __dadd_rn(a2, dot3(b[u][2], b[u][5], b[u][8], x[u])) : a2;
    }
  }
}

// b_hat - (x + a) of one row in FP64 and its |L rd|^2.
__device__ inline double row_residual64(const PcgSystem& S, int row, const float* __restrict__ bhat,
                                        const double* __restrict__ xd, double a0, double a1, double a2, double& r0,
                                        double& r1, double& r2) {
  const long long o = 3LL * row;
  r0 = (double)bhat[o] - (xd[o] + a0);
  r1 = (double)bhat[o + 1] - (xd[o + 1] + a1);
  r2 = (double)bhat[o + 2] - (xd[o + 2] + a2);
  const float* L = S.Lf + row;   // SoA [6][N4]
  const long long n4 = S.N4;
  const double t0 = (double)L[0] * r0;
  const double t1 = (double)L[n4] * r0 + (double)L[2 * n4] * r1;
  const double t2 = (double)L[3 * n4] * r0 + (double)L[4 * n4] * r1 + (double)L[5 * n4] * r2;
  return t0 * t0 + t1 * t1 + t2 * t2;
}

}  // namespace bfal
