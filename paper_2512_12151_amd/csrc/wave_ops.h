// Sums over a wavefront of 64 lanes, returned to every lane.
#pragma once

#include <hip/hip_runtime.h>

namespace bfal {

// v + (v of lane ^ 32), then ^ 16, 8, 4, 2, 1: the sums of a __shfl_xor
// butterfly, bit for bit, without its trips through LDS.  A shuffle of a
// double is two ds_bpermute at about 130 cycles of latency, and the compiler
// waits for each one: the sum of five doubles at the start of a PCG kernel took
// 5,000 cycles.  gfx950 swaps half wavefronts and rows of 16 lanes in registers
// (v_permlane32_swap: the high half of the first operand against the low half
// of the second; v_permlane16_swap: the odd rows against the even ones), so
// with v as both operands their sum is v[i] + v[i ^ 32] (^ 16) in every lane;
// inside a row the DPP moves do the rest: a rotation by 8, a rotation by 4 (the
// values repeat every 8 lanes by then), and two permutations of 4 lanes.
template <int kCtrl>
__device__ __forceinline__ double dpp_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

constexpr int kDppRowRor8 = 0x128, kDppRowRor4 = 0x124;
constexpr int kDppQuadXor2 = 0x4e;   // lanes 2, 3, 0, 1
constexpr int kDppQuadXor1 = 0xb1;   // lanes 1, 0, 3, 2

__device__ __forceinline__ double wave_sum_all(double v) {
  {
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
  }
  {
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
  }
  v += dpp_move<kDppRowRor8>(v);
  v += dpp_move<kDppRowRor4>(v);
  v += dpp_move<kDppQuadXor2>(v);
  v += dpp_move<kDppQuadXor1>(v);
  return v;
}

}  // namespace bfal
