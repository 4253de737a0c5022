// wave.h - reductions over the 64 lanes of a wave (gfx950).
#pragma once

#include <hip/hip_runtime.h>

namespace sppc {

// Sum over the 64 lanes of a wave, returned to every lane, with DPP moves instead of the
// LDS-routed lane shuffles (about 100 cycles of dependent latency instead of about 900):
// prefix sums within rows of 16 lanes (shifts 1, 2, 4, 8; lanes without a source add 0), then
// lane 15 of rows 0 and 2 into rows 1 and 3, lane 31 into rows 2 and 3, and lane 63 is read.
template <int CTRL, int ROWS>
__device__ inline double dpp_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, true);
  return __hiloint2double(hi, lo);
}
// lane l's value, l uniform over the wave
__device__ inline double lane_get(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}
__device__ inline double wave_sum(double v) {
  v += dpp_move<0x111, 0xF>(v);  // row_shr:1
  v += dpp_move<0x112, 0xF>(v);  // row_shr:2
  v += dpp_move<0x114, 0xF>(v);  // row_shr:4
  v += dpp_move<0x118, 0xF>(v);  // row_shr:8
  v += dpp_move<0x142, 0xA>(v);  // row_bcast:15 into rows 1, 3
  v += dpp_move<0x143, 0xC>(v);  // row_bcast:31 into rows 2, 3
  return lane_get(v, 63);
}
__device__ inline double wave_max(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
  return v;
}

// LDS written by lanes of this wave is visible to its other lanes (a wave's LDS accesses take
// effect in program order; this keeps the compiler from moving them across)
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace sppc
