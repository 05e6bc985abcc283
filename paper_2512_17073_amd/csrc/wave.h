// Wavefront-wide sums inside the vector registers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lrc {

// Inclusive prefix sum over the 64 lanes: four shifts within rows of 16 lanes, then the rows' last lanes broadcast onwards (a
// shuffle goes through the LDS unit, about 100 cycles for each of its six steps).
__device__ inline int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);        // row_shr 1, 2, 4, 8 (lanes without a source: 0)
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);        // lane 15 of rows 0 and 2 to rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);        // lane 31 to rows 2 and 3
  return v;
}
__device__ inline int lane_value(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }     // (lane: wave-uniform)

}  // namespace lrc
