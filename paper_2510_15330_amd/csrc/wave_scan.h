// Inclusive scan over the 64 lanes of a wave (lane 63: the sum), on the
// data-parallel permutes: six dependent adds, where lane shuffles take a
// round trip through LDS each.
#pragma once

#include <hip/hip_runtime.h>

namespace bellman {

__device__ __forceinline__ int lane_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr 1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, true);   // row_bcast 15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, true);   // row_bcast 31 into rows 2, 3
    return v;
}

}  // namespace bellman
