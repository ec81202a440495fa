// Scans over the lanes of a wave by lane shifts (data-parallel primitives), without a word through LDS.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// Inclusive sums over the wave's lanes: shifts inside the rows of 16 lanes (data-parallel primitives,
// no LDS traffic), then the totals of the rows before the lane's own.
__device__ __forceinline__ uint32_t wave_scan_add(uint32_t x, int lane)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);  // row_shr:8
    const uint32_t t0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 15), t1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 31),
                   t2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 47);
    const int row = lane >> 4;
    return x + (row >= 1 ? t0 : 0u) + (row >= 2 ? t1 : 0u) + (row >= 3 ? t2 : 0u);
}

// The same inside one row of 16 lanes only (lanes 0..15 of a wave hold the 16 values).
__device__ __forceinline__ uint32_t row_scan_add(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
    return x;
}
__device__ __forceinline__ int row_scan_max(int x)
{
    int y = __builtin_amdgcn_update_dpp(-1, x, 0x111, 0xf, 0xf, false);
    x = y > x ? y : x;
    y = __builtin_amdgcn_update_dpp(-1, x, 0x112, 0xf, 0xf, false);
    x = y > x ? y : x;
    y = __builtin_amdgcn_update_dpp(-1, x, 0x114, 0xf, 0xf, false);
    x = y > x ? y : x;
    y = __builtin_amdgcn_update_dpp(-1, x, 0x118, 0xf, 0xf, false);
    return y > x ? y : x;
}
