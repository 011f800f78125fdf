// Strip kernels that store 16 bytes at a time (back-turned image), for the
// assembly check of tests/test_wide_store_asm.py.
#define SAR_PART 9
#include "rda_kernels.inl"

template __global__ void sar::k_line_strip<64, sar::LK_FUSED, 8, true>(
    const float2*, float2*, int, sar::TileMap, const float2*, const float2*, float);
template __global__ void sar::k_line_strip<512, sar::LK_FUSED, 4, true>(
    const float2*, float2*, int, sar::TileMap, const float2*, const float2*, float);
