// Device helpers of the GEMM kernels (gemm.hip, gemm_deep.hip).
#pragma once

#include "common.hpp"

namespace hdf {

__device__ __forceinline__ int remap_tile(int bid, int total) {
  // XCD-aware order: dispatch sends consecutive workgroups round-robin over the 8
  // XCDs; give each XCD a contiguous run of tile ids (the M-tiles of one weight
  // column block are consecutive ids).
  const int per = total >> 3;
  if (bid < (per << 3)) return (bid & 7) * per + (bid >> 3);
  return bid;
}

__device__ __forceinline__ unsigned long long argmax_key(float v, int col) {
  return (static_cast<unsigned long long>(f32_order_key(v)) << 32) |
         static_cast<unsigned long long>(0xFFFFFFFFu - static_cast<uint32_t>(col));
}

}  // namespace hdf
