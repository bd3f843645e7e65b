// The 16 x 16 x 4 real matrix-core products both complex types are built from.
// Lane layouts (measured on gfx950):
//   A operand (16x4): lane l holds A[l%16][l/16]; B operand (4x16): B[l/16][l%16]
//   f64 result: lane l, element r holds D[4r + l/16][l%16]
//   f32 result: lane l, element r holds D[4(l/16) + r][l%16]
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"

namespace feast {

template <typename T> struct mfma_ops;

template <> struct mfma_ops<z64> {
  using real = double;
  using acc_t = dx4;
  __device__ static acc_t mma(real a, real b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // row of element r of the 16x16 result held by `lane`
  __device__ static int out_row(int lane, int r) { return 4 * r + (lane >> 4); }
};

template <> struct mfma_ops<c64> {
  using real = float;
  using acc_t = fx4;
  __device__ static acc_t mma(real a, real b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static int out_row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

}  // namespace feast
