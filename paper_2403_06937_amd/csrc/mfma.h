// Device helpers shared by the product kernels: matrix instructions and the order
// of tiles.
#pragma once
#include "common.h"

namespace tcm {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// 16 x 16 x 4 MFMA: lane l supplies A[l%16][l/16] and B[l/16][l%16]; output r of
// lane l is row l/16 + 4r (FP64, measured on gfx950) or 4(l/16) + r (FP32) of column
// l%16.  mma_nega: c - a b, in FP64 by the instruction's own negation modifier
// (neg:[1,0,0]).
__device__ __forceinline__ d4 mma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ d4 mma_nega(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 1);
}
__device__ __forceinline__ f4 mma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mma_nega(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(-a, b, c, 0, 0, 0);
}
// 16 x 16 x 32 in bfloat16: lane l holds 8 consecutive K values of row (column) l%16,
// outputs as in FP32.
__device__ __forceinline__ f4 mma(const u4& a, const u4& b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a),
                                                 __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}
template <typename T> struct acc_t;
template <> struct acc_t<double> { typedef d4 type; };
template <> struct acc_t<float> { typedef f4 type; };

// Consecutive workgroup ids go round the 8 XCDs; give each XCD a contiguous
// run of the tile order so that its tiles share operand rows in its L2.
__device__ __forceinline__ int xcd_linear(int pid, int total) {
  const int q = total / 8, r = total % 8;
  const int xcd = pid % 8, local = pid / 8;
  return (xcd < r ? xcd * (q + 1) : r * (q + 1) + (xcd - r) * q) + local;
}

constexpr int GROUP_M = 8;      // tile rows walked together

// Tile lin of the upper block triangle (tm <= tn) of a T x T tile grid:
// GROUP_M tile rows at a time, column by column within a group.
__device__ __forceinline__ void tri_coords(int lin, int T, int& tm, int& tn) {
  int first = 0;
  for (;;) {
    const int gs = min(T - first, GROUP_M);
    const int tri = gs * (gs - 1) / 2;              // the group's leading triangle
    const int cnt = gs * (T - first) - tri;
    if (lin < cnt) {
      if (lin < tri) {
        int c = 0;
        while ((c + 1) * (c + 2) / 2 <= lin) ++c;
        tn = first + c;
        tm = first + lin - c * (c + 1) / 2;
      } else {
        const int q = lin - tri;
        tn = first + gs - 1 + q / gs;
        tm = first + q % gs;
      }
      return;
    }
    lin -= cnt;
    first += gs;
  }
}

// The same, all rows column by column.
__device__ __forceinline__ void tri_columns(int lin, int& tm, int& tn) {
  int j = int((__builtin_sqrtf(8.f * float(lin) + 1.f) - 1.f) * 0.5f);
  while (j * (j + 1) / 2 > lin) --j;
  while ((j + 1) * (j + 2) / 2 <= lin) ++j;
  tn = j;
  tm = lin - j * (j + 1) / 2;
}

}  // namespace tcm
