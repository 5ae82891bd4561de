// Split-BF16 products of a small time step.
#pragma once
#include "gemm_bf16.h"
#include "gemm_small.h"

namespace tcm {

// C = A B (+ Cin): the FP32 result to Cf (when given) and its hi/lo planes to P
// (row-major, or transposed with p_trans).  A, B, P: 4-plane operands whose rows
// are padded to a multiple of 128 (Planes4), lda, ldb, ldp their padded K
// extents; herm: the result is Hermitian (M == N), the upper tile triangle is
// multiplied and mirrored.  Cin may be Cf.
struct SplitSmall {
  const uint16_t* A = nullptr; int64_t lda = 0;
  const uint16_t* B = nullptr; int64_t ldb = 0;
  int64_t M = 0, N = 0, Kp = 0;
  const c64* Cin = nullptr; int64_t ldcin = 0;
  c64* Cf = nullptr; int64_t ldcf = 0;
  uint16_t* P = nullptr; int64_t ldp = 0; int p_trans = 0;
  int herm = 0;
};

// Whether an N x N step takes these products, and so can read a record along: up
// to N = 640, unless TC_SPLIT_VARIANT asks for a shape of the 128 x 128 tiles.
bool split_small_step(int64_t N);
// ro: records of the state that the product multiplies, or NULL.
int split_small(const SplitSmall& p, const SmallReadout* ro, hipStream_t s);

}  // namespace tcm
