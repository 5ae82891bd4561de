// Products of small complex matrices, alone (with the record that a step's
// first product can take along) or grouped.
#pragma once
#include <vector>

#include "gemm_mfma.h"
#include "kernels.h"

namespace tcm {

// Records of the state that a product multiplies, read by one more workgroup of
// its launch: record `index`, or the one *counter holds, which is then advanced
// (captured launches).
struct SmallReadout {
  ReadoutItem item{};
  int64_t index = 0;
  int* counter = nullptr;
};

// Whether d takes the small product kernel.
bool small_product(const GemmDesc& d, bool f64);
// d of double / float complex elements, small_product(d); ro may be NULL.
template <typename T>
int small_gemm(const GemmDesc& d, const SmallReadout* ro, hipStream_t s);

// Estimated us of one group of small products with t16 tiles of 16 x 16, or t32 of
// 32 x 32, and mean K, on the better edge (*edge, may be NULL).
double small_group_us(double t16, double t32, double K, bool f64, int* edge);

// Small products of many instances in one launch.
struct SmallGroup {
  bool f64 = false;
  int edge = 16;               // tile edge
  int count = 0, tiles = 0;
  void* items_dev = nullptr;   // small_grouped_bytes(count)
};
size_t small_grouped_bytes(int count);
// Uploads the descriptors (synchronises s).
int small_grouped_build(const std::vector<GemmDesc>& ds, bool f64, void* items_dev, SmallGroup* g,
                        hipStream_t s);
int small_grouped_run(const SmallGroup& g, hipStream_t s);

}  // namespace tcm
