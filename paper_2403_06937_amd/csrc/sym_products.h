// Real FP64 products whose result is symmetric, and the Taylor coefficients of
// the exponential's cosine and sine: shared by the exponential and by its
// Frechet derivative in the adjoint.
#pragma once
#include <vector>

#include "gemm_mfma.h"
#include "kernels.h"

namespace tcm {

// Only the upper tile triangle is multiplied, and mirrored.  A, B, C: N x N
// row-major, ld N.
struct SymProducts {
  int64_t N = 0;
  void* tail = nullptr; size_t tail_bytes = 0;   // partial sums of a last round
  bool spread = false;                           // (GemmDesc's tail_ws and spread)
  hipStream_t s = nullptr;
  // C = alpha A B + beta C + gamma I.  Either the product is symmetric, or a
  // following run adds the rest of a symmetric sum to C: the entries below the
  // tile diagonal are written, never read.
  int run(const double* A, const double* B, double* C, double alpha, double beta,
          double gamma = 0.0) const {
    GemmDesc d;
    d.M = d.N = d.K = N;
    d.A = A; d.lda = N; d.a_kmaj = false;
    d.B = B; d.ldb = N; d.b_kmaj = true;
    d.C = C; d.ldc = N;
    d.alpha_re = alpha;
    if (beta != 0.0) { d.Cin = C; d.ldcin = N; d.beta_re = beta; }
    d.gamma = gamma;
    d.complex = false;
    d.herm = true;
    d.tail_ws = tail; d.tail_ws_bytes = tail_bytes; d.spread = spread;
    return gemm_f64(d, s);
  }
};

// cos B = sum cc[k] X^k, sin B = B sum cs[k] X^k with X = B^2, to degrees kc, ks in X.
inline void taylor_cos_sin(int kc, int ks, std::vector<double>* cc, std::vector<double>* cs) {
  cc->assign(kc + 1, 0.0);
  cs->assign(ks + 1, 0.0);
  double f = 1.0;   // (2k)!
  for (int k = 0; k <= kc; ++k) {
    if (k > 0) f *= double(2 * k - 1) * double(2 * k);
    (*cc)[k] = (k % 2 ? -1.0 : 1.0) / f;
  }
  f = 1.0;          // (2k+1)!
  for (int k = 0; k <= ks; ++k) {
    if (k > 0) f *= double(2 * k) * double(2 * k + 1);
    (*cs)[k] = (k % 2 ? -1.0 : 1.0) / f;
  }
}

// Coefficients from .. to of a block a[3b] + a[3b + 1] X + a[3b + 2] X^2 (+ a[9] X^3),
// as launch_lin_powers takes them.
inline LinCoef block_coef(const std::vector<double>& a, int from, int to) {
  LinCoef c{{0.0, 0.0, 0.0, 0.0}};
  for (int k = from; k <= to && k < int(a.size()); ++k) c.a[k % 3 + (k == 9 ? 3 : 0)] = a[k];
  return c;
}

}  // namespace tcm
