// HBM-bound and latency-bound kernels of libtcm: the Hamiltonian of Eq. (4),
// helpers of the matrix exponential, frame changes, per-step diagonal readout,
// FP64 renormalisation, full observables and the bfloat16 split.
//
// Reductions are deterministic: fixed per-thread strides, a butterfly of
// cross-lane exchanges inside each wavefront, then the wave results added in
// a fixed order (no atomics), so reruns are bitwise identical.
#include "kernels.h"

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>
#include "ham_entry.h"
#include "readout.h"

namespace tcm {
namespace {

constexpr int TPB = 256;

__device__ __forceinline__ int popc64(uint64_t x) { return __popcll(x); }

// Wavefront sum by a butterfly of cross-lane exchanges: every lane ends with
// the same bits (each exchange adds the same two values, and IEEE addition
// commutes).
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Block-wide sum (all threads get the result): a wavefront sum per wave, then
// the TPB / 64 wave results added in wave order.
__device__ double block_sum(double v, double* sh) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = sh[0];
#pragma unroll
  for (int w = 1; w < TPB / 64; ++w) r += sh[w];
  __syncthreads();
  return r;
}
__device__ double block_max(double v, double* sh) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = sh[0];
#pragma unroll
  for (int w = 1; w < TPB / 64; ++w) r = fmax(r, sh[w]);
  __syncthreads();
  return r;
}

// ------------------------------------------------------------ Eq. (4)
__global__ void ham_fill_kernel(ModelArgs m, double* __restrict__ H, int64_t ldh) {
  const int64_t col = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (col >= m.N) return;
  for (int64_t row = blockIdx.y; row < m.N; row += gridDim.y)
    H[row * ldh + col] = ham_entry(m, row, col);
}

// ----------------------------------------------------- expm helpers
__global__ void axpb_identity_kernel(const double* __restrict__ X, int64_t ldx, double a, double b,
                                     double* __restrict__ out, int64_t ldo, int64_t N) {
  const int64_t col = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (col >= N) return;
  for (int64_t row = blockIdx.y; row < N; row += gridDim.y)
    out[row * ldo + col] = a * X[row * ldx + col] + (row == col ? b : 0.0);
}

__global__ void lin_powers_kernel(const double* X, const double* X2, const double* X3,
                                  int64_t count, int64_t N, LinCoef c0, double* out0, LinCoef c1,
                                  double* out1, LinCoef c2, double* out2) {
  const int64_t step = int64_t(gridDim.x) * TPB;
  for (int64_t e = int64_t(blockIdx.x) * TPB + threadIdx.x; e < count; e += step) {
    const double x = X[e], x2 = X2[e], x3 = X3[e];
    const double d = e / N == e % N ? 1.0 : 0.0;
    if (out0) out0[e] = c0.a[0] * d + c0.a[1] * x + c0.a[2] * x2 + c0.a[3] * x3;
    if (out1) out1[e] = c1.a[0] * d + c1.a[1] * x + c1.a[2] * x2 + c1.a[3] * x3;
    if (out2) out2[e] = c2.a[0] * d + c2.a[1] * x + c2.a[2] * x2 + c2.a[3] * x3;
  }
}

__global__ void diff_sum_kernel(const double* __restrict__ C, const double* __restrict__ S,
                                double* __restrict__ D, double* __restrict__ E, int64_t count) {
  const int64_t step = int64_t(gridDim.x) * TPB;
  for (int64_t e = int64_t(blockIdx.x) * TPB + threadIdx.x; e < count; e += step) {
    const double c = C[e], s = S[e];
    D[e] = c - s;
    E[e] = c + s;
  }
}

// ----------------------------------------------------------- copies
__global__ void c128_to_c64_kernel(const c128* __restrict__ s, int64_t lds, c64* __restrict__ d,
                                   int64_t ldd, int64_t rows, int64_t cols) {
  const int64_t col = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (col >= cols) return;
  for (int64_t row = blockIdx.y; row < rows; row += gridDim.y) {
    const c128 v = s[row * lds + col];
    d[row * ldd + col] = c64{float(v.re), float(v.im)};
  }
}
__global__ void c64_to_c128_kernel(const c64* __restrict__ s, int64_t lds, c128* __restrict__ d,
                                   int64_t ldd, int64_t rows, int64_t cols) {
  const int64_t col = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (col >= cols) return;
  for (int64_t row = blockIdx.y; row < rows; row += gridDim.y) {
    const c64 v = s[row * lds + col];
    d[row * ldd + col] = c128{double(v.re), double(v.im)};
  }
}

// ------------------------------------------------------ rotating frame
__device__ __forceinline__ int exc_number(int64_t s, int n) {
  const uint64_t mask = (uint64_t(1) << n) - 1;
  return int(s >> n) + popc64(uint64_t(s) & mask);
}

template <typename E>
__global__ void rotating_d_kernel(ModelArgs m, const c128* __restrict__ U, int64_t ldu, double dt,
                                  E* __restrict__ D, int64_t ldd) {
  const int64_t col = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (col >= m.N) return;
  for (int64_t row = blockIdx.y; row < m.N; row += gridDim.y) {
    double sn, cs;
    sincos(m.omega_c * double(exc_number(row, m.n)) * dt, &sn, &cs);
    const c128 u = U[row * ldu + col];
    c128 v{cs * u.re - sn * u.im, cs * u.im + sn * u.re};
    if (row == col) v.re -= 1.0;
    typedef decltype(E().re) T;
    D[row * ldd + col] = E{T(v.re), T(v.im)};
  }
}

template <typename E>
__global__ void frame_phase_kernel(ModelArgs m, E* __restrict__ rho, int64_t ld, double t) {
  const int64_t col = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (col >= m.N) return;
  const int kc = exc_number(col, m.n);
  for (int64_t row = blockIdx.y; row < m.N; row += gridDim.y) {
    const int kr = exc_number(row, m.n);
    if (kr == kc) continue;
    double sn, cs;
    sincos(-m.omega_c * double(kr - kc) * t, &sn, &cs);
    const E v = rho[row * ld + col];
    const double re = double(v.re), im = double(v.im);
    rho[row * ld + col] = E{decltype(v.re)(cs * re - sn * im), decltype(v.re)(cs * im + sn * re)};
  }
}

// ------------------------------------------------------- dissipation
// Amplitude damping of the atoms on index bits b0 and b1 (b1 < 0: b0 only;
// atom i is bit n - 1 - i), probability p = 1 - e^{-gamma dt}, f = sqrt(1 - p).
// For one atom and the 2 x 2 block of rows {r, r + e} and columns {s, s + e}
// (both with the atom's bit clear) the channel K0 . K0^dag + K1 . K1^dag is
//   x00 <- x00 + p x11,  x01 <- f x01,  x10 <- f x10,  x11 <- (1 - p) x11.
// A thread owns the (2^k x 2^k) block over the k bits of the pass, so the
// update is in place with no other thread touching its elements.
__device__ __forceinline__ int64_t insert_zero_bit(int64_t q, int b) {
  return ((q >> b) << (b + 1)) | (q & ((int64_t(1) << b) - 1));
}

template <typename E, int K>
__global__ void damp_atoms_kernel(E* __restrict__ rho, int64_t ld, int64_t N, int b0, int b1,
                                  double p, double f) {
  constexpr int B = 1 << K;
  const int64_t R = N >> K;                  // reduced row / column count
  const int64_t qs = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (qs >= R) return;
  int64_t s0 = insert_zero_bit(qs, b0);
  if (K == 2) s0 = insert_zero_bit(s0, b1);
  const int64_t e[2] = {int64_t(1) << b0, K == 2 ? int64_t(1) << b1 : 0};
  for (int64_t qr = blockIdx.y; qr < R; qr += gridDim.y) {
    int64_t r0 = insert_zero_bit(qr, b0);
    if (K == 2) r0 = insert_zero_bit(r0, b1);
    double xr[B][B], xi[B][B];
#pragma unroll
    for (int u = 0; u < B; ++u)
#pragma unroll
      for (int v = 0; v < B; ++v) {
        const int64_t r = r0 + ((u & 1) ? e[0] : 0) + ((u & 2) ? e[1] : 0);
        const int64_t c = s0 + ((v & 1) ? e[0] : 0) + ((v & 2) ? e[1] : 0);
        const E x = rho[r * ld + c];
        xr[u][v] = double(x.re);
        xi[u][v] = double(x.im);
      }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int bit = 1 << k;
#pragma unroll
      for (int u = 0; u < B; ++u)
#pragma unroll
        for (int v = 0; v < B; ++v) {
          if ((u & bit) || (v & bit)) continue;
          const int u1 = u | bit, v1 = v | bit;
          xr[u][v] += p * xr[u1][v1];
          xi[u][v] += p * xi[u1][v1];
          xr[u][v1] *= f; xi[u][v1] *= f;
          xr[u1][v] *= f; xi[u1][v] *= f;
          xr[u1][v1] *= 1.0 - p; xi[u1][v1] *= 1.0 - p;
        }
    }
#pragma unroll
    for (int u = 0; u < B; ++u)
#pragma unroll
      for (int v = 0; v < B; ++v) {
        const int64_t r = r0 + ((u & 1) ? e[0] : 0) + ((u & 2) ? e[1] : 0);
        const int64_t c = s0 + ((v & 1) ? e[0] : 0) + ((v & 2) ? e[1] : 0);
        rho[r * ld + c] = E{decltype(E::re)(xr[u][v]), decltype(E::re)(xi[u][v])};
      }
  }
}

// The three channels on one 8 x 8 block held by two neighbouring lanes: lane
// h has rows u = 4 h + uu (uu = 0..3) and all 8 columns; bit k of a row or
// column index is the state of atom k of the three.
__device__ __forceinline__ void damp3_block(float (&xr)[4][8], float (&xi)[4][8], int h, float p,
                                            float f) {
  const float q1 = 1.f - p;
  // atom b2: lane 0 gains p x[u|4][v|4] (the partner's columns 4..7), then
  // scales its columns 4..7 by f; lane 1 scales columns 0..3 by f and 4..7
  // by 1 - p
#pragma unroll
  for (int uu = 0; uu < 4; ++uu)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float pr = __shfl_xor(xr[uu][v + 4], 1, 64);
      const float pi = __shfl_xor(xi[uu][v + 4], 1, 64);
      if (h == 0) {
        xr[uu][v] += p * pr;
        xi[uu][v] += p * pi;
        xr[uu][v + 4] *= f;
        xi[uu][v + 4] *= f;
      } else {
        xr[uu][v] *= f;
        xi[uu][v] *= f;
        xr[uu][v + 4] *= q1;
        xi[uu][v + 4] *= q1;
      }
    }
  // atoms b0, b1 inside the half (row bits 0, 1 of uu; column bits 0, 1 of v)
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int bit = 1 << k;
#pragma unroll
    for (int uu = 0; uu < 4; ++uu)
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        if ((uu & bit) || (v & bit)) continue;
        const int u1 = uu | bit, v1 = v | bit;
        xr[uu][v] += p * xr[u1][v1];
        xi[uu][v] += p * xi[u1][v1];
        xr[uu][v1] *= f; xi[uu][v1] *= f;
        xr[u1][v] *= f; xi[u1][v] *= f;
        xr[u1][v1] *= q1; xi[u1][v1] *= q1;
      }
  }
}

// Three atoms per pass (bits b0 < b1 < b2) for the complex FP32 state, in
// FP32 arithmetic: the same channel as above for each of the three bits, so a
// state of n atoms takes ceil(n / 3) passes over the matrix instead of
// ceil(n / 2).  The 8 x 8 block of one row and column triple is shared by two
// neighbouring lanes: lane h of the pair holds its rows u with u's bit 2
// (atom b2) equal to h, 32 complex values, so the kernel fits three waves per
// SIMD (one lane holding all 64 values needed more than 256 registers and ran
// one wave per SIMD at half of HBM bandwidth).  The channels of different
// atoms commute, so the b2 channel goes first: its only coupling between the
// halves, x[u][v] += p x[u|4][v|4] for u, v with bit 2 clear, takes the
// partner's 16 values x[u|4][v|4] by a cross-lane exchange before either lane
// changes them; the b0 and b1 channels then act inside each half.
__global__ void __launch_bounds__(TPB)
damp_atoms3_c64_kernel(c64* __restrict__ rho, int64_t ld, int64_t N, int b0, int b1, int b2,
                       float p, float f) {
  const int64_t R = N >> 3;
  const int64_t tid = int64_t(blockIdx.x) * TPB + threadIdx.x;
  const int64_t qs = tid >> 1;
  const int h = int(tid & 1);
  if (qs >= R) return;                       // both lanes of a pair leave together
  const int64_t s0 = insert_zero_bit(insert_zero_bit(insert_zero_bit(qs, b0), b1), b2);
  const int64_t e0 = int64_t(1) << b0, e1 = int64_t(1) << b1, e2 = int64_t(1) << b2;
  for (int64_t qr = blockIdx.y; qr < R; qr += gridDim.y) {
    const int64_t r0 = insert_zero_bit(insert_zero_bit(insert_zero_bit(qr, b0), b1), b2) +
                       (h ? e2 : 0);
    float xr[4][8], xi[4][8];                // rows u = 4 h + uu, all 8 columns
#pragma unroll
    for (int uu = 0; uu < 4; ++uu)
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const int64_t r = r0 + ((uu & 1) ? e0 : 0) + ((uu & 2) ? e1 : 0);
        const int64_t c = s0 + ((v & 1) ? e0 : 0) + ((v & 2) ? e1 : 0) + ((v & 4) ? e2 : 0);
        const c64 x = rho[r * ld + c];
        xr[uu][v] = x.re;
        xi[uu][v] = x.im;
      }
    damp3_block(xr, xi, h, p, f);
#pragma unroll
    for (int uu = 0; uu < 4; ++uu)
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const int64_t r = r0 + ((uu & 1) ? e0 : 0) + ((uu & 2) ? e1 : 0);
        const int64_t c = s0 + ((v & 1) ? e0 : 0) + ((v & 2) ? e1 : 0) + ((v & 4) ? e2 : 0);
        rho[r * ld + c] = c64{xr[uu][v], xi[uu][v]};
      }
  }
}

// The same three-atom pass for atoms b, b + 1, b + 2 with coalesced memory
// access.  Each 8 x 8 block's columns lie 2^b apart, so a lane pair reading its
// own block touches a different cache line with almost every load.  Here a
// workgroup takes one row triple group (the 8 rows r0 + u 2^b) and a window of
// W consecutive columns (W a multiple of 8 2^b, so the window holds W / 8 whole
// column groups): it reads the 8 x W values with 16-byte loads that cover
// contiguous rows, stages them in LDS, applies damp3_block to each block with
// two lanes per block as above, and writes the window back the same way.  LDS
// holds column w of a row at w + w / 8 (rows W + W / 8 + 2 long), which keeps
// the block reads of a wave on distinct banks for every b.
__device__ __forceinline__ int damp3_pos(int w) { return w + (w >> 3); }

__global__ void __launch_bounds__(512)
damp_atoms3_lds_c64_kernel(c64* __restrict__ rho, int64_t ld, int64_t N, int b, int W, float p,
                           float f) {
  extern __shared__ float2 sx[];
  const int pitch = W + (W >> 3) + 2;
  const int nt = W >> 2;                      // two lanes per block, W / 8 blocks
  const int t = threadIdx.x;
  const int64_t e = int64_t(1) << b;
  const int64_t c0 = int64_t(blockIdx.x) * W;
  // this lane's block and half
  const int blk = t >> 1, h = t & 1;
  const int j = blk & int(e - 1), gi = blk >> b;
  for (int64_t rg = blockIdx.y; rg < (N >> 3); rg += gridDim.y) {
    const int64_t r0 = insert_zero_bit(insert_zero_bit(insert_zero_bit(rg, b), b + 1), b + 2);
    // 8 rows x W columns: piece k * nt + t (two complex values) of every row
    float4 v[8][2];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int64_t col = c0 + 2 * (k * nt + t);
        v[u][k] = *reinterpret_cast<const float4*>(rho + (r0 + u * e) * ld + col);
      }
    __syncthreads();                          // the previous group's window is written out
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int w = 2 * (k * nt + t);       // even: w and w + 1 share a group of 8
        sx[u * pitch + damp3_pos(w)] = make_float2(v[u][k].x, v[u][k].y);
        sx[u * pitch + damp3_pos(w) + 1] = make_float2(v[u][k].z, v[u][k].w);
      }
    __syncthreads();
    {
      float xr[4][8], xi[4][8];
#pragma unroll
      for (int uu = 0; uu < 4; ++uu)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const int w = (gi << (b + 3)) | (c << b) | j;
          const float2 x = sx[(4 * h + uu) * pitch + damp3_pos(w)];
          xr[uu][c] = x.x;
          xi[uu][c] = x.y;
        }
      damp3_block(xr, xi, h, p, f);
#pragma unroll
      for (int uu = 0; uu < 4; ++uu)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const int w = (gi << (b + 3)) | (c << b) | j;
          sx[(4 * h + uu) * pitch + damp3_pos(w)] = make_float2(xr[uu][c], xi[uu][c]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int w = 2 * (k * nt + t);
        const float2 a = sx[u * pitch + damp3_pos(w)], c = sx[u * pitch + damp3_pos(w) + 1];
        *reinterpret_cast<float4*>(rho + (r0 + u * e) * ld + c0 + w) = make_float4(a.x, a.y, c.x, c.y);
      }
  }
}

// The lowest six atoms (index bits 0 .. nb - 1, nb <= 6) in one pass: the 64 x 64
// tiles of the matrix are closed under their channels.  A workgroup reads its
// tile along rows into LDS, applies the channels of two bits at a time to the
// tile's 4 x 4 blocks, one block per thread, and writes the tile back along
// rows, so the state is read and written once for six atoms; the arithmetic is
// FP64 in either storage.  HBM- (or MALL-) bound.  Bits from nb on belong to the
// photon number and are left alone; a ragged last tile holds zeros outside the
// matrix and stores nothing there.  Column w of a tile row sits at w + w / 4: the
// block reads of neighbouring lanes fall on distinct banks in every pass.
// N = 2048 FP32: 18 us against 2 x 10.8 for two three-atom passes; FP64 in place of
// three pair passes: all damping of a step 139 -> 76 us.
constexpr int D6 = 64, D6_PITCH = 79;

template <typename E>
__global__ void __launch_bounds__(TPB)
damp_atoms6_kernel(E* __restrict__ rho, int64_t ld, int64_t N, int nb, double p, double f) {
  typedef decltype(E().re) T;
  __shared__ E sx[D6 * D6_PITCH];
  auto at = [&](int r, int c) -> E& { return sx[r * D6_PITCH + c + (c >> 2)]; };
  const int t = threadIdx.x, tc = t & 63, tr = t >> 6;
  const int64_t r0 = int64_t(blockIdx.y) * D6, c0 = int64_t(blockIdx.x) * D6;
  const bool cin = c0 + tc < N;
#pragma unroll
  for (int r = tr; r < D6; r += TPB / 64)
    at(r, tc) = cin && r0 + r < N ? rho[(r0 + r) * ld + c0 + tc] : E{T(0), T(0)};
  __syncthreads();
  const int cb = t & 15, rb = t >> 4;         // the thread's block, bits b and b + 1 left out
  const double q1 = 1.0 - p;
#pragma unroll
  for (int b = 0; b < 6; b += 2) {
    if (b >= nb) break;
    const int lo = (1 << b) - 1;
    const int cc = ((cb & ~lo) << 2) | (cb & lo), rr = ((rb & ~lo) << 2) | (rb & lo);
    double xr[4][4], xi[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const E x = at(rr + (u << b), cc + (v << b));
        xr[u][v] = double(x.re);
        xi[u][v] = double(x.im);
      }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (b + k >= nb) break;
      const int bit = 1 << k;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if ((u & bit) || (v & bit)) continue;
          const int u1 = u | bit, v1 = v | bit;
          xr[u][v] += p * xr[u1][v1];
          xi[u][v] += p * xi[u1][v1];
          xr[u][v1] *= f; xi[u][v1] *= f;
          xr[u1][v] *= f; xi[u1][v] *= f;
          xr[u1][v1] *= q1; xi[u1][v1] *= q1;
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        at(rr + (u << b), cc + (v << b)) = E{T(xr[u][v]), T(xi[u][v])};
    __syncthreads();
  }
#pragma unroll
  for (int r = tr; r < D6; r += TPB / 64)
    if (cin && r0 + r < N) rho[(r0 + r) * ld + c0 + tc] = at(r, tc);
}

// Cavity damping with eta = e^{-kappa dt}: Kraus operators
// E_l = sum_m sqrt(binom(m, l)) eta^{(m-l)/2} (1 - eta)^{l/2} |m - l><m|, so
//   rho'[(m,a),(m',a')] = sum_{l >= 0} sqrt(binom(m+l, l) binom(m'+l, l))
//                         eta^{(m+m')/2} (1 - eta)^l rho[(m+l,a),(m'+l,a')].
// A thread owns one chain (a, a', m' - m = d) and walks it from the lowest
// photon numbers up, so each new value reads only entries not yet rewritten.
template <typename E>
__global__ void damp_cavity_kernel(E* __restrict__ rho, int64_t ld, int n, int c, double eta) {
  const int64_t per = int64_t(1) << n;
  const int64_t ac = int64_t(blockIdx.x) * TPB + threadIdx.x;   // column atom index a'
  if (ac >= per) return;
  const int d = int(blockIdx.z) - c;                             // m' - m
  const int mlo = d < 0 ? -d : 0;
  const int len = c + 1 - (d < 0 ? -d : d);
  const double q = 1.0 - eta;
  for (int64_t ar = blockIdx.y; ar < per; ar += gridDim.y) {
    for (int j = 0; j < len; ++j) {
      const int m = mlo + j, mp = m + d;
      double coef = pow(eta, 0.5 * double(m + mp));
      double yr = 0.0, yi = 0.0;
      for (int l = 0; j + l < len; ++l) {
        if (l > 0) coef *= sqrt(double(m + l) * double(mp + l)) / double(l) * q;
        const E x = rho[(int64_t(m + l) * per + ar) * ld + int64_t(mp + l) * per + ac];
        yr += coef * double(x.re);
        yi += coef * double(x.im);
      }
      rho[(int64_t(m) * per + ar) * ld + int64_t(mp) * per + ac] =
          E{decltype(E::re)(yr), decltype(E::re)(yi)};
    }
  }
}

// The same channel with each chain held in registers (c + 1 <= L): a thread owns
// one chain of one (a, a') pair, every element is read once and written once and
// neighbouring threads' elements are neighbours in memory.  The coefficient of
// rho[(m+l, a), (m'+l, a')] factors into a[m][l] a[m'][l] with
//   a[m][l] = eta^{m/2} (binom(m + l, l) |1 - eta|^l)^{1/2},
// L^2 numbers from the host whose index is the same for all threads of a
// workgroup, and the sign of (1 - eta)^l: -1 for odd l when eta > 1, which is the
// inverse channel of a run with a negative dt.  HBM-bound: N = 2048 FP32 11 us
// against 46 when each coefficient's roots and divisions were formed per element.
template <int L> struct CavityCoef {
  double a[L * L];
  double odd;                                // sign of (1 - eta)^l for odd l
};

template <typename E, int L>
__global__ void __launch_bounds__(TPB)
damp_cavity_reg_kernel(E* __restrict__ rho, int64_t ld, int n, int c, CavityCoef<L> k) {
  const int64_t per = int64_t(1) << n;
  const int64_t id = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (id >= per * per) return;
  const int64_t ar = id >> n, ac = id & (per - 1);
  const int d = int(blockIdx.y) - c;                             // m' - m
  const int mlo = d < 0 ? -d : 0;
  const int len = c + 1 - (d < 0 ? -d : d);
  E* __restrict__ base = rho + (int64_t(mlo) * per + ar) * ld + int64_t(mlo + d) * per + ac;
  const int64_t step = per * ld + per;
  double xr[L], xi[L];
#pragma unroll
  for (int j = 0; j < L; ++j)
    if (j < len) {
      const E x = base[j * step];
      xr[j] = double(x.re);
      xi[j] = double(x.im);
    }
#pragma unroll
  for (int j = 0; j < L; ++j) {
    if (j >= len) break;
    const double* am = k.a + (mlo + j) * L;
    const double* ap = k.a + (mlo + j + d) * L;
    double yr = 0.0, yi = 0.0;
#pragma unroll
    for (int l = 0; j + l < L; ++l) {
      if (j + l >= len) break;
      const double w = (l & 1 ? k.odd : 1.0) * am[l] * ap[l];
      yr += w * xr[j + l];
      yi += w * xi[j + l];
    }
    base[j * step] = E{decltype(E::re)(yr), decltype(E::re)(yi)};
  }
}

// ------------------------------------------------------- per-step readout
template <typename E>
__global__ void __launch_bounds__(READOUT_NT)
readout_kernel(ModelArgs m, const E* __restrict__ rho, int64_t ld,
               const int32_t* __restrict__ map, const int32_t* __restrict__ off, int k,
               double* __restrict__ pop, double* __restrict__ pdist,
               double* __restrict__ pstate) {
  __shared__ double sh[READOUT_LDS];
  readout_body(m.n, m.c, rho, ld, map, off, k, pop, pdist, pstate, sh);
}

// Each workgroup advances its own item's record index, after the body's
// barrier, by which point every thread has read it.
template <typename E>
__global__ void __launch_bounds__(READOUT_NT)
grouped_readout_kernel(const ReadoutItem* __restrict__ items, int* counter) {
  __shared__ double sh[READOUT_LDS];
  const ReadoutItem it = items[blockIdx.x];
  const int64_t r = counter[blockIdx.x];
  const int ns = (it.n < it.c ? it.n : it.c) + 1;
  readout_body(it.n, it.c, static_cast<const E*>(it.rho), it.ld, it.map, it.off, it.k,
               it.pop ? it.pop + r : nullptr, it.pdist ? it.pdist + r * (it.c + 1) : nullptr,
               it.pstate ? it.pstate + r * ns : nullptr, sh);
  if (threadIdx.x == 0) counter[blockIdx.x] = int(r) + 1;
}

// ---------------------------------------------------- FP64 renormalisation
template <typename E>
__global__ void trace_kernel(const E* __restrict__ rho, int64_t ld, int64_t N, double* scratch) {
  __shared__ double sh[TPB / 64];
  double part = 0.0;
  for (int64_t s = threadIdx.x; s < N; s += TPB) part += double(rho[s * ld + s].re);
  const double tr = block_sum(part, sh);
  if (threadIdx.x == 0) {
    scratch[0] = tr;
    if (!(tr > 0.0) || !isfinite(tr)) scratch[1] = 1.0;
  }
}

constexpr int RT = 32;  // tile edge of the pair kernels

__device__ __forceinline__ void pair_index(int64_t b, int64_t& bi, int64_t& bj) {
  // b -> (bi <= bj) over the upper triangle of tile pairs, row by row of bj:
  // bj = floor((sqrt(8b+1)-1)/2), bi = b - bj(bj+1)/2
  int64_t j = int64_t((sqrt(8.0 * double(b) + 1.0) - 1.0) * 0.5);
  while (j * (j + 1) / 2 > b) --j;
  while ((j + 1) * (j + 2) / 2 <= b) ++j;
  bj = j;
  bi = b - j * (j + 1) / 2;
}

// One workgroup per tile pair (bi, bj), (bj, bi): both tiles of C and S are read
// once, along rows, averaged with their transposes, and both tiles of U are
// written along rows.  HBM-bound: 32 bytes read and written per entry.
__global__ void assemble_cs_kernel(const double* __restrict__ Cm, const double* __restrict__ Sm,
                                   int64_t ld, double pr, double pi, c128* __restrict__ U,
                                   int64_t ldu, int64_t N) {
  __shared__ double2 t[RT][RT + 1];
  int64_t bi, bj;
  pair_index(blockIdx.x, bi, bj);
  const int tx = threadIdx.x % RT, ty = threadIdx.x / RT;   // 32 x 8
  for (int r = ty; r < RT; r += TPB / RT) {
    const int64_t i = bj * RT + r, j = bi * RT + tx;
    if (i < N && j < N) t[r][tx] = make_double2(Cm[i * ld + j], Sm[i * ld + j]);
  }
  __syncthreads();
  double2 v[RT / (TPB / RT)];
#pragma unroll
  for (int q = 0; q < RT / (TPB / RT); ++q) {
    const int r = ty + q * (TPB / RT);
    const int64_t i = bi * RT + r, j = bj * RT + tx;
    if (i < N && j < N) {
      const double2 b = t[tx][r];
      const double c = 0.5 * (Cm[i * ld + j] + b.x), s = 0.5 * (Sm[i * ld + j] + b.y);
      v[q] = make_double2(pr * c + pi * s, pi * c - pr * s);    // (pr + i pi)(c - i s)
      U[i * ldu + j] = c128{v[q].x, v[q].y};
    }
  }
  if (bi == bj) return;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < RT / (TPB / RT); ++q) t[tx][ty + q * (TPB / RT)] = v[q];
  __syncthreads();
  for (int r = ty; r < RT; r += TPB / RT) {
    const int64_t i = bj * RT + r, j = bi * RT + tx;
    if (i < N && j < N) U[i * ldu + j] = c128{t[r][tx].x, t[r][tx].y};
  }
}

template <typename E>
__global__ void renorm_kernel(E* __restrict__ rho, int64_t ld, int64_t N, const double* scratch) {
  __shared__ double2 tA[RT][RT + 1];
  __shared__ double2 tB[RT][RT + 1];
  if (scratch[1] != 0.0) return;   // non-finite / non-positive trace: leave rho as is
  const double inv = 1.0 / scratch[0];
  int64_t bi, bj;
  pair_index(blockIdx.x, bi, bj);
  const int tx = threadIdx.x % RT, ty = threadIdx.x / RT;   // 32 x 8
  // load tile (bi, bj) and (bj, bi)
  for (int r = ty; r < RT; r += TPB / RT) {
    const int64_t i = bi * RT + r, j = bj * RT + tx;
    if (i < N && j < N) { const E v = rho[i * ld + j]; tA[r][tx] = make_double2(v.re, v.im); }
    const int64_t i2 = bj * RT + r, j2 = bi * RT + tx;
    if (i2 < N && j2 < N) { const E v = rho[i2 * ld + j2]; tB[r][tx] = make_double2(v.re, v.im); }
  }
  __syncthreads();
  // element (i, j) in tile A pairs with (j, i) = tB[tx][r]
  for (int r = ty; r < RT; r += TPB / RT) {
    const int64_t i = bi * RT + r, j = bj * RT + tx;
    if (i < N && j < N) {
      const double2 a = tA[r][tx], b = tB[tx][r];
      double re = 0.5 * (a.x + b.x) * inv, im = 0.5 * (a.y - b.y) * inv;
      if (i == j) im = 0.0;
      typedef decltype(E().re) T;
      rho[i * ld + j] = E{T(re), T(im)};
      if (bi != bj) rho[j * ld + i] = E{T(re), T(-im)};
    }
  }
}

// ------------------------------------------------------------ observables
// Eq. (13), symmetric reading: <v_m| rho |v_m> with v_m the normalised equal
// sum of the binom(n, m) basis states with m photons and n - m excited atoms,
// i.e. the sum of Re rho_st over those pairs divided by binom(n, m).
// Workgroup (b, mm) of pass 1: wave w takes atom pattern l = 4 b + w as its row
// and sums its row of the photon block mm over the columns with the same
// excitation count; partials[mm nblk + b].
template <typename E>
__device__ __forceinline__ void dicke_rows(int n, int mm, int64_t b, int64_t nblk,
                                           const E* __restrict__ rho, int64_t ld,
                                           double* __restrict__ partials, double* sh) {
  const int64_t per = int64_t(1) << n;
  const int64_t l = b * (TPB / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  double acc = 0.0;
  if (l < per && popc64(uint64_t(l)) == n - mm) {
    const E* row = rho + (mm * per + l) * ld + mm * per;
    for (int64_t t = lane; t < per; t += 64)
      if (popc64(uint64_t(t)) == n - mm) acc += double(row[t].re);
  }
  acc = wave_sum(acc);
  if (lane == 0) sh[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = sh[0];
    for (int w = 1; w < TPB / 64; ++w) r += sh[w];
    partials[int64_t(mm) * nblk + b] = r;
  }
}

// Pass 1: workgroups 0 .. G - 1 walk the tile pairs (bi <= bj), G apart: per
// workgroup the sums of |rho_ij|^2 and of Im rho_ss, the Hermiticity maximum and
// the count of non-finite entries go to partials, the diagonal to diag[].  The
// remaining workgroups take the rows of the Dicke readings.  HBM-bound: every
// entry is read once, the next pair's entries while the current pair is
// reduced.  The squares of the Hermiticity differences are compared and one
// root taken at the end; values whose square leaves the normal range go through
// hypot.
// The whole readout (both passes): N = 5120 complex FP64 240 -> 97 us (4.3
// TB/s), N = 12288 962 -> 441 us (5.5 TB/s), FP32 893 -> 294 us, N = 32 22 -> 13
// us; one workgroup reading every tile pair's sums and all outputs' diagonals in
// turn took half of it before.
template <typename E>
__global__ void __launch_bounds__(TPB)
obs_pass1(const E* __restrict__ rho, int64_t ld, int64_t N, int64_t npairs, int G,
          double* __restrict__ partials, double* __restrict__ diag, int n, int64_t nblk,
          double* __restrict__ dicke) {
  __shared__ double sh[TPB / 64];
  if (int(blockIdx.x) >= G) {
    const int64_t d = int64_t(blockIdx.x) - G;
    dicke_rows(n, int(d / nblk), d % nblk, nblk, rho, ld, dicke, sh);
    return;
  }
  constexpr int Q = RT / (TPB / RT);          // entries of each tile per thread
  __shared__ E tB[RT][RT + 1];
  const int tx = threadIdx.x % RT, ty = threadIdx.x / RT;
  typedef decltype(E().re) T;
  E a[Q], b[Q];
  auto load = [&](int64_t pair, E (&x)[Q], E (&y)[Q]) {
    int64_t bi, bj;
    pair_index(pair, bi, bj);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int r = ty + q * (TPB / RT);
      const int64_t i = bi * RT + r, j = bj * RT + tx;
      x[q] = i < N && j < N ? rho[i * ld + j] : E{T(0), T(0)};
      const int64_t i2 = bj * RT + r, j2 = bi * RT + tx;
      y[q] = i2 < N && j2 < N ? rho[i2 * ld + j2] : E{T(0), T(0)};
    }
  };
  double pur = 0.0, sq = 0.0, far = 0.0, bad = 0.0, tim = 0.0;
  load(blockIdx.x, a, b);
  for (int64_t pair = blockIdx.x; pair < npairs; pair += G) {
    int64_t bi, bj;
    pair_index(pair, bi, bj);
    E na[Q], nb[Q];
    load(pair + G < npairs ? pair + G : pair, na, nb);
#pragma unroll
    for (int q = 0; q < Q; ++q) tB[ty + q * (TPB / RT)][tx] = b[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int r = ty + q * (TPB / RT);
      const E t = tB[tx][r];
      const double ax = double(a[q].re), ay = double(a[q].im);
      if (!isfinite(ax) || !isfinite(ay)) bad += 1.0;
      pur += ax * ax + ay * ay;
      if (bi != bj) {
        const double bx = double(b[q].re), by = double(b[q].im);
        if (!isfinite(bx) || !isfinite(by)) bad += 1.0;
        pur += bx * bx + by * by;
      }
      const double dx = ax - double(t.re), dy = ay + double(t.im);
      const double s = dx * dx + dy * dy;
      if (s >= 1e-290 && s <= 1e290) sq = fmax(sq, s);
      else if (dx != 0.0 || dy != 0.0) far = fmax(far, hypot(dx, dy));
      if (bi == bj && r == tx) {
        const int64_t i = bi * RT + r;
        if (i < N) diag[i] = ax;
        tim += ay;                            // 0 past the matrix
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      a[q] = na[q];
      b[q] = nb[q];
    }
  }
  const double P = block_sum(pur, sh);
  const double Hm = block_max(fmax(sqrt(sq), far), sh);
  const double B = block_sum(bad, sh);
  const double I = block_sum(tim, sh);
  if (threadIdx.x == 0) {
    double* out = partials + 4 * int64_t(blockIdx.x);
    out[0] = P;
    out[1] = Hm;
    out[2] = B;
    out[3] = I;
  }
}

// Pass 2: one workgroup per output: 0 the sums over pass 1's workgroups, 1 the
// diagonal's scalars, then atom_pop, photon_dist, photon_state, exc_dist and
// dicke entry by entry (those whose pointer is not NULL have workgroups).
struct ObsOut {
  double *scalars, *atom_pop, *photon_dist, *photon_state, *exc_dist, *dicke;
};

__global__ void __launch_bounds__(TPB)
obs_pass2(int n, int c, int64_t N, const double* __restrict__ partials, int G,
          const double* __restrict__ diag, const double* __restrict__ dpart, int64_t nblk,
          ObsOut o) {
  __shared__ double sh[TPB / 64];
  const uint64_t mask = (uint64_t(1) << n) - 1;
  const int64_t per = int64_t(1) << n;
  const bool first = threadIdx.x == 0;
  int w = blockIdx.x;
  if (w == 0) {
    double pur = 0.0, herm = 0.0, bad = 0.0, tim = 0.0;
    for (int b = threadIdx.x; b < G; b += TPB) {
      pur += partials[4 * b];
      herm = fmax(herm, partials[4 * b + 1]);
      bad += partials[4 * b + 2];
      tim += partials[4 * b + 3];
    }
    pur = block_sum(pur, sh);
    herm = block_max(herm, sh);
    bad = block_sum(bad, sh);
    tim = block_sum(tim, sh);
    if (first) {
      o.scalars[1] = tim;
      o.scalars[2] = pur;
      o.scalars[3] = herm;
      o.scalars[7] = bad > 0.0 ? 1.0 : 0.0;
    }
    return;
  }
  if (w == 1) {
    double tr = 0.0, ex = 0.0, ph = 0.0, nx = 0.0;
    for (int64_t s = threadIdx.x; s < N; s += TPB) {
      const double d = diag[s];
      const int pc = popc64(uint64_t(s) & mask);
      const int64_t mm = s >> n;
      tr += d;
      ex += double(pc) * d;
      ph += double(mm) * d;
      nx += double(mm + pc) * d;
    }
    tr = block_sum(tr, sh);
    ex = block_sum(ex, sh);
    ph = block_sum(ph, sh);
    nx = block_sum(nx, sh);
    if (first) {
      o.scalars[0] = tr;
      o.scalars[4] = ex;
      o.scalars[5] = ph;
      o.scalars[6] = nx;
    }
    return;
  }
  w -= 2;
  if (o.atom_pop) {
    if (w < n) {
      double p = 0.0;
      for (int64_t s = threadIdx.x; s < N; s += TPB)
        if ((uint64_t(s) >> (n - 1 - w)) & 1) p += diag[s];
      p = block_sum(p, sh);
      if (first) o.atom_pop[w] = p;
      return;
    }
    w -= n;
  }
  if (o.photon_dist) {
    if (w <= c) {
      double p = 0.0;
      for (int64_t s = w * per + threadIdx.x; s < (w + 1) * per; s += TPB) p += diag[s];
      p = block_sum(p, sh);
      if (first) o.photon_dist[w] = p;
      return;
    }
    w -= c + 1;
  }
  const int ns = (n < c ? n : c) + 1;
  if (o.photon_state) {
    // Eq. (13), sector reading: m photons and n - m excited atoms
    if (w < ns) {
      double p = 0.0;
      for (int64_t s = w * per + threadIdx.x; s < (w + 1) * per; s += TPB)
        if (popc64(uint64_t(s) & mask) == n - w) p += diag[s];
      p = block_sum(p, sh);
      if (first) o.photon_state[w] = p;
      return;
    }
    w -= ns;
  }
  if (o.exc_dist) {
    if (w <= n + c) {
      double p = 0.0;
      for (int64_t s = threadIdx.x; s < N; s += TPB)
        if (int(s >> n) + popc64(uint64_t(s) & mask) == w) p += diag[s];
      p = block_sum(p, sh);
      if (first) o.exc_dist[w] = p;
      return;
    }
    w -= n + c + 1;
  }
  // symmetric reading: the sum of the rows' partials / binom(n, m)
  double p = 0.0;
  for (int64_t b = threadIdx.x; b < nblk; b += TPB) p += dpart[int64_t(w) * nblk + b];
  p = block_sum(p, sh);
  if (first) {
    double binom = 1.0;
    for (int j = 1; j <= w; ++j) binom = binom * double(n - w + j) / double(j);
    o.dicke[w] = p / binom;
  }
}

// ------------------------------------------------------------ adjoint helpers
template <typename E>
__global__ void excitation_op_kernel(ModelArgs m, E* __restrict__ O, int64_t ld) {
  const int64_t col = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (col >= m.N) return;
  const uint64_t mask = (uint64_t(1) << m.n) - 1;
  typedef decltype(E().re) T;
  for (int64_t row = blockIdx.y; row < m.N; row += gridDim.y) {
    const T v = row == col ? T(popc64(uint64_t(row) & mask)) : T(0);
    O[row * ld + col] = E{v, T(0)};
  }
}

__global__ void accumulate_c64_kernel(const c64* __restrict__ T, int64_t ldt, c128* __restrict__ M,
                                      int64_t ldm, int64_t N) {
  const int64_t col = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (col >= N) return;
  for (int64_t row = blockIdx.y; row < N; row += gridDim.y) {
    const c64 t = T[row * ldt + col];
    c128 v = M[row * ldm + col];
    v.re += double(t.re);
    v.im += double(t.im);
    M[row * ldm + col] = v;
  }
}

__global__ void shifted_h_kernel(ModelArgs m, const double* __restrict__ H, int64_t ldh, double mu,
                                 double scale, double* __restrict__ out) {
  const int64_t col = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (col >= m.N) return;
  for (int64_t row = blockIdx.y; row < m.N; row += gridDim.y) {
    double h = H[row * ldh + col];
    if (row == col) h -= m.omega_c * double(exc_number(row, m.n)) + mu;
    out[row * m.N + col] = h * scale;
  }
}

// One workgroup per tile pair: both tiles of M are read along rows and both
// tiles of the planes written along rows.
__global__ void sym_planes_kernel(const c128* __restrict__ M, int64_t N, double a,
                                  double* __restrict__ re, double* __restrict__ im) {
  __shared__ double2 tA[RT][RT + 1];
  __shared__ double2 tB[RT][RT + 1];
  int64_t bi, bj;
  pair_index(blockIdx.x, bi, bj);
  const int tx = threadIdx.x % RT, ty = threadIdx.x / RT;   // 32 x 8
  for (int r = ty; r < RT; r += TPB / RT) {
    const int64_t i = bi * RT + r, j = bj * RT + tx;
    if (i < N && j < N) { const c128 v = M[i * N + j]; tA[r][tx] = make_double2(v.re, v.im); }
    const int64_t i2 = bj * RT + r, j2 = bi * RT + tx;
    if (i2 < N && j2 < N) { const c128 v = M[i2 * N + j2]; tB[r][tx] = make_double2(v.re, v.im); }
  }
  __syncthreads();
  for (int r = ty; r < RT; r += TPB / RT) {
    const int64_t i = bi * RT + r, j = bj * RT + tx;
    if (i < N && j < N) {
      const double2 p = tA[r][tx], q = tB[tx][r];
      re[i * N + j] = 0.5 * a * (p.x + q.x);
      im[i * N + j] = 0.5 * a * (p.y + q.y);
    }
    const int64_t i2 = bj * RT + r, j2 = bi * RT + tx;
    if (bi != bj && i2 < N && j2 < N) {
      const double2 p = tB[r][tx], q = tA[tx][r];
      re[i2 * N + j2] = 0.5 * a * (p.x + q.x);
      im[i2 * N + j2] = 0.5 * a * (p.y + q.y);
    }
  }
}

// One workgroup per parameter: blocks 0..n-1 give dL/dg_i, n..2n-1 dL/ddelta_i.
__global__ void grad_trace_kernel(ModelArgs m, const double* __restrict__ Gr,
                                  const double* __restrict__ Gi, int stride, int64_t ld, double pr,
                                  double pi, double dt, double* __restrict__ grad_g,
                                  double* __restrict__ grad_delta) {
  __shared__ double sh[TPB / 64];
  const int n = m.n;
  const int p = blockIdx.x;
  const int i = p % n;
  const int64_t per = int64_t(1) << n;
  const uint64_t bit = uint64_t(1) << (n - 1 - i);
  double acc = 0.0;   // Im(ph * sum)
  if (p < n) {
    // pairs s = (mm, l) with bit set, mm < c; t = s + 2^n - bit
    for (int64_t s = threadIdx.x; s < int64_t(m.c) * per; s += TPB) {
      if (!(uint64_t(s) & bit)) continue;
      const int64_t t = s + per - int64_t(bit);
      const double w = sqrt(double((s >> n) + 1));
      const int64_t a = (s * ld + t) * stride, b = (t * ld + s) * stride;
      const double zr = w * (Gr[a] + Gr[b]), zi = w * (Gi[a] + Gi[b]);
      acc += pr * zi + pi * zr;
    }
  } else {
    for (int64_t s = threadIdx.x; s < m.N; s += TPB) {
      if (!(uint64_t(s) & bit)) continue;
      const int64_t a = s * (ld + 1) * stride;
      acc += pr * Gi[a] + pi * Gr[a];
    }
  }
  const double tot = block_sum(acc, sh);
  if (threadIdx.x == 0) {
    if (p < n) grad_g[i] = 2.0 * dt * tot;
    else grad_delta[i] = 2.0 * dt * tot;
  }
}

// --------------------------------------------------------- bfloat16 split
__device__ __forceinline__ uint16_t rne_bf16(float x) {
  const uint32_t b = __float_as_uint(x);
  if ((b & 0x7F800000u) == 0x7F800000u && (b & 0x007FFFFFu) != 0)
    return uint16_t((b >> 16) | 0x40u);                       // NaN stays (quiet) NaN
  const uint32_t upper = b >> 16, rem = b & 0xFFFFu;
  const uint32_t up = (rem > 0x8000u) || (rem == 0x8000u && (upper & 1u));
  return uint16_t(upper + up);
}

__global__ void split_bf16_kernel(const float* __restrict__ x, int64_t count,
                                  uint16_t* __restrict__ hi, uint16_t* __restrict__ lo) {
  for (int64_t i = int64_t(blockIdx.x) * TPB + threadIdx.x; i < count;
       i += int64_t(gridDim.x) * TPB) {
    const float v = x[i];
    const uint16_t h = rne_bf16(v);
    const float r = v - __uint_as_float(uint32_t(h) << 16);
    hi[i] = h;
    lo[i] = rne_bf16(r);
  }
}

dim3 grid2(int64_t cols, int64_t rows) {
  const int64_t gx = (cols + TPB - 1) / TPB;
  const int64_t gy = rows < 4096 ? rows : 4096;
  return dim3(unsigned(gx > 0 ? gx : 1), unsigned(gy > 0 ? gy : 1));
}

unsigned grid1(int64_t count) {
  const int64_t g = (count + TPB - 1) / TPB;
  return unsigned(g < 16384 ? g : 16384);
}

int64_t npairs_of(int64_t N) {
  const int64_t T = (N + RT - 1) / RT;
  return T * (T + 1) / 2;
}

}  // namespace

int launch_ham_fill(const ModelArgs& m, double* H, int64_t ldh, hipStream_t s) {
  if (m.N == 0) return TC_OK;
  hipLaunchKernelGGL(ham_fill_kernel, grid2(m.N, m.N), dim3(TPB), 0, s, m, H, ldh);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_axpb_identity(const double* X, int64_t ldx, double a, double b, double* out,
                         int64_t ldo, int64_t N, hipStream_t s) {
  if (N == 0) return TC_OK;
  hipLaunchKernelGGL(axpb_identity_kernel, grid2(N, N), dim3(TPB), 0, s, X, ldx, a, b, out, ldo, N);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_assemble_cs(const double* Cm, const double* Sm, int64_t ld, double pr, double pi,
                       c128* U, int64_t ldu, int64_t N, hipStream_t s) {
  if (N == 0) return TC_OK;
  hipLaunchKernelGGL(assemble_cs_kernel, dim3(unsigned(npairs_of(N))), dim3(TPB), 0, s, Cm, Sm, ld,
                     pr, pi, U, ldu, N);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_lin_powers(const double* X, const double* X2, const double* X3, int64_t N, LinCoef c0,
                      double* out0, LinCoef c1, double* out1, LinCoef c2, double* out2,
                      hipStream_t s) {
  if (N == 0) return TC_OK;
  hipLaunchKernelGGL(lin_powers_kernel, dim3(grid1(N * N)), dim3(TPB), 0, s, X, X2, X3, N * N, N,
                     c0, out0, c1, out1, c2, out2);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_diff_sum(const double* C, const double* S, double* D, double* E, int64_t N,
                    hipStream_t s) {
  if (N == 0) return TC_OK;
  hipLaunchKernelGGL(diff_sum_kernel, dim3(grid1(N * N)), dim3(TPB), 0, s, C, S, D, E, N * N);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_copy_c128_to_c64(const c128* src, int64_t lds, c64* dst, int64_t ldd, int64_t rows,
                            int64_t cols, hipStream_t s) {
  if (rows == 0 || cols == 0) return TC_OK;
  hipLaunchKernelGGL(c128_to_c64_kernel, grid2(cols, rows), dim3(TPB), 0, s, src, lds, dst, ldd, rows, cols);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_copy_c64_to_c128(const c64* src, int64_t lds, c128* dst, int64_t ldd, int64_t rows,
                            int64_t cols, hipStream_t s) {
  if (rows == 0 || cols == 0) return TC_OK;
  hipLaunchKernelGGL(c64_to_c128_kernel, grid2(cols, rows), dim3(TPB), 0, s, src, lds, dst, ldd, rows, cols);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_rotating_d(const ModelArgs& m, const c128* U, int64_t ldu, double dt, c128* D,
                      int64_t ldd, hipStream_t s) {
  if (m.N == 0) return TC_OK;
  hipLaunchKernelGGL(rotating_d_kernel<c128>, grid2(m.N, m.N), dim3(TPB), 0, s, m, U, ldu, dt, D, ldd);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_rotating_d_c64(const ModelArgs& m, const c128* U, int64_t ldu, double dt, c64* D,
                          int64_t ldd, hipStream_t s) {
  if (m.N == 0) return TC_OK;
  hipLaunchKernelGGL(rotating_d_kernel<c64>, grid2(m.N, m.N), dim3(TPB), 0, s, m, U, ldu, dt, D, ldd);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_frame_phase_c128(const ModelArgs& m, c128* rho, int64_t ld, double t, hipStream_t s) {
  if (m.N == 0) return TC_OK;
  hipLaunchKernelGGL(frame_phase_kernel<c128>, grid2(m.N, m.N), dim3(TPB), 0, s, m, rho, ld, t);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_frame_phase_c64(const ModelArgs& m, c64* rho, int64_t ld, double t, hipStream_t s) {
  if (m.N == 0) return TC_OK;
  hipLaunchKernelGGL(frame_phase_kernel<c64>, grid2(m.N, m.N), dim3(TPB), 0, s, m, rho, ld, t);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

template <typename E, int L>
int launch_cavity(const ModelArgs& m, E* rho, int64_t ld, double eta, hipStream_t s) {
  CavityCoef<L> k;
  k.odd = eta > 1.0 ? -1.0 : 1.0;
  for (int mm = 0; mm < L; ++mm) {
    double v = std::pow(eta, 0.5 * mm);
    for (int l = 0; l < L; ++l) {
      if (l > 0) v *= std::sqrt(double(mm + l) / double(l) * std::fabs(1.0 - eta));
      k.a[mm * L + l] = v;
    }
  }
  const int64_t pairs = int64_t(1) << (2 * m.n);
  hipLaunchKernelGGL((damp_cavity_reg_kernel<E, L>),
                     dim3(unsigned((pairs + TPB - 1) / TPB), unsigned(2 * m.c + 1)), dim3(TPB), 0, s,
                     rho, ld, m.n, m.c, k);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

template <typename E>
int launch_dissipation_t(const ModelArgs& m, E* rho, int64_t ld, double dt, hipStream_t s) {
  if (m.N == 0) return TC_OK;
  if (m.gamma > 0.0) {
    const double p = -expm1(-m.gamma * dt);        // 1 - e^{-gamma dt}
    const double f = sqrt(1.0 - p);
    // atoms on bits 0 .. 5 in one pass
    int b = m.n < 6 ? m.n : 6;
    const unsigned tiles = unsigned((m.N + D6 - 1) / D6);
    hipLaunchKernelGGL(damp_atoms6_kernel<E>, dim3(tiles, tiles), dim3(TPB), 0,
                       s, rho, ld, m.N, b, p, f);
    TC_TRY_HIP(hipGetLastError());
    if constexpr (std::is_same<E, c64>::value) {
      for (; b + 3 <= m.n; b += 3) {
        // Bits 6 .. 8 take the coalesced pass: its 512-column windows hold their
        // column groups of 8 2^6 exactly.  The groups of higher bits need wider
        // windows than LDS has room for, and an odd row stride breaks the 16-byte
        // alignment: those take the per-block kernel.
        if (b == 6 && ld % 2 == 0 && (reinterpret_cast<uintptr_t>(rho) & 15) == 0) {
          constexpr int W = 512;
          const size_t lds = size_t(8) * size_t(W + W / 8 + 2) * sizeof(float2);
          const int64_t groups = m.N >> 3;
          hipLaunchKernelGGL(damp_atoms3_lds_c64_kernel,
                             dim3(unsigned(m.N / W), unsigned(groups < 4096 ? groups : 4096)),
                             dim3(unsigned(W / 4)), lds, s, rho, ld, m.N, b, W, float(p), float(f));
        } else {
          const int64_t R = m.N >> 3;            // two lanes per 8 x 8 block
          hipLaunchKernelGGL(damp_atoms3_c64_kernel, grid2(2 * R, R), dim3(TPB), 0, s, rho, ld,
                             m.N, b, b + 1, b + 2, float(p), float(f));
        }
        TC_TRY_HIP(hipGetLastError());
      }
    }
    for (; b < m.n; b += 2) {
      if (b + 1 < m.n) {
        const int64_t R = m.N >> 2;
        hipLaunchKernelGGL((damp_atoms_kernel<E, 2>), grid2(R, R), dim3(TPB), 0, s, rho, ld, m.N,
                           b, b + 1, p, f);
      } else {
        const int64_t R = m.N >> 1;
        hipLaunchKernelGGL((damp_atoms_kernel<E, 1>), grid2(R, R), dim3(TPB), 0, s, rho, ld, m.N,
                           b, -1, p, f);
      }
      TC_TRY_HIP(hipGetLastError());
    }
  }
  if (m.kappa > 0.0 && m.c > 0) {
    const double eta = exp(-m.kappa * dt);
    if (m.c + 1 <= 8) return launch_cavity<E, 8>(m, rho, ld, eta, s);
    if (m.c + 1 <= 16) return launch_cavity<E, 16>(m, rho, ld, eta, s);
    const int64_t per = int64_t(1) << m.n;
    hipLaunchKernelGGL(damp_cavity_kernel<E>,
                       dim3(unsigned((per + TPB - 1) / TPB), unsigned(per < 4096 ? per : 4096),
                            unsigned(2 * m.c + 1)),
                       dim3(TPB), 0, s, rho, ld, m.n, m.c, eta);
    TC_TRY_HIP(hipGetLastError());
  }
  return TC_OK;
}

int launch_dissipation_c128(const ModelArgs& m, c128* rho, int64_t ld, double dt, hipStream_t s) {
  return launch_dissipation_t(m, rho, ld, dt, s);
}

int launch_dissipation_c64(const ModelArgs& m, c64* rho, int64_t ld, double dt, hipStream_t s) {
  return launch_dissipation_t(m, rho, ld, dt, s);
}

int launch_readout_c128(const ModelArgs& m, const c128* rho, int64_t ld, double* pop,
                        double* pdist, hipStream_t s, const int32_t* map, double* pstate,
                        const int32_t* off, int k) {
  hipLaunchKernelGGL(readout_kernel<c128>, dim3(1), dim3(READOUT_NT), 0, s, m, rho, ld, map, off, k,
                     pop, pdist, pstate);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_readout_c64(const ModelArgs& m, const c64* rho, int64_t ld, double* pop,
                       double* pdist, hipStream_t s, const int32_t* map, double* pstate,
                       const int32_t* off, int k) {
  hipLaunchKernelGGL(readout_kernel<c64>, dim3(1), dim3(READOUT_NT), 0, s, m, rho, ld, map, off, k,
                     pop, pdist, pstate);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

template <typename E>
static int renorm_impl(E* rho, int64_t ld, int64_t N, double* scratch, hipStream_t s) {
  if (N == 0) return TC_OK;
  hipLaunchKernelGGL(trace_kernel<E>, dim3(1), dim3(TPB), 0, s, rho, ld, N, scratch);
  TC_TRY_HIP(hipGetLastError());
  const int64_t np = npairs_of(N);
  hipLaunchKernelGGL(renorm_kernel<E>, dim3(unsigned(np)), dim3(TPB), 0, s, rho, ld, N, scratch);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_renorm_c128(c128* rho, int64_t ld, int64_t N, double* scratch, hipStream_t s) {
  return renorm_impl(rho, ld, N, scratch, s);
}
int launch_renorm_c64(c64* rho, int64_t ld, int64_t N, double* scratch, hipStream_t s) {
  return renorm_impl(rho, ld, N, scratch, s);
}

// The partials buffer's size.  Its layout: 4 per workgroup of pass 1 (G of them,
// at most OBS_WGS and at most one per tile pair), the diagonal (N), the Dicke
// partials ((min(n, c) + 1) ceil(2^n / 4) <= N / 4 for n >= 3, at most 3 below).
constexpr int OBS_WGS = 1024;

size_t observables_partials_count(int64_t N) {
  return size_t(3 * npairs_of(N) + N + 8 + N);
}

int launch_observables(const ModelArgs& m, const void* rho, int dtype, int64_t ld,
                       double* partials, double* scalars, double* atom_pop,
                       double* photon_dist, double* exc_dist, double* photon_state,
                       double* dicke, hipStream_t s) {
  const int64_t N = m.N;
  const int64_t np = npairs_of(N);
  const int G = int(np < OBS_WGS ? np : OBS_WGS);
  double* diag = partials + 4 * int64_t(G);
  double* dpart = diag + N;
  const int64_t per = int64_t(1) << m.n;
  const int64_t nblk = (per + TPB / 64 - 1) / (TPB / 64);
  const int ns = (m.n < m.c ? m.n : m.c) + 1;
  if (size_t(4 * int64_t(G) + N + ns * nblk) > observables_partials_count(N)) {
    set_error("observables: the partial sums exceed their buffer");
    return TC_ERR_WORKSPACE;
  }
  const dim3 grid(unsigned(G + (dicke ? ns * nblk : 0)));
  if (dtype == TC_C128)
    hipLaunchKernelGGL(obs_pass1<c128>, grid, dim3(TPB), 0, s, static_cast<const c128*>(rho), ld, N,
                       np, G, partials, diag, m.n, nblk, dpart);
  else
    hipLaunchKernelGGL(obs_pass1<c64>, grid, dim3(TPB), 0, s, static_cast<const c64*>(rho), ld, N,
                       np, G, partials, diag, m.n, nblk, dpart);
  TC_TRY_HIP(hipGetLastError());
  const ObsOut o{scalars, atom_pop, photon_dist, photon_state, exc_dist, dicke};
  const int outs = 2 + (atom_pop ? m.n : 0) + (photon_dist ? m.c + 1 : 0) +
                   (photon_state ? ns : 0) + (exc_dist ? m.n + m.c + 1 : 0) + (dicke ? ns : 0);
  hipLaunchKernelGGL(obs_pass2, dim3(unsigned(outs)), dim3(TPB), 0, s, m.n, m.c, N, partials, G,
                     diag, dpart, nblk, o);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_split_bf16(const float* x, int64_t count, uint16_t* hi, uint16_t* lo, hipStream_t s) {
  if (count == 0) return TC_OK;
  int64_t blocks = (count + TPB - 1) / TPB;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(split_bf16_kernel, dim3(unsigned(blocks)), dim3(TPB), 0, s, x, count, hi, lo);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_grouped_readout(const ReadoutItem* items_dev, int count, bool c128_storage,
                           int* counter, hipStream_t s) {
  if (count == 0) return TC_OK;
  if (c128_storage)
    hipLaunchKernelGGL(grouped_readout_kernel<c128>, dim3(unsigned(count)), dim3(READOUT_NT), 0, s,
                       items_dev, counter);
  else
    hipLaunchKernelGGL(grouped_readout_kernel<c64>, dim3(unsigned(count)), dim3(READOUT_NT), 0, s,
                       items_dev, counter);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_excitation_op_c128(const ModelArgs& m, c128* O, int64_t ld, hipStream_t s) {
  if (m.N == 0) return TC_OK;
  hipLaunchKernelGGL(excitation_op_kernel<c128>, grid2(m.N, m.N), dim3(TPB), 0, s, m, O, ld);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_excitation_op_c64(const ModelArgs& m, c64* O, int64_t ld, hipStream_t s) {
  if (m.N == 0) return TC_OK;
  hipLaunchKernelGGL(excitation_op_kernel<c64>, grid2(m.N, m.N), dim3(TPB), 0, s, m, O, ld);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_accumulate_c64(const c64* T, int64_t ldt, c128* M, int64_t ldm, int64_t N,
                          hipStream_t s) {
  if (N == 0) return TC_OK;
  hipLaunchKernelGGL(accumulate_c64_kernel, grid2(N, N), dim3(TPB), 0, s, T, ldt, M, ldm, N);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_shifted_h(const ModelArgs& m, const double* H, int64_t ldh, double mu, double scale,
                     double* out, int64_t N, hipStream_t s) {
  if (m.N == 0) return TC_OK;
  hipLaunchKernelGGL(shifted_h_kernel, grid2(N, N), dim3(TPB), 0, s, m, H, ldh, mu, scale, out);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_sym_planes(const c128* M, int64_t N, double a, double* re, double* im, hipStream_t s) {
  if (N == 0) return TC_OK;
  hipLaunchKernelGGL(sym_planes_kernel, dim3(unsigned(npairs_of(N))), dim3(TPB), 0, s, M, N, a, re,
                     im);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

int launch_grad_trace(const ModelArgs& m, const double* Gr, const double* Gi, int stride,
                      int64_t ld, double ph_re, double ph_im, double dt, double* grad_g,
                      double* grad_delta, hipStream_t s) {
  hipLaunchKernelGGL(grad_trace_kernel, dim3(unsigned(2 * m.n)), dim3(TPB), 0, s, m, Gr, Gi, stride,
                     ld, ph_re, ph_im, dt, grad_g, grad_delta);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

}  // namespace tcm
