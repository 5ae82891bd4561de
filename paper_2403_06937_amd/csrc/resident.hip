// LDS-resident stepping of small instances: every step of Eq. (6) in a single
// launch, one workgroup per instance, with the product operand, rho and the
// intermediate X held in LDS for the whole run.
//
// At N = 32 a step is two 32 x 32 x 32 complex products (0.5 Mflop), far too
// little to fill even one CU; launched as separate kernels per step the run
// is bound by launch latency.  Here the launch is paid once per run (it also
// forms the operand and undoes the frame) and each step costs the products'
// arithmetic and two workgroup barriers.
//
// Per step, for every output (i, j):
//   X[i][j]  = sum_k op[i][k] R[k][j]        (+ R[i][j] in the rotating frame)
//   R'[i][j] = sum_k X[i][k] conj(op[j][k])  (+ X[i][j] in the rotating frame)
// i.e. X = op R, R' = X op^dag: op = U in the lab frame, D = U~ - I in the
// rotating frame (U~ = I + D).  The matrices sit in LDS padded with zeros to
// 16 NB, and each of four waves forms 16 x 16 output blocks of one block row
// with the 16 x 16 x 4 MFMA of the storage precision (four real products per
// complex block, FP64 or FP32 accumulation).  Renormalisation (every
// renorm_every steps) is Hermitisation and division by Re Tr R in FP64, and the
// records (excited-atom population, photon-number distribution, P({m>) of
// Eq. (13)) are read from the diagonal in FP64 by a fifth wave.
//
// Bound by the MFMA issue of one CU (N = 32 FP64: 32 instructions of 64 cycles
// per wave and product, 1.7 us a step) plus the latency between the two
// products.  To keep that small the K loop is unrolled for each NB, the waves'
// op fragments stay in registers for the whole run (they never change; with one
// block per wave both products' fragments), and the barriers wait for LDS only,
// not for the record wave's stores.  Per step with two kinds of records: FP64
// N = 32 4.18 -> 2.60 us (2.35 without records), N = 48 10.8 -> 9.4, FP32 N = 64
// 11.3 -> 9.4.  Reading all of a product's other fragments ahead of its first
// MFMA made N = 32 slower (2.82 -> 3.11 us at the time).
#include <cmath>

#include "kernels.h"
#include "mfma.h"

namespace tcm {
namespace {

constexpr int PWAVES = 4;                  // waves that form the product blocks
constexpr int RTPB = 64 * (PWAVES + 1);    // plus one wave for the records

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Workgroup barrier that waits for this wave's LDS accesses, not for its
// global stores (the records).
__device__ __forceinline__ void sync_lds() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <typename T> struct Acc;
template <> struct Acc<double> {
  typedef d4 type;
  static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <> struct Acc<float> {
  typedef f4 type;
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// many: one item per workgroup in device memory, or NULL for `one`.
template <typename T, int NB>
__global__ void __launch_bounds__(RTPB)
resident_kernel(const ResidentItem one, const ResidentItem* __restrict__ many, ResidentRun a) {
  typedef cplx<T> E;
  typedef typename Acc<T>::type V;
  constexpr int NP = 16 * NB, KS = 4 * NB;
  // waves to a block row, blocks per wave; with one block per wave the second
  // product's operand fragments stay in registers too
  constexpr int WPR = NB == 1 ? 1 : NB == 2 ? 2 : 1, CPW = NB / WPR;
  constexpr bool HOLD2 = CPW == 1;
  // one element of padding per row: the 16 rows of a fragment read fall on
  // distinct banks
  constexpr int LD = NP + 1;
  __shared__ E sU[NP * LD];
  __shared__ E sA[NP * LD];
  __shared__ E sB[NP * LD];
  __shared__ int bad;
  __shared__ double trace;
  const ResidentItem it = many ? many[blockIdx.x] : one;
  const int N = it.N, n = it.n, c = it.c;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t mask = (1u << n) - 1;
  // excitation number of position s (one sector: k for all)
  auto exc = [&](int s) { return it.k >= 0 ? it.k : (s >> n) + __popc(uint32_t(s) & mask); };
  for (int idx = threadIdx.x; idx < NP * NP; idx += RTPB) {
    const int i = idx / NP, j = idx - (idx / NP) * NP;
    E u{T(0), T(0)}, r{T(0), T(0)};
    if (i < N && j < N) {
      c128 v = it.U[int64_t(i) * it.ldu + j];
      if (a.rot) {                        // e^{i w_c k_i dt} U - I
        double sn, cs;
        sincos(it.omega_c * double(exc(i)) * a.dt, &sn, &cs);
        v = c128{cs * v.re - sn * v.im, cs * v.im + sn * v.re};
        if (i == j) v.re -= 1.0;
      }
      u = E{T(v.re), T(v.im)};
      if (a.rho_c128) {
        const c128 x = static_cast<const c128*>(it.rho)[int64_t(i) * it.ldr + j];
        r = E{T(x.re), T(x.im)};
      } else {
        const c64 x = static_cast<const c64*>(it.rho)[int64_t(i) * it.ldr + j];
        r = E{T(x.re), T(x.im)};
      }
    }
    sU[i * LD + j] = u;
    sA[i * LD + j] = r;
  }
  if (threadIdx.x == 0) {
    bad = 0;
    it.scratch[0] = 0.0;
    it.scratch[1] = 0.0;
  }
  __syncthreads();
  E* R = sA;
  E* X = sB;
  const int ns = (n < c ? n : c) + 1;
  const bool rec = it.pop || it.pdist || it.pstate;
  const int lr = lane & 15, lk = lane >> 4;
  const bool works = wave < WPR * NB;
  const int i0 = 16 * (wave / WPR), jb = (wave % WPR) * CPW;

  // lane m of the record wave owns photon number m (c + 1 <= N <= 64): its
  // states are first .. last - 1
  int first = 0, last = 0;
  if (wave == PWAVES && lane <= c) {
    if (it.k < 0) {
      first = lane << n;
      last = first + (1 << n);
    } else {
      for (int m = 0; m <= lane; ++m) {
        const int e = it.k - m;             // C(n, e) states
        int cnt = e >= 0 && e <= n ? 1 : 0;
        for (int q = 1; cnt && q <= e; ++q) cnt = cnt * (n - e + q) / q;
        first = last;
        last += cnt;
      }
    }
  }
  // records of R's diagonal, by the last wave while the others run the next
  // step's first product (which only reads R)
  auto record = [&](int64_t r) {
    if (wave != PWAVES) return;
    double part = 0.0, st = 0.0, ex = 0.0;
    for (int s0 = first; s0 < last; s0 += 8) {
      double d[8];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        d[q] = s0 + q < last ? double(R[(s0 + q) * (LD + 1)].re) : 0.0;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int pc = it.k >= 0 ? it.k - lane : __popc(uint32_t(s0 + q) & mask);
        part += d[q];
        ex += double(pc) * d[q];
        if (pc == n - lane) st += d[q];
      }
    }
    if (it.pdist && lane <= c) it.pdist[r * (c + 1) + lane] = part;
    if (it.pstate && lane < ns) it.pstate[r * ns + lane] = st;
    if (it.pop) {
      for (int o = 1; o <= c; o <<= 1) ex += __shfl_xor(ex, o, 64);   // lanes past c hold 0
      if (lane == 0) it.pop[r] = ex;
    }
  };

  // operand fragments for the whole run: A[i][k] = op[i][k] of the first
  // product, and B[k][j] = conj(op[j][k]) of the second (sign left to the MFMA)
  E u1[KS], u2[HOLD2 ? KS : 1];
  if (works) {
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      u1[q] = sU[(i0 + lr) * LD + 4 * q + lk];
      if constexpr (HOLD2) u2[q] = sU[(16 * jb + lr) * LD + 4 * q + lk];
    }
  }
  auto finish_block = [&](E* dst, const E* add, const V (&re)[CPW], const V (&im)[CPW]) {
#pragma unroll
    for (int b = 0; b < CPW; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = (i0 + Acc<T>::row(lane, r)) * LD + 16 * (jb + b) + lr;
        T xr = re[b][r], xi = im[b][r];
        if (a.rot) {
          const E y = add[o];
          xr += y.re;
          xi += y.im;
        }
        dst[o] = E{xr, xi};
      }
  };

  // the record wave shares a SIMD with a product wave; its few instructions go
  // first (complex FP32 N = 64 with records 10.0 -> 9.4 us a step)
  if (wave == PWAVES) __builtin_amdgcn_s_setprio(3);
  if (rec) record(0);
  // step counts at which the next renormalisation and record fall
  int64_t next_renorm = a.renorm_every > 0 ? a.renorm_every : -1;
  int64_t next_record = a.record_every, rindex = 0;
  for (int64_t step = 1; step <= a.steps; ++step) {
    // X = op R (+ R).  The padding of op and R is zero, so X's padding is too.
    if (works) {
      V re[CPW], im[CPW];
#pragma unroll
      for (int b = 0; b < CPW; ++b) re[b] = im[b] = V{0, 0, 0, 0};
#pragma unroll
      for (int q = 0; q < KS; ++q)
#pragma unroll
        for (int b = 0; b < CPW; ++b) {
          const E y = R[(4 * q + lk) * LD + 16 * (jb + b) + lr];
          re[b] = mma(u1[q].re, y.re, re[b]);
          im[b] = mma(u1[q].re, y.im, im[b]);
          re[b] = mma_nega(u1[q].im, y.im, re[b]);
          im[b] = mma(u1[q].im, y.re, im[b]);
        }
      finish_block(X, R, re, im);
    }
    sync_lds();
    // R = X op^dag (+ X)
    if (works) {
      V re[CPW], im[CPW];
#pragma unroll
      for (int b = 0; b < CPW; ++b) re[b] = im[b] = V{0, 0, 0, 0};
#pragma unroll
      for (int q = 0; q < KS; ++q) {
        const E x = X[(i0 + lr) * LD + 4 * q + lk];
#pragma unroll
        for (int b = 0; b < CPW; ++b) {
          E y;
          if constexpr (HOLD2) y = u2[q];
          else y = sU[(16 * (jb + b) + lr) * LD + 4 * q + lk];
          re[b] = mma(x.re, y.re, re[b]);
          im[b] = mma(x.im, y.re, im[b]);
          re[b] = mma(x.im, y.im, re[b]);
          im[b] = mma_nega(x.re, y.im, im[b]);
        }
      }
      finish_block(R, X, re, im);
    }
    sync_lds();
    if (step == next_renorm) {
      next_renorm += a.renorm_every;
      if (threadIdx.x < 64) {
        const double tr = wave_sum(lane < N ? double(R[lane * (LD + 1)].re) : 0.0);
        if (lane == 0) {
          trace = tr;
          it.scratch[0] = tr;
          if (!(tr > 0.0) || !isfinite(tr)) {
            bad = 1;
            it.scratch[1] = 1.0;
          }
        }
      }
      __syncthreads();
      if (!bad) {                       // once a trace was bad, rho is left as it is
        const double inv = 1.0 / trace;
        for (int idx = threadIdx.x; idx < NP * NP; idx += RTPB) {
          const int i = idx / NP, j = idx - (idx / NP) * NP;
          const E p = R[i * LD + j], q = R[j * LD + i];
          const double re = 0.5 * (double(p.re) + double(q.re)) * inv;
          const double im = i == j ? 0.0 : 0.5 * (double(p.im) - double(q.im)) * inv;
          X[i * LD + j] = E{T(re), T(im)};
        }
        __syncthreads();
        E* t = R;
        R = X;
        X = t;
      }
    }
    // the record wave reads R's diagonal while the product waves run the next
    // step's first product, which only reads R; R is next written after the
    // barrier that follows it
    if (rec && step == next_record) {
      next_record += a.record_every;
      record(++rindex);
    }
  }
  __syncthreads();
  // back to the lab frame: rho_ij e^{-i w_c (k_i - k_j) t}
  const double t = double(a.steps) * a.dt;
  for (int idx = threadIdx.x; idx < N * N; idx += RTPB) {
    const int i = idx / N, j = idx - (idx / N) * N;
    E v = R[i * LD + j];
    const int dk = exc(i) - exc(j);
    if (a.rot && dk != 0 && t != 0.0) {
      double sn, cs;
      sincos(-it.omega_c * double(dk) * t, &sn, &cs);
      const double re = double(v.re), im = double(v.im);
      v = E{T(cs * re - sn * im), T(cs * im + sn * re)};
    }
    if (a.rho_c128)
      static_cast<c128*>(it.rho)[int64_t(i) * it.ldr + j] = c128{double(v.re), double(v.im)};
    else
      static_cast<c64*>(it.rho)[int64_t(i) * it.ldr + j] = c64{float(v.re), float(v.im)};
  }
}

template <typename T, int NB>
int launch(const ResidentItem* one, const ResidentItem* many_dev, int count, const ResidentRun& a,
           hipStream_t s) {
  hipLaunchKernelGGL((resident_kernel<T, NB>), dim3(unsigned(count)), dim3(RTPB), 0, s,
                     one ? *one : ResidentItem(), many_dev, a);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

}  // namespace

int launch_resident(bool f64, int maxN, const ResidentItem* one, const ResidentItem* many_dev,
                    int count, const ResidentRun& a, hipStream_t s) {
  if (maxN > (f64 ? RESIDENT_MAX_N_C128 : RESIDENT_MAX_N_C64) || (!one && !many_dev)) {
    set_error("LDS-resident stepping: N too large");
    return TC_ERR_UNSUPPORTED;
  }
  const int nb = (maxN + 15) / 16;
  if (f64) {
    if (nb == 1) return launch<double, 1>(one, many_dev, count, a, s);
    if (nb == 2) return launch<double, 2>(one, many_dev, count, a, s);
    return launch<double, 3>(one, many_dev, count, a, s);
  }
  if (nb == 1) return launch<float, 1>(one, many_dev, count, a, s);
  if (nb == 2) return launch<float, 2>(one, many_dev, count, a, s);
  if (nb == 3) return launch<float, 3>(one, many_dev, count, a, s);
  return launch<float, 4>(one, many_dev, count, a, s);
}

}  // namespace tcm
