// Complex FP64 / FP32 products of small matrices (the time step at N up to
// about a thousand), one workgroup per 16 x 16 or 32 x 32 output tile.
//
// Such a product has too few 128 x 128 or 64 x 64 tiles to occupy the chip, and
// its time is a chain of latencies: launch, first loads, a long serial K loop
// with a barrier per K tile, partial sums through memory.  Here
//   * the tile is small enough that about every CU has one;
//   * the 8 waves of the workgroup divide K between them (wave w takes the
//     8-deep slices w, w + 8, ...), each for the whole tile, so the serial K
//     loop is an eighth as long and needs no barrier;
//   * a wave reads its MFMA fragments straight from L2 into registers (no LDS
//     staging: nothing is shared between waves that hold different K), a few
//     slices ahead: lane l takes A[l%16][2(l/16), +1] and B[2(l/16), +1][l%16]
//     of a slice, i.e. both operands list K in the order 0 2 4 6 | 1 3 5 7, so
//     that a lane's two A elements are neighbours in memory;
//   * the waves' partial tiles are added in wave order through LDS (results are
//     deterministic), then the epilogue writes rows, and the conjugate
//     transpose of an off-diagonal tile of a Hermitian result.
// The MFMA work of a 16 x 16 tile per slice (8 FP64 instructions, 512 cycles)
// covers its 4 KB of L2 reads; at 32 x 32 the ratio doubles.  An element's value
// depends only on K and its operands, not on the tile shape, so a product gives
// the same bits alone and in a group.
#include "gemm_small.h"

#include <algorithm>
#include <cmath>

#include "mfma.h"
#include "profile.h"
#include "readout.h"

namespace tcm {
namespace {

struct SmallParams {
  int M, N, K;
  const void* A; int64_t lda;
  const void* B; int64_t ldb;
  void* C; int64_t ldc;
  const void* Cin; int64_t ldcin;
  double alpha_re, alpha_im, beta_re, beta_im, gamma;
  int conj_a, conj_b, herm;
  int tiles_n, tiles;
};

constexpr int NW = 8, NT = 64 * NW;
static_assert(NT == READOUT_NT, "the last workgroup of a launch may read the records");

// Operand elements, through address-space-1 pointers: the grouped kernel takes
// its operand pointers from a descriptor array, where the compiler cannot tell
// them from LDS and would issue flat loads.
template <typename T> struct pair_t {
  typedef T type __attribute__((ext_vector_type(2), aligned(sizeof(T))));
};
template <typename T>
__device__ __forceinline__ typename pair_t<T>::type gload(const cplx<T>* p) {
  typedef __attribute__((address_space(1))) const typename pair_t<T>::type G;
  return *(G*)p;
}
template <typename T>
__device__ __forceinline__ void gstore(cplx<T>* p, cplx<T> x) {
  typedef __attribute__((address_space(1))) typename pair_t<T>::type G;
  *(G*)p = typename pair_t<T>::type{x.re, x.im};
}

// Tile lin of the product p (row by row of tiles, or the upper tile triangle
// column by column).
template <typename T, int TM, int TN, int DEPTH, bool KCHK>
__device__ __forceinline__ void small_tile_body(const SmallParams& p, int lin, cplx<T>* lds) {
  typedef cplx<T> E;
  typedef typename acc_t<T>::type V;
  typedef typename pair_t<T>::type v2;
  constexpr int NB = TM * TN;
  int tm, tn;
  if (p.herm) {
    tri_columns(lin, tm, tn);
  } else {
    tm = lin / p.tiles_n;
    tn = lin - tm * p.tiles_n;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, q2 = 2 * (lane >> 4);
  const int m0 = tm * 16 * TM, n0 = tn * 16 * TN;
  const int K = p.K;
  const E* __restrict__ A = static_cast<const E*>(p.A);
  const E* __restrict__ B = static_cast<const E*>(p.B);
  // rows and columns past the matrix read its last one; their outputs are not stored
  const E* pa[TM];
  const E* pb[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) pa[i] = A + int64_t(min(m0 + 16 * i + lr, p.M - 1)) * p.lda;
#pragma unroll
  for (int j = 0; j < TN; ++j) pb[j] = B + min(n0 + 16 * j + lr, p.N - 1);
  const T sa = p.conj_a ? T(-1) : T(1), sb = p.conj_b ? T(-1) : T(1);

  V re[TM][TN], im[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      re[i][j] = V{0, 0, 0, 0};
      im[i][j] = V{0, 0, 0, 0};
    }
  const int slices = (K + 7) / 8;
  const int mine = wave < slices ? (slices - wave + NW - 1) / NW : 0;
  v2 a[DEPTH][TM][2], b[DEPTH][TN][2];
  // the it-th slice of this wave into register set d; past the last one it
  // repeats the last one (in bounds, never used)
  auto load = [&](int d, int it) {
    const int k = 8 * (wave + NW * min(it, mine - 1)) + q2;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int kk = KCHK ? min(k + h, K - 1) : k + h;
#pragma unroll
      for (int i = 0; i < TM; ++i) a[d][i][h] = gload(pa[i] + kk);
#pragma unroll
      for (int j = 0; j < TN; ++j) b[d][j][h] = gload(pb[j] + int64_t(kk) * p.ldb);
    }
  };
  auto mul = [&](int d, int it) {
    const int k = 8 * (wave + NW * it) + q2;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v2 x[TM], y[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        x[i] = a[d][i][h];
        x[i].y *= sa;
        if (KCHK && k + h >= K) x[i] = v2{0, 0};
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        y[j] = b[d][j][h];
        y[j].y *= sb;
        if (KCHK && k + h >= K) y[j] = v2{0, 0};
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          re[i][j] = mma(x[i].x, y[j].x, re[i][j]);
          im[i][j] = mma(x[i].x, y[j].y, im[i][j]);
          re[i][j] = mma_nega(x[i].y, y[j].y, re[i][j]);
          im[i][j] = mma(x[i].y, y[j].x, im[i][j]);
        }
    }
  };
  if (mine > 0) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) load(d, d);
    for (int it = 0; it < mine; it += DEPTH) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        if (it + d < mine) mul(d, it + d);
        load(d, it + d + DEPTH);
      }
    }
  }
  // partial tiles: [wave][block][r][lane]
  E* mineP = lds + wave * NB * 256;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        mineP[((i * TN + j) * 4 + r) * 64 + lane] = E{re[i][j][r], im[i][j][r]};
  __syncthreads();
  constexpr int W = 16 * TN;               // tile columns
  constexpr int PT = (NB * 256 + NT - 1) / NT;
  const T ar = T(p.alpha_re), ai = T(p.alpha_im), br = T(p.beta_re), bi = T(p.beta_im);
  const bool use_beta = p.Cin != nullptr && (p.beta_re != 0.0 || p.beta_im != 0.0);
  const bool mirror = p.herm && tm != tn;
  E out[PT];
#pragma unroll
  for (int z = 0; z < PT; ++z) {
    const int e = tid + z * NT;
    if (e >= NB * 256) break;
    const int row = e / W, col = e % W, rr = row & 15;
    const int slot = ((row >> 4) * TN + (col >> 4)) * 256 +
                     (sizeof(T) == 8 ? rr * 16 + (col & 15)
                                     : (rr & 3) * 64 + (rr >> 2) * 16 + (col & 15));
    E s = lds[slot];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      const E t = lds[w * NB * 256 + slot];
      s.re += t.re;
      s.im += t.im;
    }
    const int gr = m0 + row, gc = n0 + col;
    E o{ar * s.re - ai * s.im, ar * s.im + ai * s.re};
    if (gr < p.M && gc < p.N) {
      if (use_beta) {
        const v2 y = gload(static_cast<const E*>(p.Cin) + int64_t(gr) * p.ldcin + gc);
        o.re += br * y.x - bi * y.y;
        o.im += br * y.y + bi * y.x;
      }
      if (gr == gc) o.re += T(p.gamma);
      gstore(static_cast<E*>(p.C) + int64_t(gr) * p.ldc + gc, o);
    }
    out[z] = o;
  }
  if (!mirror) return;
  // conj of the tile, transposed through LDS so that rows are written
  constexpr int H = 16 * TM, LD = W + 1;
  static_assert(H * LD <= NW * NB * 256, "the transposed tile fits the partial tiles' LDS");
  __syncthreads();
#pragma unroll
  for (int z = 0; z < PT; ++z) {
    const int e = tid + z * NT;
    if (e < NB * 256) lds[(e / W) * LD + e % W] = out[z];
  }
  __syncthreads();
#pragma unroll
  for (int z = 0; z < PT; ++z) {
    const int e = tid + z * NT;
    if (e >= NB * 256) break;
    const int row = e / H, col = e % H;    // of the mirrored tile
    const int gr = n0 + row, gc = m0 + col;
    if (gr < p.N && gc < p.M) {
      const E v = lds[col * LD + row];
      gstore(static_cast<E*>(p.C) + int64_t(gr) * p.ldc + gc, E{v.re, -v.im});
    }
  }
}

// One product; the launch's last workgroup reads the records of ro when the
// launch has one workgroup more than tiles.
template <typename T, int TM, int TN, int DEPTH, bool KCHK>
__global__ void __launch_bounds__(NT) small_kernel(const SmallParams p, const SmallReadout ro) {
  typedef cplx<T> E;
  __shared__ E lds[NW * TM * TN * 256];
  if (int(blockIdx.x) >= p.tiles) {
    const ReadoutItem& it = ro.item;
    const int64_t r = ro.counter ? int64_t(*ro.counter) : ro.index;
    const int ns = (it.n < it.c ? it.n : it.c) + 1;
    readout_body(it.n, it.c, static_cast<const E*>(it.rho), it.ld, it.map, it.off, it.k,
                 it.pop ? it.pop + r : nullptr, it.pdist ? it.pdist + r * (it.c + 1) : nullptr,
                 it.pstate ? it.pstate + r * ns : nullptr, reinterpret_cast<double*>(lds));
    if (ro.counter && threadIdx.x == 0) *ro.counter = int(r) + 1;   // after the body's barrier
    return;
  }
  small_tile_body<T, TM, TN, DEPTH, KCHK>(p, xcd_linear(blockIdx.x, p.tiles), lds);
}

struct SmallItem {
  SmallParams p;
  int tile_begin;
};

// The products of many instances in one launch, one workgroup per tile of the
// concatenated tile list.
template <typename T, int TM, int TN, int DEPTH>
__global__ void __launch_bounds__(NT) small_grouped_kernel(const SmallItem* __restrict__ items,
                                                           int count) {
  __shared__ cplx<T> lds[NW * TM * TN * 256];
  const int t = blockIdx.x;
  int lo = 0, hi = count - 1;            // last item with tile_begin <= t
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (items[mid].tile_begin <= t) lo = mid; else hi = mid - 1;
  }
  const SmallParams p = items[lo].p;
  small_tile_body<T, TM, TN, DEPTH, true>(p, t - items[lo].tile_begin, lds);
}

int64_t tile_count(int64_t M, int64_t N, bool herm, int edge) {
  const int64_t a = (M + edge - 1) / edge, b = (N + edge - 1) / edge;
  return herm ? a * (a + 1) / 2 : a * b;
}

SmallParams make_params(const GemmDesc& d, int edge) {
  SmallParams p;
  p.M = int(d.M); p.N = int(d.N); p.K = int(d.K);
  p.A = d.A; p.lda = d.lda; p.B = d.B; p.ldb = d.ldb;
  p.C = d.C; p.ldc = d.ldc; p.Cin = d.Cin; p.ldcin = d.ldcin;
  p.alpha_re = d.alpha_re; p.alpha_im = d.alpha_im;
  p.beta_re = d.beta_re; p.beta_im = d.beta_im; p.gamma = d.gamma;
  p.conj_a = d.conj_a; p.conj_b = d.conj_b;
  p.herm = d.herm && d.M == d.N;
  p.tiles_n = int((d.N + edge - 1) / edge);
  p.tiles = int(tile_count(d.M, d.N, p.herm, edge));
  return p;
}

// One product on 16 x 16 or 32 x 32 tiles: a round (one tile to a CU) of the smaller ones costs 7/16 of
// one of the larger ones, not a quarter (two operand reads per MFMA more, and
// the launch's fixed time): FP64 step at N = 320 26 and 31 us, at N = 384 39 and
// 36 us, at N = 512 50 and 42 us.
int choose_edge(int64_t t16, int64_t t32) {
  const int64_t cus = device_cus();
  return 7 * ((t16 + cus - 1) / cus) < 16 * ((t32 + cus - 1) / cus) ? 16 : 32;
}

}  // namespace

// A group's tiles run in rounds of one workgroup per CU (FP32 32 x 32 tiles two to a
// CU), and a round of small tiles costs what its 8 waves' load, reduction and
// dispatch take, whatever K: fitted to groups of 4 to 400 instances of N = 8 .. 192
// (us a step of two products, 16 x 16 / 32 x 32: FP64 4 x N = 112 17 / 20, 40 x 44 19 / 18,
// 100 x 64 68 / 36, 40 x 160 133 / 81; FP32 16 x 48 14.2 / 14.5, 40 x 64 33 / 17, 100 x 128
// 201 / 65).
double small_group_us(double t16, double t32, double K, bool f64, int* edge) {
  const double cus = device_cus(), r16 = std::ceil(t16 / cus), r32 = t32 / cus;
  const double us16 = r16 * (std::min(4.8, 1.5 + 0.05 * K) + 0.004 * std::max(0.0, K - 160.0));
  double us32;
  if (f64)
    us32 = std::ceil(r32) * (K < 60.0 ? 2.5 + 0.078 * K : std::max(5.7 + 0.023 * K, 0.04 * K));
  else
    us32 = r32 <= 1.0 ? 2.5 + 0.03 * K
                      : std::min(3.0, 0.04 * K) +
                            (K < 60.0 ? 1.6 + 0.04 * K : std::max(3.75, 0.031 * K)) * r32;
  const bool fine = us16 < us32 || t16 <= t32;
  if (edge) *edge = fine ? 16 : 32;
  return fine ? us16 : us32;
}

namespace {

template <typename T, int TM, int TN, int DEPTH>
int launch_small(const SmallParams& p, const SmallReadout* ro, hipStream_t s) {
  const dim3 grid(unsigned(p.tiles + (ro ? 1 : 0))), block(NT);
  const SmallReadout r = ro ? *ro : SmallReadout();
  if (p.K % 8 == 0)
    hipLaunchKernelGGL((small_kernel<T, TM, TN, DEPTH, false>), grid, block, 0, s, p, r);
  else
    hipLaunchKernelGGL((small_kernel<T, TM, TN, DEPTH, true>), grid, block, 0, s, p, r);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

template <typename T, int TM, int TN, int DEPTH>
int launch_grouped(const SmallGroup& g, hipStream_t s) {
  hipLaunchKernelGGL((small_grouped_kernel<T, TM, TN, DEPTH>), dim3(unsigned(g.tiles)), dim3(NT), 0,
                     s, static_cast<const SmallItem*>(g.items_dev), g.count);
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

}  // namespace

// Step times (both products, FP64 / FP32): N = 64 12.9 / 10.2 us against 27.6 /
// 19.4 on 64 x 64 and 128 x 128 LDS tiles, 160 13.3 / 10.6 against 64 / 45.  Above
// the limits larger tiles' smaller operand traffic wins: FP64 direct tiles with a
// buffer to spread their last round, 512 43 us against 64, 640 70 against 91, 768
// 131 against 125, 1024 237 against 227; FP32 128 x 128 tiles, 1024 128 against 146,
// 1536 372 against 403.
bool small_product(const GemmDesc& d, bool f64) {
  const int64_t most = f64 ? (d.spread ? 704 : 1024) : 1536;
  return d.complex && !d.a_kmaj && d.b_kmaj && !d.c_trans && !d.cin_trans && d.M <= most &&
         d.N <= most && d.K >= 1 && d.K <= (int64_t(1) << 20);
}

template <typename T>
int small_gemm(const GemmDesc& d, const SmallReadout* ro, hipStream_t s) {
  const bool herm = d.herm && d.M == d.N;
  const int edge = choose_edge(tile_count(d.M, d.N, herm, 16), tile_count(d.M, d.N, herm, 32));
  const SmallParams p = make_params(d, edge);
  ProfileScope prof(sizeof(T) == 8 ? TC_KERNEL_GEMM_F64 : TC_KERNEL_GEMM_F32, s);
  return edge == 32 ? launch_small<T, 2, 2, 2>(p, ro, s) : launch_small<T, 1, 1, 4>(p, ro, s);
}

template int small_gemm<double>(const GemmDesc&, const SmallReadout*, hipStream_t);
template int small_gemm<float>(const GemmDesc&, const SmallReadout*, hipStream_t);

size_t small_grouped_bytes(int count) { return size_t(count) * sizeof(SmallItem); }

int small_grouped_build(const std::vector<GemmDesc>& ds, bool f64, void* items_dev, SmallGroup* g,
                        hipStream_t s) {
  int64_t t16 = 0, t32 = 0, t = 0;
  double work = 0.0;
  for (const GemmDesc& d : ds) {
    if (!small_product(d, f64)) {
      set_error("grouped small products: a product is not a small one");
      return TC_ERR_UNSUPPORTED;
    }
    t16 += tile_count(d.M, d.N, d.herm, 16);
    t32 += tile_count(d.M, d.N, d.herm, 32);
    work += double(tile_count(d.M, d.N, d.herm, 32)) * double(d.K);
  }
  small_group_us(double(t16), double(t32), ds.empty() ? 0.0 : work / double(t32), f64, &g->edge);
  std::vector<SmallItem> items;
  for (const GemmDesc& d : ds) {
    SmallItem it;
    it.p = make_params(d, g->edge);
    it.tile_begin = int(t);
    t += it.p.tiles;
    items.push_back(it);
  }
  if (t > (int64_t(1) << 30)) { set_error("too many tiles in one group"); return TC_ERR_UNSUPPORTED; }
  g->f64 = f64;
  g->count = int(items.size());
  g->tiles = int(t);
  g->items_dev = items_dev;
  if (!items.empty()) {
    TC_TRY_HIP(hipMemcpyAsync(items_dev, items.data(), items.size() * sizeof(SmallItem),
                              hipMemcpyHostToDevice, s));
    TC_TRY_HIP(hipStreamSynchronize(s));   // items is host memory of this call
  }
  return TC_OK;
}

int small_grouped_run(const SmallGroup& g, hipStream_t s) {
  if (g.tiles == 0) return TC_OK;
  ProfileScope prof(g.f64 ? TC_KERNEL_GEMM_F64 : TC_KERNEL_GEMM_F32, s);
  if (g.f64)
    return g.edge == 32 ? launch_grouped<double, 2, 2, 2>(g, s) : launch_grouped<double, 1, 1, 4>(g, s);
  return g.edge == 32 ? launch_grouped<float, 2, 2, 2>(g, s) : launch_grouped<float, 1, 1, 4>(g, s);
}

}  // namespace tcm
