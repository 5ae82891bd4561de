// Split-BF16 products of small matrices (a time step at N up to 640), one
// workgroup per 16 x 16 or 32 x 32 output tile.
//
// Such a product has too few 128 x 128 tiles for the chip; cutting their K into
// ranges leaves partial tiles to write, read and finish in a second launch.
// Here, as in the small FP64 / FP32 kernel, the tile is chosen so that about
// every CU has one, the workgroup's waves divide K (wave w takes the 32-deep
// slices w, w + NW, ...), and the partial tiles are added in wave order through
// LDS, so that results are deterministic.  The plane layout makes the operands'
// fragments contiguous (lane l of a 16 x 16 x 32 MFMA holds 8 consecutive K
// values of row l%16 of one plane, 16 bytes; a row's four planes of a slice are
// 256 bytes), so a wave reads them straight from L2 into registers and nothing
// is staged.  Bound by latency up to N = 320 (16 x 16 tiles), then by the
// operands' L2 reads (a 32 x 32 tile asks for 85 bytes a clock and CU at full
// MFMA rate).  Step time against 128 x 128 tiles with K ranges: N = 96 12 and 33
// us, 160 13 and 49, 256 16 and 51, 384 30 and 55, 512 35 and 63, 640 52 and 64;
// from 768 on (90 and 68) the large tiles' smaller operand traffic wins.  64 x 64
// tiles of 4 waves, one wave per SIMD, took 82 us at N = 640 and 180 at 1280 (97
// on the large tiles): half of the chip's L2 misses wait in each round.
#include "gemm_bf16_small.h"

#include <algorithm>

#include "mfma.h"
#include "profile.h"
#include "readout.h"

namespace tcm {
namespace {

// hi = RNE_bf16(x), or lo = RNE_bf16(x - hi), as bits (the hardware conversion).
__device__ __forceinline__ uint16_t bits(float x) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(x));
}
__device__ __forceinline__ uint16_t part(float x, bool lo) {
  const uint16_t h = bits(x);
  return lo ? bits(x - __uint_as_float(uint32_t(h) << 16)) : h;
}

constexpr int NW = 8, DEPTH = 2;           // waves; register sets of operand slices
static_assert(64 * NW == READOUT_NT, "the last workgroup of a launch may read the records");

template <int TM, int TN>
__global__ void __launch_bounds__(64 * NW)
split_small_kernel(const SplitSmall p, int tiles_n, int tiles, const SmallReadout ro) {
  constexpr int NT = 64 * NW, NB = TM * TN, H = 16 * TM, W = 16 * TN;
  __shared__ float2 lds[NW * NB * 256];
  if (int(blockIdx.x) >= tiles) {
    const ReadoutItem& it = ro.item;
    const int64_t r = ro.counter ? int64_t(*ro.counter) : ro.index;
    const int ns = (it.n < it.c ? it.n : it.c) + 1;
    readout_body<c64>(it.n, it.c, static_cast<const c64*>(it.rho), it.ld, it.map, it.off, it.k,
                          it.pop ? it.pop + r : nullptr,
                          it.pdist ? it.pdist + r * (it.c + 1) : nullptr,
                          it.pstate ? it.pstate + r * ns : nullptr,
                          reinterpret_cast<double*>(lds));
    if (ro.counter && threadIdx.x == 0) *ro.counter = int(r) + 1;   // after the body's barrier
    return;
  }
  const int lin = xcd_linear(blockIdx.x, tiles);
  int tm, tn;
  if (p.herm) {
    tri_columns(lin, tm, tn);
  } else {
    tm = lin / tiles_n;
    tn = lin - tm * tiles_n;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lc = lane >> 4;
  const int m0 = tm * H, n0 = tn * W;
  // byte offsets of this lane's fragment rows; the planes are padded with rows
  // up to a multiple of 128, so a tile never leaves them
  const char* pa = reinterpret_cast<const char*>(p.A) + int64_t(m0 + lr) * p.lda * 8 + lc * 16;
  const char* pb = reinterpret_cast<const char*>(p.B) + int64_t(n0 + lr) * p.ldb * 8 + lc * 16;
  const int64_t sa = 16 * p.lda * 8, sb = 16 * p.ldb * 8;    // 16 rows down
  const int slices = int(p.Kp / SPLIT_BK);
  const int mine = wave < slices ? (slices - wave + NW - 1) / NW : 0;
  f4 re[TM][TN], im[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      re[i][j] = f4{0, 0, 0, 0};
      im[i][j] = f4{0, 0, 0, 0};
    }
  u4 a[DEPTH][TM][4], b[DEPTH][TN][4];
  // past the last slice the load repeats it (in bounds, never used)
  auto load = [&](int d, int it) {
    const int64_t o = int64_t(wave + NW * min(it, mine - 1)) * 256;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        a[d][i][q] = *reinterpret_cast<const u4*>(pa + i * sa + o + q * 64);
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        b[d][j][q] = *reinterpret_cast<const u4*>(pb + j * sb + o + q * 64);
  };
  const u4 sgn = u4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
  auto mul = [&](int d) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const u4 nih = a[d][i][PL_IH] ^ sgn, nil = a[d][i][PL_IL] ^ sgn;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        f4 x = re[i][j], y = im[i][j];
        x = mma(a[d][i][PL_RH], b[d][j][PL_RH], x);
        y = mma(a[d][i][PL_RH], b[d][j][PL_IH], y);
        x = mma(a[d][i][PL_RH], b[d][j][PL_RL], x);
        y = mma(a[d][i][PL_RH], b[d][j][PL_IL], y);
        x = mma(a[d][i][PL_RL], b[d][j][PL_RH], x);
        y = mma(a[d][i][PL_RL], b[d][j][PL_IH], y);
        x = mma(nih, b[d][j][PL_IH], x);
        y = mma(a[d][i][PL_IH], b[d][j][PL_RH], y);
        x = mma(nih, b[d][j][PL_IL], x);
        y = mma(a[d][i][PL_IH], b[d][j][PL_RL], y);
        x = mma(nil, b[d][j][PL_IH], x);
        y = mma(a[d][i][PL_IL], b[d][j][PL_RH], y);
        re[i][j] = x;
        im[i][j] = y;
      }
    }
  };
  if (mine > 0) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) load(d, d);
    for (int it = 0; it < mine; it += DEPTH) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        if (it + d < mine) mul(d);
        load(d, it + d + DEPTH);
      }
    }
  }
  // partial tiles: [wave][block][r][lane], element row 4 (lane/16) + r of a block
  float2* part_tile = lds + wave * NB * 256;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        part_tile[((i * TN + j) * 4 + r) * 64 + lane] = make_float2(re[i][j][r], im[i][j][r]);
  __syncthreads();
  constexpr int PT = (NB * 256 + NT - 1) / NT;
  float2 out[PT];
#pragma unroll
  for (int z = 0; z < PT; ++z) {
    const int e = tid + z * NT;
    if (e >= NB * 256) break;
    const int row = e / W, col = e % W, rr = row & 15;
    const int slot = ((row >> 4) * TN + (col >> 4)) * 256 + (rr & 3) * 64 + (rr >> 2) * 16 + (col & 15);
    float2 s = lds[slot];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      const float2 t = lds[w * NB * 256 + slot];
      s.x += t.x;
      s.y += t.y;
    }
    const int gr = m0 + row, gc = n0 + col;
    const bool in = gr < p.M && gc < p.N;
    if (in && p.Cin) {
      const c64 y = p.Cin[int64_t(gr) * p.ldcin + gc];
      s.x += y.re;
      s.y += y.im;
    }
    if (!in) s = make_float2(0.f, 0.f);     // padding of the planes stays zero
    if (in && p.Cf) p.Cf[int64_t(gr) * p.ldcf + gc] = c64{s.x, s.y};
    out[z] = s;
  }
  // the finished tile in LDS, for the mirrored result and the planes
  constexpr int LD = W + 1;
  static_assert(H * LD <= NW * NB * 256, "the tile fits the partial tiles' LDS");
  __syncthreads();
#pragma unroll
  for (int z = 0; z < PT; ++z) {
    const int e = tid + z * NT;
    if (e < NB * 256) lds[(e / W) * LD + e % W] = out[z];
  }
  __syncthreads();
  const bool mirror = p.herm && tm != tn;
  if (mirror && p.Cf) {
    for (int e = tid; e < NB * 256; e += NT) {
      const int row = e / H, col = e % H;    // of the mirrored tile
      const int gr = n0 + row, gc = m0 + col;
      if (gr < p.N && gc < p.M) {
        const float2 v = lds[col * LD + row];
        p.Cf[int64_t(gr) * p.ldcf + gc] = c64{v.x, -v.y};
      }
    }
  }
  // 16-byte chunks of the hi/lo planes: 8 consecutive K of one plane row.
  // along: the plane rows are the tile's rows and K its columns, else the other
  // way round; flip: the imaginary planes negated (the mirrored element).
  auto planes = [&](bool along, bool flip) {
    const int rows = along ? H : W, kc = (along ? W : H) / 8;
    const int64_t r0 = along ? m0 : n0, k0 = along ? n0 : m0;
    for (int e = tid; e < rows * kc * 4; e += NT) {
      const int q = e & 3, c = (e >> 2) % kc, r = (e >> 2) / kc;
      uint32_t w[4];
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        uint32_t v[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const int k = 8 * c + 2 * h + g;
          const float2 x = along ? lds[r * LD + k] : lds[k * LD + r];
          const float y = q >= PL_IH ? (flip ? -x.y : x.y) : x.x;
          v[g] = part(y, (q & 1) != 0);
        }
        w[h] = v[0] | (v[1] << 16);
      }
      *reinterpret_cast<u4*>(p.P + plane_offset(p.ldp, r0 + r, k0 + 8 * c, q)) = u4{w[0], w[1], w[2], w[3]};
    }
  };
  planes(!p.p_trans, false);
  if (mirror) planes(p.p_trans, true);
}

template <int TM, int TN>
int launch(const SplitSmall& p, const SmallReadout* ro, hipStream_t s) {
  const int64_t a = (p.M + 16 * TM - 1) / (16 * TM), b = (p.N + 16 * TN - 1) / (16 * TN);
  const int tiles = int(p.herm ? a * (a + 1) / 2 : a * b);
  ProfileScope prof(TC_KERNEL_SPLIT_BF16, s);
  hipLaunchKernelGGL((split_small_kernel<TM, TN>), dim3(unsigned(tiles + (ro ? 1 : 0))),
                     dim3(64 * NW), 0, s, p, int(b), tiles, ro ? *ro : SmallReadout());
  TC_TRY_HIP(hipGetLastError());
  return TC_OK;
}

}  // namespace

bool split_small_step(int64_t N) {
  return N <= 640 && split_variant() == 0;
}

int split_small(const SplitSmall& p, const SmallReadout* ro, hipStream_t s) {
  const int64_t rows = round_up(p.M, SPLIT_BM), cols = round_up(p.N, SPLIT_BN);
  if (p.M <= 0 || p.N <= 0 || p.Kp <= 0 || p.Kp % SPLIT_BK != 0 || p.lda < p.Kp || p.ldb < p.Kp ||
      (p.herm && p.M != p.N) || p.P == nullptr || p.ldp < (p.p_trans ? rows : cols) ||
      (p.herm && p.ldp < rows)) {
    set_error("small split product: bad operand shape");
    return TC_ERR_INVALID_ARGUMENT;
  }
  // 16 x 16 tiles up to N = 320 (22 us a step against 27), above 32 x 32 (N = 384:
  // 30 against 33)
  return p.N <= 320 ? launch<1, 1>(p, ro, s) : launch<2, 2>(p, ro, s);
}

}  // namespace tcm
