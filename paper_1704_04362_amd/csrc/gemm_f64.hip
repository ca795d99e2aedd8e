// Per-slice complex products in float64 on the matrix cores
// (v_mfma_f64_16x16x4f64: A lane l = A[l % 16][l / 16], B lane l =
// B[l / 16][l % 16], D lane l register v = D[4 v + l / 16][l % 16]).
//
// Four wavefronts own a 32 x 32 or 64 x 64 tile of one slice (16 x 16 or
// 32 x 32 each) as four real products per complex one; 16-deep steps of both
// operands are loaded one step ahead into registers (unconditionally, from
// clamped addresses) and staged in one of two LDS buffers, k-major with a row
// stride of 16 mod 32 doubles, so that the 4 x 16 fragment reads spread evenly
// over the banks; one barrier per step.
//
// Bound by the matrix cores (64 cycles per instruction of 2,048 operations;
// 58 TFLOP/s measured from registers). Measured against the vector kernel this
// replaces (a float64 multiply-add per lane in 8 cycles, tiles padded to 64 x 64):
// 31 slices of 257 x 380 x 201 411 -> 180 us, 33 of 512 x 512 x 512 1504 -> 708,
// 65 of 300 x 1024 x 32 405 -> 186, 25 of 28 x 1732 x 39 528 -> 171.
#include <algorithm>

#include "common.hpp"

namespace tp {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int NT = 256, BK = 16;

struct DArgs {
  int64_t M, N, Kd;
  const double *are, *aim, *bre, *bim;
  double *cre, *cim;
  int64_t lda, ldb, ldc, sa, sb, sc;
  int64_t K;
  int real_last;
  const int64_t* kdim_dev;
  int tm, tn;  // output tiles per slice
  int runs;    // launch order, see cgemm_f64_kernel
};

// One operand's 16-deep step in registers: TM (or TN) x 16 complex values,
// E per thread. `along_k`: the stored matrix is contiguous in the contraction
// (rows of A, or B^H stored), else in the output index.
template <int T>
struct Step {
  static constexpr int E = T * BK / NT;
  double r[E], i[E];
};

template <int T, bool ALONG>
__device__ __forceinline__ void place(int e, int& o, int& k) {
  const int f = threadIdx.x + e * NT;
  if (ALONG) {
    k = f % BK;
    o = f / BK;
  } else {
    o = f % T;
    k = f / T;
  }
}

template <int T, bool ALONG, bool REAL>
__device__ __forceinline__ void load_step(Step<T>& s, const double* re, const double* im, int64_t ld, int64_t o0,
                                          int64_t k0, int64_t no, int64_t nk) {
#pragma unroll
  for (int e = 0; e < Step<T>::E; ++e) {
    int o, k;
    place<T, ALONG>(e, o, k);
    const int64_t go = o0 + o < no ? o0 + o : no - 1, gk = k0 + k < nk ? k0 + k : nk - 1;
    const int64_t off = ALONG ? go * ld + gk : gk * ld + go;
    s.r[e] = re[off];
    s.i[e] = REAL ? 0.0 : im[off];
  }
}

// zeros past the ends (contraction and output), conjugated if `conj`
template <int T, int S, bool ALONG, bool CONJ, bool REAL>
__device__ __forceinline__ void store_step(const Step<T>& s, double (*br)[S], double (*bi)[S], int64_t o0, int64_t k0,
                                           int64_t no, int64_t nk) {
#pragma unroll
  for (int e = 0; e < Step<T>::E; ++e) {
    int o, k;
    place<T, ALONG>(e, o, k);
    const bool in = o0 + o < no && k0 + k < nk;
    br[k][o] = in ? s.r[e] : 0.0;
    if (!REAL) bi[k][o] = in ? (CONJ ? -s.i[e] : s.i[e]) : 0.0;
  }
}

// W: 16 x 16 blocks per wavefront and side (tiles of 32 W); HA, HB: the operand
// is a conjugate transpose; REAL: the slice is real
template <int W>
struct Stage {
  static constexpr int T = 32 * W, S = T + 16;
  double ar[2][BK][S], ai[2][BK][S], br[2][BK][S], bi[2][BK][S];
};

template <int W, bool HA, bool HB, bool REAL>
__device__ __forceinline__ void product(const DArgs& g, Stage<W>& st, int64_t k, int64_t m0, int64_t n0) {
  constexpr int T = Stage<W>::T, S = Stage<W>::S;
  const int tid = threadIdx.x, l = tid & 63, w = tid >> 6, gr = l >> 4, j = l & 15;
  int64_t Kd = g.Kd;
  if (g.kdim_dev) {
    const int64_t lim = *g.kdim_dev;
    Kd = lim < Kd ? (lim < 0 ? 0 : lim) : Kd;
  }
  const double *are = g.are + k * g.sa, *aim = g.aim + k * g.sa, *bre = g.bre + k * g.sb, *bim = g.bim + k * g.sb;
  const int mw = 16 * W * (w >> 1), nw = 16 * W * (w & 1);
  d4 cr[W][W], ci[W][W];
#pragma unroll
  for (int a = 0; a < W; ++a)
#pragma unroll
    for (int b = 0; b < W; ++b) cr[a][b] = ci[a][b] = d4{0.0, 0.0, 0.0, 0.0};
  Step<T> sa, sb;
  auto load = [&](int64_t k0) {
    load_step<T, !HA, REAL>(sa, are, aim, g.lda, m0, k0, g.M, Kd);
    load_step<T, HB, REAL>(sb, bre, bim, g.ldb, n0, k0, g.N, Kd);
  };
  if (Kd > 0) load(0);
  int buf = 0;
  for (int64_t k0 = 0; k0 < Kd; k0 += BK, buf ^= 1) {
    store_step<T, S, !HA, HA, REAL>(sa, st.ar[buf], st.ai[buf], m0, k0, g.M, Kd);
    store_step<T, S, HB, HB, REAL>(sb, st.br[buf], st.bi[buf], n0, k0, g.N, Kd);
    // (this buffer's readers of two steps ago have passed the barrier of the
    // last step)
    __syncthreads();
    load(k0 + BK < Kd ? k0 + BK : k0);
#pragma unroll
    for (int kk = 0; kk < BK / 4; ++kk) {
      double xr[W], xi[W], yr[W], yi[W];
#pragma unroll
      for (int a = 0; a < W; ++a) {
        xr[a] = st.ar[buf][4 * kk + gr][mw + 16 * a + j];
        yr[a] = st.br[buf][4 * kk + gr][nw + 16 * a + j];
        if (!REAL) {
          xi[a] = st.ai[buf][4 * kk + gr][mw + 16 * a + j];
          yi[a] = st.bi[buf][4 * kk + gr][nw + 16 * a + j];
        }
      }
#pragma unroll
      for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < W; ++b) {
          cr[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[a], yr[b], cr[a][b], 0, 0, 0);
          if (!REAL) ci[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[a], yi[b], ci[a][b], 0, 0, 0);
        }
      if (REAL) continue;
#pragma unroll
      for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < W; ++b) {
          cr[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(-xi[a], yi[b], cr[a][b], 0, 0, 0);
          ci[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xi[a], yr[b], ci[a][b], 0, 0, 0);
        }
    }
  }
  double *cre = g.cre + k * g.sc, *cim = g.cim + k * g.sc;
#pragma unroll
  for (int a = 0; a < W; ++a)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t m = m0 + mw + 16 * a + 4 * v + gr;
      if (m >= g.M) continue;
#pragma unroll
      for (int b = 0; b < W; ++b) {
        const int64_t n = n0 + nw + 16 * b + j;
        if (n >= g.N) continue;
        cre[m * g.ldc + n] = cr[a][b][v];
        cim[m * g.ldc + n] = REAL ? 0.0 : ci[a][b][v];
      }
    }
}

// Workgroup L runs on XCD L mod 8. With `runs`, every XCD takes a contiguous run
// of tiles, so that a slice's operands are read through one L2 (32 x 32 tiles
// read twice the bytes per product: 218 -> 195 us at 31 slices of 257 x 380 x
// 201); with few slices, or 64 x 64 tiles, the round robin spreads the cheap
// real slices better (5 slices of 1000 x 100 x 1000: 84 against 104 us).
template <int W, bool HA, bool HB>
__global__ __launch_bounds__(NT, 2) void cgemm_f64_kernel(DArgs g) {
  __shared__ Stage<W> st;
  const int64_t per = (int64_t)g.tm * g.tn, total = per * g.K, q = (total + 7) / 8;
  // (rows of the grid are a multiple of 8 long: B mod 8 = blockIdx.x mod 8)
  const int64_t B = (int64_t)blockIdx.y * gridDim.x + blockIdx.x, L = g.runs ? (B % 8) * q + B / 8 : B;
  if (B >= 8 * q || L >= total) return;
  const int64_t k = L / per, t = L - k * per;
  const int64_t m0 = (t / g.tn) * Stage<W>::T, n0 = (t % g.tn) * Stage<W>::T;
  if (k == 0 || (g.real_last && k == g.K - 1))
    product<W, HA, HB, true>(g, st, k, m0, n0);
  else
    product<W, HA, HB, false>(g, st, k, m0, n0);
}

template <int W>
void (*pick(bool ha, bool hb))(DArgs) {
  if (ha) return hb ? cgemm_f64_kernel<W, true, true> : cgemm_f64_kernel<W, true, false>;
  return hb ? cgemm_f64_kernel<W, false, true> : cgemm_f64_kernel<W, false, false>;
}

}  // namespace

// 64 x 64 tiles read half the operand bytes per product, 32 x 32 ones pad less
// and fill more CUs: the smaller of the rounds over 256 CUs times the tile's
// work, with a tenth more for the 32 x 32 tiles' operand reads.
int cgemm_f64mfma(const CGemm& p, hipStream_t st) {
  const int64_t t64 = ((p.M + 63) / 64) * ((p.N + 63) / 64) * p.K, t32 = ((p.M + 31) / 32) * ((p.N + 31) / 32) * p.K;
  const bool wide = 40 * ((t64 + 255) / 256) <= 11 * ((t32 + 255) / 256);
  const int64_t T = wide ? 64 : 32, blocks = wide ? t64 : t32;
  // a launch's x extent holds 2^32 work-items: at most 2^23 workgroups a row of the grid
  const int64_t gx = std::min<int64_t>((blocks + 7) / 8 * 8, 1 << 23), gy = (blocks + gx - 1) / gx;
  if (gy > 65535) return fail(TP_EUNSUPPORTED, "product too large for one launch");
  DArgs g{p.M, p.N, p.Kd, (const double*)p.are, (const double*)p.aim, (const double*)p.bre, (const double*)p.bim,
          (double*)p.cre, (double*)p.cim, p.lda, p.ldb, p.ldc, p.sa, p.sb, p.sc, p.K,
          p.real_last ? 1 : 0, p.kdim_dev, (int)((p.M + T - 1) / T), (int)((p.N + T - 1) / T),
          !wide && p.K >= 24 ? 1 : 0};
  auto kernel = wide ? pick<2>(p.op_a != 0, p.op_b != 0) : pick<1>(p.op_a != 0, p.op_b != 0);
  hipLaunchKernelGGL(kernel, dim3((unsigned)gx, (unsigned)gy), dim3(NT), 0, st, g);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

}  // namespace tp
