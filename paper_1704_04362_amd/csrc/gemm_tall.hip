// Per-slice complex products with a narrow result: C_k = op(A_k) B_k with
// at most 64 columns and a long contraction, op = identity or conjugate
// transpose. These are the range-finder products of the randomized t-SVD
// and of the leverage estimates in t-CUR (Algorithms 4 and 5): Y = X Omega,
// Z = X^H Q and the projections, with X a full Fourier slice and Omega / Q
// a few dozen columns wide. Float32 products run on the float32 matrix cores
// (v_mfma_f32_16x16x4f32); split-precision products keep
// hi*hi + hi*lo + lo*hi of bf16 parts (v_mfma_f32_16x16x32_bf16), float32
// accumulation in both.
//
// Tiling: a 256-thread workgroup owns 64 rows x NB (32 or 64) columns of
// one Fourier slice and walks the contraction in 32-deep steps; wavefront w
// owns rows 16 w .. 16 w + 15 and all NB columns. In float32 a step's A and B tiles are
// staged in LDS (two buffers) and the next step's values are loaded into
// registers while the current step is on the matrix cores.
#include "common.hpp"

namespace tp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int TM = 64, KB = 32, TT = 256;

struct TArgs {
  int64_t M, N, Kd;
  const float *are, *aim, *bre, *bim;
  float *cre, *cim;
  int64_t lda, ldb, ldc, sa, sb, sc;
  int64_t K;
  int real_last;
  const int64_t* kdim_dev;
  // split contraction: part p of ksplit takes an equal share of the live
  // contraction, in whole steps, and writes its planes to pre / pim [p][k][M][N]
  int ksplit;
  float *pre, *pim;
};

__device__ __forceinline__ bf16x8 bneg(bf16x8 x) {
  u32x4 u = __builtin_bit_cast(u32x4, x);
  u ^= 0x80008000u;
  return __builtin_bit_cast(bf16x8, u);
}

// Loader of one 32-deep step into registers. A values: entry u of the
// thread is (m, kk) with, for op = N, m = e / KB, kk = e % KB (rows of A
// read along k) and, for op = C, kk = e / TM, m = e % TM (rows of A^stored
// read along m), e = tid + TT u. B values: (kk, n) = (e / NB, e % NB).
template <int OPA, int NB>
struct StepLoad {
  static constexpr int RA = TM * KB / TT, RB = KB * NB / TT;
  float ar[RA], ai[RA], br[RB], bi[RB];

  __device__ __forceinline__ static void a_index(int e, int& m, int& kk) {
    if (OPA == 0) {
      m = e / KB;
      kk = e % KB;
    } else {
      kk = e / TM;
      m = e % TM;
    }
  }

  __device__ __forceinline__ void load(const TArgs& g, const float* are, const float* aim, const float* bre,
                                       const float* bim, int64_t m0, int64_t k0, int64_t kd, bool real, int tid) {
#pragma unroll
    for (int u = 0; u < RA; ++u) {
      int m, kk;
      a_index(tid + TT * u, m, kk);
      const int64_t gm = m0 + m, gk = k0 + kk;
      const bool in = gm < g.M && gk < kd;
      const int64_t off = OPA == 0 ? gm * g.lda + gk : gk * g.lda + gm;
      ar[u] = in ? are[off] : 0.f;
      const float v = (in && !real) ? aim[off] : 0.f;
      ai[u] = OPA == 0 ? v : -v;  // conjugate for op = C
    }
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const int e = tid + TT * u, kk = e / NB, n = e % NB;
      const int64_t gk = k0 + kk;
      const bool in = n < g.N && gk < kd;
      br[u] = in ? bre[gk * g.ldb + n] : 0.f;
      bi[u] = (in && !real) ? bim[gk * g.ldb + n] : 0.f;
    }
  }
};

// The contraction range of this workgroup's part: its first k and length
__device__ __forceinline__ int64_t tall_kd(const TArgs& g, int64_t& kbeg) {
  int64_t kd = g.Kd;
  if (g.kdim_dev) {
    const int64_t lim = *g.kdim_dev;
    kd = lim < kd ? (lim < 0 ? 0 : lim) : kd;
  }
  kbeg = 0;
  if (g.ksplit > 1) {
    const int64_t chunk = ((kd + g.ksplit - 1) / g.ksplit + KB - 1) / KB * KB;
    kbeg = (int64_t)blockIdx.x * chunk;
    kd = kbeg < kd ? (kd - kbeg < chunk ? kd - kbeg : chunk) : 0;
    if (kd == 0) kbeg = 0;
  }
  return kd;
}

// lane (gq, c) holds C[m0 + 16 w + 4 gq + v][16 nt + c], v = 0..3
template <int NB>
__device__ __forceinline__ void tall_store(const TArgs& g, int64_t k, int64_t m0, int wave, int gq, int c,
                                           const f32x4 (&cr)[NB / 16], const f32x4 (&ci)[NB / 16], bool real) {
  const bool parted = g.ksplit > 1;
  const int64_t plane = ((int64_t)blockIdx.x * g.K + k) * g.M * g.N, ldc = parted ? g.N : g.ldc;
  float* cre = parted ? g.pre + plane : g.cre + k * g.sc;
  float* cim = parted ? g.pim + plane : g.cim + k * g.sc;
#pragma unroll
  for (int nt = 0; nt < NB / 16; ++nt) {
    const int64_t n = 16 * nt + c;
    if (n >= g.N) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t m = m0 + 16 * wave + 4 * gq + v;
      if (m < g.M) {
        cre[m * ldc + n] = cr[nt][v];
        cim[m * ldc + n] = real ? 0.f : ci[nt][v];
      }
    }
  }
}

// float32 matrix cores. LDS holds A^T (k rows, m contiguous; column m of
// row kk at m ^ ((kk >> 2) & 15)) and B (k rows, n contiguous).
template <int OPA, int NB>
__global__ __launch_bounds__(TT) void cgemm_tall_kernel(TArgs g) {
  constexpr int LDA = TM + 16, LDB = NB + 16, NTL = NB / 16;
  __shared__ float as[2][2][KB][LDA];
  __shared__ float bs[2][2][KB][LDB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int gq = lane >> 4, c = lane & 15;
  const int64_t k = blockIdx.z, m0 = (int64_t)blockIdx.y * TM;
  const bool real = (k == 0) || (g.real_last && k == g.K - 1);
  int64_t kbeg;
  const int64_t kd = tall_kd(g, kbeg), oa = k * g.sa + (OPA == 0 ? kbeg : kbeg * g.lda), ob = k * g.sb + kbeg * g.ldb;
  const float *are = g.are + oa, *aim = g.aim + oa, *bre = g.bre + ob, *bim = g.bim + ob;
  using L = StepLoad<OPA, NB>;
  L ld;
  auto put = [&](int b) {
#pragma unroll
    for (int u = 0; u < L::RA; ++u) {
      int m, kk;
      L::a_index(tid + TT * u, m, kk);
      const int ms = m ^ ((kk >> 2) & 15);
      as[b][0][kk][ms] = ld.ar[u];
      as[b][1][kk][ms] = ld.ai[u];
    }
#pragma unroll
    for (int u = 0; u < L::RB; ++u) {
      const int e = tid + TT * u, kk = e / NB, n = e % NB;
      bs[b][0][kk][n] = ld.br[u];
      bs[b][1][kk][n] = ld.bi[u];
    }
  };
  f32x4 cr[NTL], ci[NTL];
#pragma unroll
  for (int nt = 0; nt < NTL; ++nt) cr[nt] = ci[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int64_t nsteps = (kd + KB - 1) / KB;
  if (nsteps > 0) {
    ld.load(g, are, aim, bre, bim, m0, 0, kd, real, tid);
    put(0);
    __syncthreads();
  }
  for (int64_t st = 0; st < nsteps; ++st) {
    const int b = (int)(st & 1);
    if (st + 1 < nsteps) ld.load(g, are, aim, bre, bim, m0, (st + 1) * KB, kd, real, tid);
#pragma unroll
    for (int s = 0; s < KB / 4; ++s) {
      const int kk = 4 * s + gq;
      const int ms = (16 * wave + c) ^ ((kk >> 2) & 15);
      const float xr = as[b][0][kk][ms], xi = as[b][1][kk][ms];
#pragma unroll
      for (int nt = 0; nt < NTL; ++nt) {
        const float yr = bs[b][0][kk][16 * nt + c], yi = bs[b][1][kk][16 * nt + c];
        // Re += Ar Br - Ai Bi, Im += Ar Bi + Ai Br
        cr[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(xr, yr, cr[nt], 0, 0, 0);
        cr[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(-xi, yi, cr[nt], 0, 0, 0);
        ci[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(xr, yi, ci[nt], 0, 0, 0);
        ci[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(xi, yr, ci[nt], 0, 0, 0);
      }
    }
    if (st + 1 < nsteps) put(b ^ 1);
    __syncthreads();
  }
  tall_store<NB>(g, k, m0, wave, gq, c, cr, ci, real);
}

// Split bf16 matrix cores. A wavefront owns its 16 rows of op(A) alone, so a
// lane loads its 8 values of a 32-deep step (row c, k = 8 gq ..) straight from
// HBM, two steps ahead, and splits them in registers; only B, shared by the
// wavefronts, goes through LDS: four planes (hi re, lo re, hi im, lo im) of B^T as
// [n][k], 64 deep at a time, quads of k written at once (NB = 32: two buffers;
// 64: one, for two workgroups a CU). Bound: reading A. 1024 x 30 x 1024 over
// 65 slices (545 MB): op = N 216 -> 131 us, op = C 315 -> 135 (replaced: both
// operands split value by value into LDS by predicated loads).
template <int NB>
struct TallLds {
  // 160-byte rows (32 mod 64): the 16-byte fragment reads are free of bank conflicts
  static constexpr int KC = 64, LK = KC + 16, bufs = NB == 32 ? 2 : 1;
  __bf16 b[bufs][4][NB][LK];
};

__device__ __forceinline__ void split8(const float (&x)[8], bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const __bf16 h = (__bf16)x[e];
    hi[e] = h;
    lo[e] = (__bf16)(x[e] - (float)h);
  }
}

template <int OPA, int NB, bool REAL>
__device__ __forceinline__ void tall_split_body(const TArgs& g, int64_t k, int64_t m0, int64_t kbeg, int64_t kd,
                                                TallLds<NB>& lds) {
  using L = TallLds<NB>;
  constexpr int NTL = NB / 16, NP = REAL ? 1 : 2, KC = L::KC, RB = KC * NB / 4 / TT;
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int gq = lane >> 4, c = lane & 15;
  // rows beyond M and columns beyond N read the last one; they are never stored
  const int64_t m = m0 + 16 * wave + c < g.M ? m0 + 16 * wave + c : g.M - 1;
  const int64_t oa = k * g.sa + (OPA == 0 ? kbeg : kbeg * g.lda), ob = k * g.sb + kbeg * g.ldb;
  const float* ap[2] = {g.are + oa, g.aim + oa};
  const float* bp[2] = {g.bre + ob, g.bim + ob};
  const int64_t a0 = OPA == 0 ? m * g.lda + 8 * gq : 8 * gq * g.lda + m, astep = OPA == 0 ? KB : KB * g.lda;
  const int64_t nfull = kd / KB, last = nfull - 1, nch = (nfull + 1) / 2;

  float a[2][NP][8], rb[RB][NP][4];
  auto load_a = [&](float (&x)[NP][8], int64_t st) {
    const int64_t o = a0 + (st < last ? st : last) * astep;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if constexpr (OPA == 0) {
        __builtin_memcpy(x[p], ap[p] + o, 16);
        __builtin_memcpy(x[p] + 4, ap[p] + o + 4, 16);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[p][e] = ap[p][o + e * g.lda];
      }
    }
  };
  auto load_b = [&](int64_t ch) {
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const int e = tid + TT * u, n = e % NB < g.N ? e % NB : (int)g.N - 1;
      const int64_t k0 = ch * KC + 4 * (e / NB);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t kk = k0 + v < kd ? k0 + v : kd - 1;
#pragma unroll
        for (int p = 0; p < NP; ++p) rb[u][p][v] = bp[p][kk * g.ldb + n];
      }
    }
  };
  auto put_b = [&](int buf) {
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const int e = tid + TT * u, n = e % NB, kq = 4 * (e / NB);
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        bf16x4 hi, lo;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          hi[v] = (__bf16)rb[u][p][v];
          lo[v] = (__bf16)(rb[u][p][v] - (float)hi[v]);
        }
        *reinterpret_cast<bf16x4*>(&lds.b[buf][2 * p][n][kq]) = hi;
        *reinterpret_cast<bf16x4*>(&lds.b[buf][2 * p + 1][n][kq]) = lo;
      }
    }
  };
  f32x4 cr[NTL], ci[NTL];
#pragma unroll
  for (int nt = 0; nt < NTL; ++nt) cr[nt] = ci[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  struct Split {
    bf16x8 h[NP], l[NP];
  };
  auto products = [&](const Split& x, int buf, int k0) {
    const int col = k0 + 8 * gq;
    bf16x8 aih, ail, nih, nil;
    if constexpr (!REAL) {  // conjugate for op = C
      const bf16x8 th = bneg(x.h[1]), tl = bneg(x.l[1]);
      aih = OPA == 0 ? x.h[1] : th;
      ail = OPA == 0 ? x.l[1] : tl;
      nih = OPA == 0 ? th : x.h[1];
      nil = OPA == 0 ? tl : x.l[1];
    }
#pragma unroll
    for (int nt = 0; nt < NTL; ++nt) {
      const int n = 16 * nt + c;
      const bf16x8 brh = *reinterpret_cast<const bf16x8*>(&lds.b[buf][0][n][col]);
      const bf16x8 brl = *reinterpret_cast<const bf16x8*>(&lds.b[buf][1][n][col]);
      // Re += Ar Br - Ai Bi, Im += Ar Bi + Ai Br (three split terms each)
      cr[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.h[0], brh, cr[nt], 0, 0, 0);
      cr[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.h[0], brl, cr[nt], 0, 0, 0);
      cr[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.l[0], brh, cr[nt], 0, 0, 0);
      if constexpr (!REAL) {
        const bf16x8 bih = *reinterpret_cast<const bf16x8*>(&lds.b[buf][2][n][col]);
        const bf16x8 bil = *reinterpret_cast<const bf16x8*>(&lds.b[buf][3][n][col]);
        cr[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(nih, bih, cr[nt], 0, 0, 0);
        cr[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(nih, bil, cr[nt], 0, 0, 0);
        cr[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(nil, bih, cr[nt], 0, 0, 0);
        ci[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.h[0], bih, ci[nt], 0, 0, 0);
        ci[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.h[0], bil, ci[nt], 0, 0, 0);
        ci[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.l[0], bih, ci[nt], 0, 0, 0);
        ci[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aih, brh, ci[nt], 0, 0, 0);
        ci[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aih, brl, ci[nt], 0, 0, 0);
        ci[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ail, brh, ci[nt], 0, 0, 0);
      }
    }
  };
  auto split_a = [&](const float (&x)[NP][8]) {
    Split s;
#pragma unroll
    for (int p = 0; p < NP; ++p) split8(x[p], s.h[p], s.l[p]);
    return s;
  };
  if (nfull > 0) {
    load_b(0);
    load_a(a[0], 0);
    load_a(a[1], 1);
    put_b(0);
    __syncthreads();
    for (int64_t ch = 0; ch < nch; ++ch) {
      const int buf = L::bufs == 2 ? (int)(ch & 1) : 0;
      load_b(ch + 1 < nch ? ch + 1 : ch);  // (past the end: the same again, never used)
      {
        const Split x = split_a(a[0]);
        load_a(a[0], 2 * ch + 2);
        products(x, buf, 0);
      }
      if (2 * ch + 1 < nfull) {
        const Split x = split_a(a[1]);
        load_a(a[1], 2 * ch + 3);
        products(x, buf, KB);
      }
      if (L::bufs == 1) __syncthreads();
      put_b(L::bufs == 2 ? buf ^ 1 : 0);
      __syncthreads();
    }
  }
  // the last k < 32, zero beyond the contraction
  if (const int64_t kt = nfull * KB; kt < kd) {
    for (int e = tid; e < KB * NB; e += TT) {
      const int kk = e / NB, n = e % NB;
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const float v = kt + kk < kd && n < g.N ? bp[p][(kt + kk) * g.ldb + n] : 0.f;
        const __bf16 h = (__bf16)v;
        lds.b[0][2 * p][n][kk] = h;
        lds.b[0][2 * p + 1][n][kk] = (__bf16)(v - (float)h);
      }
    }
    float x[NP][8];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int64_t kk = kt + 8 * gq + e;
        x[p][e] = kk < kd ? ap[p][OPA == 0 ? m * g.lda + kk : kk * g.lda + m] : 0.f;
      }
    __syncthreads();
    products(split_a(x), 0, 0);
  }
  tall_store<NB>(g, k, m0, wave, gq, c, cr, ci, REAL);
}

template <int OPA, int NB>
__global__ __launch_bounds__(TT, 2) void cgemm_tall_split_kernel(TArgs g) {
  __shared__ __align__(16) TallLds<NB> lds;
  int64_t kbeg;
  const int64_t k = blockIdx.z, m0 = (int64_t)blockIdx.y * TM, kd = tall_kd(g, kbeg);
  if ((k == 0) || (g.real_last && k == g.K - 1))
    tall_split_body<OPA, NB, true>(g, k, m0, kbeg, kd, lds);
  else
    tall_split_body<OPA, NB, false>(g, k, m0, kbeg, kd, lds);
}

template <int OPA, int NB>
void launch_tall(const TArgs& g, int split, dim3 grid, hipStream_t st) {
  if (split)
    hipLaunchKernelGGL((cgemm_tall_split_kernel<OPA, NB>), grid, dim3(TT), 0, st, g);
  else
    hipLaunchKernelGGL((cgemm_tall_kernel<OPA, NB>), grid, dim3(TT), 0, st, g);
}

}  // namespace

// Parts of a split contraction, at least four steps each; whole rt-product in
// us, one part / parts: 1000 x 20 x 12 over 256 picks 71 / 31 in float32, 69 / 29
// in bf16x3, over 6000 2147 / 306 and 2117 / 250; 40 x 40 x 5 over 1700 190 / 34
// and 153 / 28.
int cgemm_tall_ksplit(int64_t K, bool real_last, int64_t M, int64_t N, int64_t Kd) {
  return N > 64 ? 1 : contraction_parts(K, real_last, (M + TM - 1) / TM, Kd / KB, 4);
}

// Takes float32 products C_k = op(A_k) B_k (op_b = N) with at most 64
// result columns (any contraction length), in float32 (split = 0)
// or split bf16 (split = 1); *handled says whether it did.
int cgemm_tall(const CGemm& p, int split, hipStream_t st, bool* handled) {
  *handled = false;
  if (p.op_b != 0 || p.N < 1 || p.N > 64 || p.Kd < 1 || p.M < 32) return TP_OK;
  if (p.K > 65535 || (p.M + TM - 1) / TM > 65535) return TP_OK;
  TArgs g{p.M, p.N, p.Kd, (const float*)p.are, (const float*)p.aim, (const float*)p.bre, (const float*)p.bim,
          (float*)p.cre, (float*)p.cim, p.lda, p.ldb, p.ldc, p.sa, p.sb, p.sc, p.K, p.real_last ? 1 : 0,
          p.kdim_dev, 1, p.part_re, p.part_im};
  const int parts = cgemm_tall_ksplit(p.K, p.real_last, p.M, p.N, p.Kd);
  if (p.part_re && p.part_im && p.part_cap >= int64_t(parts) * p.K * p.M * p.N) g.ksplit = parts;
  const dim3 grid((unsigned)g.ksplit, (unsigned)((p.M + TM - 1) / TM), (unsigned)p.K);
  if (p.op_a == 0) {
    if (p.N <= 32)
      launch_tall<0, 32>(g, split, grid, st);
    else
      launch_tall<0, 64>(g, split, grid, st);
  } else {
    if (p.N <= 32)
      launch_tall<1, 32>(g, split, grid, st);
    else
      launch_tall<1, 64>(g, split, grid, st);
  }
  TP_LAUNCH_CHECK();
  if (g.ksplit > 1)
    if (int rc = reduce_parts(p.part_re, p.part_im, g.ksplit, p.K, p.M, p.N, (float*)p.cre, (float*)p.cim, p.ldc, p.sc,
                              st))
      return rc;
  *handled = true;
  return TP_OK;
}

}  // namespace tp
