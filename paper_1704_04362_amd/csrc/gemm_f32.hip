// Per-slice complex products in float32 on the float32 matrix cores
// (v_mfma_f32_16x16x4f32): the slice loop of Algorithm 1 and the large
// Fourier-domain products of the dense t-SVD (Gram matrices A^H A, A A^H
// and U = A V) when the arithmetic is plain float32 (TP_PREC_F32).
//
// Complex slices use three real products (3M):
//   P1 = Ar Br, P2 = Ai Bi, P3 = (Ar + Ai)(Br + Bi),
//   Re C = P1 - P2, Im C = P3 - P1 - P2,
// with the sums Ar + Ai and Br + Bi formed once per staged element, so the
// matrix cores do three quarters of the four-product work (this kernel is
// bound by them); the real slices (DC, Nyquist) take P1 alone. Conjugate
// transposes (op = 1) are applied while staging: the operand is read
// transposed and its imaginary part negated before the sum is formed.
//
// Tiling: a 256-thread workgroup owns a 128 x 128 (64 x 64) tile of one
// Fourier slice; each of its four wavefronts owns 64 x 64 (32 x 32), that is 4 x 4
// (2 x 2) matrix-core tiles of 16 x 16, three accumulators each. One wavefront a
// SIMD (three) hides little, so a step's address arithmetic is one 32-bit
// offset a value that stays the same over the steps, and the operations are
// compiled in: 33 slices of 512 x 2048 x 512 1302 -> 1204 us (88 TFLOP/s
// executed), 51 of 256 x 256 x 256 A^H A 101 -> 88. Either tile adds an
// output's products in the same order. A 16-deep step of both operands is
// staged through registers (loaded one step ahead, never predicated off)
// into one of two LDS buffers as three planes (re, im, re + im), stored per
// row with the contraction index permuted so that a lane's four values for
// the four 4-deep sub-steps are one 16-byte chunk: position 4 (k mod 4) +
// k / 4 of the row, chunk c of row r stored at chunk c ^ (r mod 4). A
// fragment read (16 rows x 4 chunks per wavefront) then covers 1 KB of LDS
// once.
//
// Products with few output tiles and a long contraction split the
// contraction into parts that write float32 partial planes, summed in part
// order afterwards (deterministic).
#include <type_traits>

#include "common.hpp"

namespace tp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int FM = 128, FN = 128, FK = 16, FT = 256;  // (tiles of 32 W, W = 4 or 2)

struct FArgs {
  int64_t M, N, Kd;
  const float *are, *aim, *bre, *bim;
  float *cre, *cim;
  int64_t lda, ldb, ldc, sa, sb, sc;
  int op_a, op_b;
  int64_t K;
  int real_last;
  const int64_t* kdim_dev;
  int ksplit;
  float *pre, *pim;  // partial planes [part][K][M][N] when ksplit > 1
};

// LDS float offset of element (row, k) of a staged 16-deep operand block
__device__ __forceinline__ int lds_pos(int row, int k) {
  const int c = k & 3, w = k >> 2;
  return row * 16 + 4 * (c ^ (row & 3)) + w;
}

// Stages one 16-deep step of an operand (rows of op(X): 32 W x 16) from
// global memory into registers. along_k: the stored operand is contiguous
// along the contraction index (op_a = 0 for A, op_b = 1 for B); otherwise
// along the rows. Thread t covers 2 W elements. Loads are never predicated
// off: an element outside the operand reads the slice origin instead (always
// valid) and is cleared when it is stored to LDS, so all loads of a step stay
// in flight together behind the products of the current step.
template <int W>
struct Stage {
  float re[2 * W], im[2 * W];
  uint32_t keep;  // bit p: element p lies inside the operand
};

template <int W>
__device__ __forceinline__ void stage_coords(const bool along_k, int p, int& row, int& kk) {
  const int t = threadIdx.x;
  if (along_k) {
    row = (t >> 4) + 16 * p;
    kk = t & 15;
  } else {
    row = t % (32 * W);
    kk = t / (32 * W) + FT / (32 * W) * p;
  }
}

template <bool REAL, int W, typename Off>
__device__ __forceinline__ void load_stage(Stage<W>& s, const float* xr, const float* xi, int64_t ld, bool along_k,
                                           int64_t r0, int64_t rows, int64_t k0, int64_t kend) {
  s.keep = 0;
  // a uniform origin and the values' offsets in the tile (Off: 32 bits below
  // ld = 2^23), of which only the test for the end of the contraction is not
  // the same in every step
  const int rlim = (int)(rows - r0 < 32 * W ? rows - r0 : 32 * W), klim = (int)(kend - k0 < FK ? kend - k0 : FK);
  const int64_t o = along_k ? r0 * ld + k0 : k0 * ld + r0;
  xr += o;
  xi += o;
#pragma unroll
  for (int p = 0; p < 2 * W; ++p) {
    int row, kk;
    stage_coords<W>(along_k, p, row, kk);
    const Off r = row < rlim ? row : 0, l = (Off)ld;
    const Off tr = along_k ? r * l : r, tk = along_k ? (Off)kk : kk * l;
    const Off t = tr + (kk < klim ? tk : 0u);
    s.re[p] = xr[t];
    if (!REAL) s.im[p] = xi[t];
    s.keep |= row < rlim && kk < klim ? (1u << p) : 0u;
  }
}

template <bool REAL, int W>
__device__ __forceinline__ void store_stage(const Stage<W>& s, bool along_k, bool conj, float* lre, float* lim,
                                            float* lsum) {
#pragma unroll
  for (int p = 0; p < 2 * W; ++p) {
    int row, kk;
    stage_coords<W>(along_k, p, row, kk);
    const bool ok = (s.keep >> p) & 1u;
    const int o = lds_pos(row, kk);
    const float vr = ok ? s.re[p] : 0.f;
    lre[o] = vr;
    if (!REAL) {
      const float vi = ok ? (conj ? -s.im[p] : s.im[p]) : 0.f;
      lim[o] = vi;
      lsum[o] = vr + vi;
    }
  }
}

template <bool REAL, int W, int OPA, int OPB, typename Off>
__device__ __forceinline__ void f32_body(const FArgs& g, int64_t k, int part, float* lds) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const int64_t m0 = (int64_t)blockIdx.y * (32 * W), n0 = (int64_t)blockIdx.x * (32 * W);
  int64_t Kd = g.Kd;
  if (g.kdim_dev) {
    const int64_t lim = *g.kdim_dev;
    Kd = lim < Kd ? (lim < 0 ? 0 : lim) : Kd;
  }
  const int64_t kchunk = g.ksplit > 1 ? ((Kd + g.ksplit - 1) / g.ksplit + FK - 1) / FK * FK : Kd;
  const int64_t kbeg = (int64_t)part * kchunk;
  const int64_t kend = kbeg + kchunk < Kd ? kbeg + kchunk : Kd;
  const float* are = g.are + k * g.sa;
  const float* aim = g.aim + k * g.sa;
  const float* bre = g.bre + k * g.sb;
  const float* bim = g.bim + k * g.sb;
  constexpr bool a_along_k = OPA == 0, b_along_k = OPB != 0, a_conj = OPA != 0, b_conj = OPB != 0;

  // LDS: 2 buffers x [A re, A im, A sum, B re, B im, B sum] x 32 W rows x 16
  constexpr int PL = 32 * W * FK;
  auto buf = [&](int b, int which) { return lds + (b * 6 + which) * PL; };

  // p1 = Ar Br, p2 = Ai Bi, p3 = (Ar + Ai)(Br + Bi)
  f32x4 p1[W][W], p2[W][W], p3[W][W];
#pragma unroll
  for (int i = 0; i < W; ++i)
#pragma unroll
    for (int j = 0; j < W; ++j) {
      p1[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      p2[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      p3[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

  Stage<W> sa, sb;
  const int64_t nsteps = kend > kbeg ? (kend - kbeg + FK - 1) / FK : 0;
  if (nsteps > 0) {
    load_stage<REAL, W, Off>(sa, are, aim, g.lda, a_along_k, m0, g.M, kbeg, kend);
    load_stage<REAL, W, Off>(sb, bre, bim, g.ldb, b_along_k, n0, g.N, kbeg, kend);
  }
  const int fr = lane & 15, fq = lane >> 4;
  for (int64_t st = 0; st < nsteps; ++st) {
    const int b = (int)(st & 1);
    store_stage<REAL, W>(sa, a_along_k, a_conj, buf(b, 0), buf(b, 1), buf(b, 2));
    store_stage<REAL, W>(sb, b_along_k, b_conj, buf(b, 3), buf(b, 4), buf(b, 5));
    __syncthreads();
    if (st + 1 < nsteps) {
      const int64_t k0 = kbeg + (st + 1) * FK;
      load_stage<REAL, W, Off>(sa, are, aim, g.lda, a_along_k, m0, g.M, k0, kend);
      load_stage<REAL, W, Off>(sb, bre, bim, g.ldb, b_along_k, n0, g.N, k0, kend);
    }
    // fragments: lane (fq, fr) reads row fr of a 16-row tile, chunk fq:
    // the values for k = fq + 4 s, s = 0..3 (sub-step s of the 16-deep step)
    f32x4 br_[W], bi_[W], bs_[W];
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const int row = wc * (16 * W) + j * 16 + fr;
      const int o = row * 16 + 4 * (fq ^ (row & 3));
      br_[j] = *reinterpret_cast<const f32x4*>(buf(b, 3) + o);
      if (!REAL) {
        bi_[j] = *reinterpret_cast<const f32x4*>(buf(b, 4) + o);
        bs_[j] = *reinterpret_cast<const f32x4*>(buf(b, 5) + o);
      }
    }
#pragma unroll
    for (int i = 0; i < W; ++i) {
      const int row = wr * (16 * W) + i * 16 + fr;
      const int o = row * 16 + 4 * (fq ^ (row & 3));
      const f32x4 ar = *reinterpret_cast<const f32x4*>(buf(b, 0) + o);
      f32x4 ai = f32x4{0.f, 0.f, 0.f, 0.f}, as = f32x4{0.f, 0.f, 0.f, 0.f};
      if (!REAL) {
        ai = *reinterpret_cast<const f32x4*>(buf(b, 1) + o);
        as = *reinterpret_cast<const f32x4*>(buf(b, 2) + o);
      }
      // product-outer order: consecutive matrix-core operations update
      // different accumulators, so none waits for the one before it
#pragma unroll
      for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int j = 0; j < W; ++j)
          p1[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[s], br_[j][s], p1[i][j], 0, 0, 0);
        if (!REAL) {
#pragma unroll
          for (int j = 0; j < W; ++j)
            p2[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ai[s], bi_[j][s], p2[i][j], 0, 0, 0);
#pragma unroll
          for (int j = 0; j < W; ++j)
            p3[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(as[s], bs_[j][s], p3[i][j], 0, 0, 0);
        }
      }
    }
    __syncthreads();
  }

  // lane holds rows 4 (lane / 16) + v, column lane % 16 of each 16 x 16 tile
  float *cre, *cim;
  int64_t ldc;
  if (g.ksplit > 1) {
    const int64_t per = g.M * g.N;
    cre = g.pre + ((int64_t)part * g.K + k) * per;
    cim = g.pim + ((int64_t)part * g.K + k) * per;
    ldc = g.N;
  } else {
    cre = g.cre + k * g.sc;
    cim = g.cim + k * g.sc;
    ldc = g.ldc;
  }
#pragma unroll
  for (int i = 0; i < W; ++i)
#pragma unroll
    for (int j = 0; j < W; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t gm = m0 + wr * (16 * W) + i * 16 + 4 * fq + v;
        const int64_t gn = n0 + wc * (16 * W) + j * 16 + fr;
        if (gm < g.M && gn < g.N) {
          const float a = p1[i][j][v], c = p2[i][j][v];
          cre[gm * ldc + gn] = REAL ? a : a - c;
          cim[gm * ldc + gn] = REAL ? 0.f : p3[i][j][v] - a - c;
        }
      }
}

template <int W, int OPA, int OPB, typename Off>
__global__ __launch_bounds__(FT, W == 4 ? 1 : 3) void cgemm_f32_kernel(FArgs g) {
  __shared__ __attribute__((aligned(16))) float lds[2 * 6 * 32 * W * FK];  // 96 or 48 KB
  const int part = (int)(blockIdx.z % (unsigned)g.ksplit);
  const int64_t k = blockIdx.z / (unsigned)g.ksplit;
  const bool real = k == 0 || (g.real_last && k == g.K - 1);
  if (real)
    f32_body<true, W, OPA, OPB, Off>(g, k, part, lds);
  else
    f32_body<false, W, OPA, OPB, Off>(g, k, part, lds);
}

}  // namespace

// Parts of a split contraction for the float32 matrix-core product, at least
// eight steps each. Whole rt-product in us, before (one part up to a
// contraction of 2048, then at least 64 steps a part) / now:
// 300 x 300 x 5 over 256 picks 103 / 33, 1700 571 / 77, 6000 548 / 206; 512 x
// 512 x 12 over 256 144 / 64, 6000 1890 / 813; 500 x 300 x 8 over 256 101 / 40, 6000
// 482 / 398 (counted in tiles of 128, whichever are taken).
int cgemm_f32_ksplit(int64_t K, bool real_last, int64_t M, int64_t N, int64_t Kd) {
  return contraction_parts(K, real_last, ((M + FM - 1) / FM) * ((N + FN - 1) / FN), Kd / FK, 8);
}

// Tiles of 128 (one workgroup a CU) or 64: the one whose workgroups take the
// fewest rounds over the 256 CUs, complex tiles first, a real one a third of the
// time, a tile of 64 0.28 of one of 128 (a quarter of its products; measured
// over 128 x 128 tiles that are full: 33 slices of 512 x 512 x 512 317 us in
// tiles of 128, 357 of 64). Ragged sides and few tiles go to 64: 41 slices of
// 301 x 777 x 259 452 / 283, 17 of 100 x 100 x 100 37 / 16, 12 of 384 x 384 x 384
// 113 / 72.
static bool f32_wide(const CGemm& p, int ksplit) {
  const int64_t nreal = p.real_last && p.K > 1 ? 2 : 1;
  const auto tiles = [&](int64_t side, int64_t slices) {
    return (p.M + side - 1) / side * ((p.N + side - 1) / side) * slices * ksplit;
  };
  const int64_t c4 = tiles(128, p.K - nreal), r4 = tiles(128, nreal), c2 = tiles(64, p.K - nreal), r2 = tiles(64, nreal);
  const int64_t thirds = std::max(3 * ((c4 + 255) / 256), (3 * c4 + r4 + 255) / 256);
  return 100 * thirds <= 3 * 28 * ((3 * c2 + r2 + 767) / 768);
}

// Takes float32 products with at least 16 rows and columns and a contraction
// of at least 64; reports handled = false for the others.
int cgemm_f32mfma(const CGemm& p, hipStream_t st, bool* handled) {
  *handled = false;
  if (p.M < 16 || p.N < 16 || p.Kd < 64) return TP_OK;
  if (p.K > 65535) return TP_OK;
  int ksplit = cgemm_f32_ksplit(p.K, p.real_last, p.M, p.N, p.Kd);
  if (ksplit > 1 && (!p.part_re || !p.part_im || p.part_cap < int64_t(ksplit) * p.K * p.M * p.N)) ksplit = 1;
  if (p.K * ksplit > 65535) ksplit = 1;
  FArgs g{p.M, p.N, p.Kd, (const float*)p.are, (const float*)p.aim, (const float*)p.bre, (const float*)p.bim,
          (float*)p.cre, (float*)p.cim, p.lda, p.ldb, p.ldc, p.sa, p.sb, p.sc, p.op_a, p.op_b, p.K,
          p.real_last ? 1 : 0, p.kdim_dev, ksplit, p.part_re, p.part_im};
  // (64-row tiles of more than 4,194,240 rows pass the 65,535 rows of the grid)
  const bool near = p.lda < (1 << 23) && p.ldb < (1 << 23), wide = !near || p.M > 64 * 65535 || f32_wide(p, ksplit);
  const int64_t side = wide ? 128 : 64, gx = (p.N + side - 1) / side, gy = (p.M + side - 1) / side;
  if (gx > 0x7fffffff || gy > 65535) return TP_OK;
  const dim3 grid((unsigned)gx, (unsigned)gy, (unsigned)(p.K * ksplit));
  const auto launch = [&](auto w, auto off) {
    constexpr int W = decltype(w)::value;
    using Off = decltype(off);
    const auto kernel = p.op_a ? (p.op_b ? cgemm_f32_kernel<W, 1, 1, Off> : cgemm_f32_kernel<W, 1, 0, Off>)
                               : (p.op_b ? cgemm_f32_kernel<W, 0, 1, Off> : cgemm_f32_kernel<W, 0, 0, Off>);
    hipLaunchKernelGGL(kernel, grid, dim3(FT), 0, st, g);
  };
  if (!near)
    launch(std::integral_constant<int, 4>{}, uint64_t{});
  else if (wide)
    launch(std::integral_constant<int, 4>{}, uint32_t{});
  else
    launch(std::integral_constant<int, 2>{}, uint32_t{});
  TP_LAUNCH_CHECK();
  if (ksplit > 1)
    if (int rc = reduce_parts(p.part_re, p.part_im, ksplit, p.K, p.M, p.N, (float*)p.cre, (float*)p.cim, p.ldc, p.sc, st))
      return rc;
  *handled = true;
  return TP_OK;
}

}  // namespace tp
