// Singular value thresholding of every Fourier slice (the closed-form
// L-update of Algorithm 7 with the tensor nuclear norm of eq. tnuc), the
// elementwise updates of the ADMM loops (completion, eq. tlow6, and robust
// PCA, eq. tlow7) and the slice gathers that feed CUR t-NN (Algorithm 6).
//
// SVD by block one-sided Jacobi on rows: every slice M (n1 x n2) is kept as
// X = U^H M together with Uh = U^H (both row-major, float32 planar). A step
// takes a pair of 16-row blocks (32 rows), forms their Gram matrix
// G = X_p X_p^H in float64, diagonalises it with the LDS Jacobi solver
// (G = V diag V^H) and rotates both X_p and Uh_p by V^H, which makes the 32
// rows mutually orthogonal. A round-robin tournament over the blocks visits
// all block pairs in a sweep; the disjoint pairs of a round are independent
// workgroups. A slice is converged when every pair in a sweep had
// max |G_st| / max(G_ss, G_tt) below the tolerance (measured against the
// larger row: rows stored in float32 keep a rounding floor of about
// eps_32 times the larger row); later launches for it return at once, so a
// fixed launch sequence needs no host synchronisation.
// At the end the rows of X are U^H M = Sigma V^H: sigma_i = ||x_i||, and
//   L = U diag(max(1 - tau / sigma_i, 0)) X = Uh^H (D X).
#include <cmath>

#include "common.hpp"
#include "jacobi.hpp"
#include "jacobi32.hpp"
#include "svt.hpp"

namespace tp {
namespace {

constexpr int RB = 16;       // rows per block
constexpr int PR = 2 * RB;   // rows per pair
constexpr int NT = 256;
constexpr int PT = 512;      // threads of a pair step
// Cyclic Jacobi sweeps on the 32 x 32 Gram matrix of a pair step. The outer
// sweeps revisit every pair until all of them are orthogonal, so a pair step
// need not diagonalise its Gram matrix exactly: one inner sweep costs about
// one more outer sweep in total against a full inner solve, at a fraction of
// the price per step.
constexpr int kInnerSweeps = 1;
// A pair whose off-diagonal mass is within this of its Gram matrix's (Frobenius
// norms) is not rotated: below, its entries are rounding of the large rows'
// products, and the loop of api_svt.cpp needs the pair steps' bits unchanged.
// (The sums are taken only where no single entry decides: 32 entries of at most
// the largest a side, so the norm is at most 32 times that one.)
constexpr double kPairTol = 1e-14;

struct PairArgs {
  int64_t K, n1, n2;
  int64_t k0;        // first slice of this launch (blockIdx.y counts from it)
  float *xre, *xim;  // K x n1 x n2
  float *ure, *uim;  // K x n1 x n1
  int nb;            // number of blocks (even; the last may be partial or empty)
  int real_last;
  float* ratio;      // (nb-1) x K x (nb/2) ratios of this sweep, per round
  const int* conv;   // K flags
  double tol;
};

__device__ __forceinline__ int tournament(int pos, int round, int nb) {
  return pos == 0 ? 0 : 1 + ((pos - 1 + round) % (nb - 1));
}

typedef double d4 __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4f64: A lane l = A[l % 16][l / 16], B lane l =
// B[l / 16][l % 16], D lane l register v = D[4 v + l / 16][l % 16], as
// measured on gfx950.
#define TP_MFMA64(a, b, c) __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0)

// Gram matrix G_st = sum_j x_s[j] conj(x_t[j]) of the 32 staged rows, straight
// from global memory into the operand layout: lane (row r, group g) reads the
// four columns 16 q + 4 g .. + 3 of its row with one 16-byte load, and a 4 x 4
// transposition over the lane groups hands it column 16 q + 4 kk + g for the
// product kk. A 16 x 16 block's re = Xr Xr^T + Xi Xi^T and im = Xi Xr^T - Xr Xi^T
// run over all columns in order. Of the eight only seven are formed, one per
// wavefront (re of block (1,0) is that of (0,1) transposed). Four column groups'
// loads are in flight at a time (kAhead).
__device__ __forceinline__ void swap32(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
// v[c] of lane group g becomes v[g] of lane group c
__device__ __forceinline__ void transpose4(float (&v)[4]) {
  swap32(v[0], v[2]);
  swap32(v[1], v[3]);
  swap16(v[0], v[1]);
  swap16(v[2], v[3]);
}

struct GramCols {
  float r[4], i[4];
};

// missing rows and the imaginary part of a real slice to zero, then to the
// operand layout
__device__ __forceinline__ void gram_fix(GramCols& z, bool live, bool real) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    z.r[e] = live ? z.r[e] : 0.f;
    z.i[e] = live && !real ? z.i[e] : 0.f;
  }
  transpose4(z.r);
  transpose4(z.i);
}

template <bool IM>
__device__ __forceinline__ void gram_products(const GramCols& x, const GramCols& y, d4& acc) {
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const double ar = (double)x.r[kk], ai = (double)x.i[kk];
    const double br = (double)y.r[kk], bi = (double)y.i[kk];
    acc = TP_MFMA64(IM ? ai : ar, br, acc);
    acc = TP_MFMA64(IM ? -ar : ai, bi, acc);
  }
}

template <bool IM, bool DIAG>
__device__ __forceinline__ d4 gram_block(const float* re, const float* im, int64_t ncols, const int* rows, bool real,
                                         int ba, int bb) {
  const int l = threadIdx.x & 63, g = l >> 4;
  const int ra = rows[16 * ba + (l & 15)], rb = rows[16 * bb + (l & 15)];
  const bool alive = ra >= 0, blive = rb >= 0;
  const int64_t oa = (int64_t)(alive ? ra : 0) * ncols, ob = (int64_t)(blive ? rb : 0) * ncols;
  const int64_t nq = ncols / 16;  // whole groups of 16 columns
  struct Pair {
    GramCols a, b;
  };
  auto load = [&](int64_t q, Pair& z) {
    const int64_t c = 16 * (q < nq ? q : nq - 1) + 4 * g;
    __builtin_memcpy(z.a.r, re + oa + c, 16);
    __builtin_memcpy(z.a.i, im + oa + c, 16);
    if (!DIAG) {
      __builtin_memcpy(z.b.r, re + ob + c, 16);
      __builtin_memcpy(z.b.i, im + ob + c, 16);
    }
  };
  d4 acc = {0.0, 0.0, 0.0, 0.0};
  auto use = [&](const Pair& z) {
    GramCols x = z.a, y = z.b;
    gram_fix(x, alive, real);
    if (DIAG)
      y = x;
    else
      gram_fix(y, blive, real);
    gram_products<IM>(x, y, acc);
  };
  if (nq > 0) {
    // unconditional loads (past the end the last group again), so that they
    // stay in flight over the products
    constexpr int kAhead = 4;
    Pair z[kAhead];
#pragma unroll
    for (int t = 0; t < kAhead; ++t) load(t, z[t]);
    for (int64_t q = 0; q < nq; q += kAhead) {
#pragma unroll
      for (int t = 0; t < kAhead; ++t) {
        if (q + t < nq) use(z[t]);
        load(q + t + kAhead, z[t]);
      }
    }
  }
  if (16 * nq < ncols) {
    Pair z;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t c = 16 * nq + 4 * g + e;
      const bool in = c < ncols;
      const int64_t o = in ? c : 0;
      z.a.r[e] = in ? re[oa + o] : 0.f;
      z.a.i[e] = in ? im[oa + o] : 0.f;
      z.b.r[e] = in && !DIAG ? re[ob + o] : 0.f;
      z.b.i[e] = in && !DIAG ? im[ob + o] : 0.f;
    }
    use(z);
  }
  return acc;
}

// Rotation of the 32 rows of X and of U^H by V^H in place: out_s =
// sum_t conj(V_ts) in_t, on the float64 matrix cores (re = Vr xr + Vi xi,
// im = Vr xi - Vi xr). The 32-column tiles of X and then of U^H are dealt to the
// wavefronts. Lane (group g, j) reads columns 2j, 2j + 1 of the tile from
// rows 4 kk + g straight into the operand layout (the even columns form one
// 16-column product, the odd ones another): every element is read and
// written once, nothing is staged or synchronised, and a tile's loads are in
// flight during the products of the one before (the first tile's during the
// inner sweep).
struct RotTile {
  float2 r[8], i[8];
};

struct RotArgs {
  float *xre, *xim, *ure, *uim;
  int64_t n1, n2, nx;  // nx: tiles of X
  bool real, full;     // full: all 32 rows exist
};

__device__ __forceinline__ void rot_tile(const RotArgs& a, int64_t t, float*& re, float*& im, int64_t& ncols,
                                         int64_t& c0) {
  const bool x = t < a.nx;
  re = x ? a.xre : a.ure;
  im = x ? a.xim : a.uim;
  ncols = x ? a.n2 : a.n1;
  c0 = 32 * (x ? t : t - a.nx);
}

// Unconditional loads from clamped addresses (matrices have at least two
// columns where there is something to rotate): they stay in flight. The last
// column of an odd number comes as the second of its pair (rot_fix).
__device__ __forceinline__ void rot_load(const RotArgs& a, int64_t t, const int (&row)[8], RotTile& z) {
  float *re, *im;
  int64_t ncols, c0;
  rot_tile(a, t, re, im, ncols, c0);
  int64_t c = c0 + 2 * (threadIdx.x & 15);
  c = c + 2 > ncols ? ncols - 2 : c;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) {
    const int64_t o = (int64_t)(row[kk] < 0 ? 0 : row[kk]) * ncols + c;
    __builtin_memcpy(&z.r[kk], re + o, 8);
    __builtin_memcpy(&z.i[kk], im + o, 8);
  }
}

// missing rows and the imaginary part of a real slice to zero
__device__ __forceinline__ void rot_fix(const RotArgs& a, int64_t t, const int (&row)[8], RotTile& z) {
  float *re, *im;
  int64_t ncols, c0;
  rot_tile(a, t, re, im, ncols, c0);
  if (!a.real && a.full && c0 + 32 <= ncols) return;
  const bool last = c0 + 2 * (threadIdx.x & 15) + 1 == ncols;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) {
    if (last) {
      z.r[kk].x = z.r[kk].y;
      z.i[kk].x = z.i[kk].y;
    }
    if (row[kk] < 0) z.r[kk] = float2{0.f, 0.f};
    if (row[kk] < 0 || a.real) z.i[kk] = float2{0.f, 0.f};
  }
}

__device__ __forceinline__ void rot_store(const RotArgs& a, int64_t t, const int* rows, int h, const d4 (&outr)[2],
                                          const d4 (&outi)[2]) {
  float *re, *im;
  int64_t ncols, c0;
  rot_tile(a, t, re, im, ncols, c0);
  const int l = threadIdx.x & 63, g = l >> 4;
  const int64_t c = c0 + 2 * (l & 15);
  const bool whole = c0 + 32 <= ncols;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int s = rows[16 * h + 4 * v + g];
    const int64_t o = (int64_t)s * ncols + c;
    const float2 wr{(float)outr[0][v], (float)outr[1][v]}, wi{(float)outi[0][v], (float)outi[1][v]};
    if (whole && a.full) {
      __builtin_memcpy(re + o, &wr, 8);
      if (!a.real) __builtin_memcpy(im + o, &wi, 8);
    } else if (s >= 0 && c < ncols) {
      re[o] = wr.x;
      if (!a.real) im[o] = wi.x;
      if (c + 1 < ncols) {
        re[o + 1] = wr.y;
        if (!a.real) im[o + 1] = wi.y;
      }
    }
  }
}

// `x` holds the wavefront's first tile
__device__ __forceinline__ void rotate_rows(const RotArgs& a, const Cz* V, const int* rows, const int (&row)[8],
                                            RotTile& x) {
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = l >> 4, j = l & 15;
  const int64_t nt = a.nx + (a.n1 + 31) / 32;
  for (int64_t t = w; t < nt; t += PT / 64) {
    if (t != w) rot_load(a, t, row, x);
    rot_fix(a, t, row, x);
#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
      d4 outr[2], outi[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) outr[q] = outi[q] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        const Cz v = V[(4 * kk + g) * 32 + 16 * h + j];
        // converted again for the second half: 64 registers of doubles less
        asm volatile("" : "+v"(x.r[kk].x), "+v"(x.r[kk].y), "+v"(x.i[kk].x), "+v"(x.i[kk].y));
        const double br[2] = {(double)x.r[kk].x, (double)x.r[kk].y}, bi[2] = {(double)x.i[kk].x, (double)x.i[kk].y};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          outr[q] = TP_MFMA64(v.x, br[q], outr[q]);
          outi[q] = TP_MFMA64(v.x, bi[q], outi[q]);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          outr[q] = TP_MFMA64(v.y, bi[q], outr[q]);
          outi[q] = TP_MFMA64(-v.y, br[q], outi[q]);
        }
      }
      rot_store(a, t, rows, h, outr, outi);
    }
  }
}

// Whether the off-diagonal mass of h is within kPairTol of the total
__device__ __forceinline__ bool negligible(const Cz* h, double (*red)[PT / 64]) {
  const int tid = threadIdx.x, w = tid >> 6;
  double off = 0.0, tot = 0.0;
  for (int e = tid; e < PR * PR; e += PT) {
    const double m = fma(h[e].x, h[e].x, h[e].y * h[e].y);
    tot += m;
    off += e % (PR + 1) ? m : 0.0;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    off += __shfl_xor(off, o);
    tot += __shfl_xor(tot, o);
  }
  __syncthreads();
  if ((tid & 63) == 0) {
    red[0][w] = off;
    red[1][w] = tot;
  }
  __syncthreads();
  off = tot = 0.0;
  for (int q = 0; q < PT / 64; ++q) {
    off += red[0][q];
    tot += red[1][q];
  }
  return off <= kPairTol * kPairTol * tot;
}

// One pair step of one slice, eight wavefronts. On one CU for 256 columns
// (cycles of a 2.2 GHz CU): Gram matrix 31,000, test and symmetrisation 3,000,
// inner sweep 46,000 (31 rounds bound by float64 issue, see jacobi32.hpp),
// rotations 33,000 (the rate of the float64 matrix cores), against 184,000 in
// all for four wavefronts staging float64 rows through LDS with H and V of the
// sweep updated there. 408 pair steps (51 slices of 256 x 256) take 93 us on
// one stream (168 before), a cold 256 x 256 x 100 thresholding 15.3 ms (19.4),
// ten completion iterations 46 ms (58.5); the results are the same bits.
__global__ __launch_bounds__(PT, 4) void svt_pair_kernel(PairArgs a, int round) {
  // raw Gram matrix (planar, row stride 33) over H[1] and V until the sweep
  __shared__ union {
    Jacobi32Shared jac;
    struct {
      Cz h0[32 * 32];
      double re[PR][PR + 1], im[PR][PR + 1];
    } raw;
  } sh;
  __shared__ int rows[PR];
  __shared__ double ratio_red[PT / 64], mass_red[2][PT / 64];
  __shared__ int top;  // upper half of the largest diagonal entry
  const int64_t k = a.k0 + blockIdx.y;
  const int pair = blockIdx.x;
  const int tid = threadIdx.x, l = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (a.conv[k]) return;
  const bool real = k == 0 || (a.real_last && k == a.K - 1);
  const int ba = tournament(pair, round, a.nb), bb = tournament(a.nb - 1 - pair, round, a.nb);
  if (tid < PR) {
    const int blk = tid < RB ? ba : bb;
    const int64_t r = (int64_t)blk * RB + (tid % RB);
    rows[tid] = r < a.n1 ? (int)r : -1;
  }
  if (tid == 0) top = 0;
  const RotArgs rot{a.xre + k * a.n1 * a.n2, a.xim + k * a.n1 * a.n2, a.ure + k * a.n1 * a.n1,
                    a.uim + k * a.n1 * a.n1, a.n1,                    a.n2,
                    (a.n2 + 31) / 32,        real,                    (int64_t)(max(ba, bb) + 1) * RB <= a.n1};
  __syncthreads();
  if (w < 7) {
    auto put = [&](const d4& acc, int s0, int t0, bool is_im) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int s = s0 + 4 * v + (l >> 4), t = t0 + (l & 15);
        if (is_im) {
          sh.raw.im[s][t] = acc[v];
        } else {
          sh.raw.re[s][t] = acc[v];
          if (s0 != t0) sh.raw.re[t][s] = acc[v];
          if (s == t) atomicMax(&top, __double2hiint(acc[v]));
        }
      }
    };
    const int blk = w == 0 || w == 1 ? 0 : 1;  // diagonal blocks: wavefronts 0, 1, 5, 6
    if (w == 0 || w == 5)
      put(gram_block<false, true>(rot.xre, rot.xim, a.n2, rows, real, blk, blk), 16 * blk, 16 * blk, false);
    else if (w == 1 || w == 6)
      put(gram_block<true, true>(rot.xre, rot.xim, a.n2, rows, real, blk, blk), 16 * blk, 16 * blk, true);
    else if (w == 2)
      put(gram_block<false, false>(rot.xre, rot.xim, a.n2, rows, real, 0, 1), 0, 16, false);
    else
      put(gram_block<true, false>(rot.xre, rot.xim, a.n2, rows, real, w == 3 ? 0 : 1, w == 3 ? 1 : 0),
          w == 3 ? 0 : 16, w == 3 ? 16 : 0, true);
  }
  __syncthreads();
  // largest off-diagonal entry relative to the larger squared norm of its
  // two rows, |G_st| / max(G_ss, G_tt). Rows are stored in float32, so a
  // rotation leaves rounding of size eps_32 |x_big| in the smaller row and
  // |G_st| cannot fall below ~eps_32 max(G_ss, G_tt): the usual
  // |G_st| / sqrt(G_ss G_tt) would never reach the tolerance for pairs whose
  // norms differ by more than tol / eps_32 and every call would run its
  // full sweep budget. Scaled by the larger row, the residual rotation
  // angle is below tol relative to the pair's spectral gap, which bounds
  // the error of the thresholded result by ~tol ||M||.
  double mr = 0.0;
  // (from above the largest diagonal entry)
  const double bound = __hiloint2double(top + 0x100000, 0) * (PR * kPairTol);
  bool large = false;  // one entry of more than kPairTol of the Frobenius norm
#pragma unroll
  for (int q = 0; q < PR * PR / PT; ++q) {
    const int e = tid + PT * q, s = e / PR, t = e - s * PR;
    const double gr = sh.raw.re[s][t], gi = sh.raw.im[s][t];
    const double hr = sh.raw.re[t][s], hi = sh.raw.im[t][s];
    // exactly Hermitian
    const double re = s == t ? gr : 0.5 * (gr + hr);
    const double im = s < t ? 0.5 * (gi - hi) : (s > t ? -(0.5 * (hi - gi)) : 0.0);
    if (s != t) {
      const double d = fmax(sh.raw.re[s][s], sh.raw.re[t][t]);
      if (d > 0.0) mr = fmax(mr, sqrt(fma(gr, gr, gi * gi)) / d);
      large |= fmax(fabs(re), fabs(im)) > bound;
    }
    sh.raw.h0[e] = Cz{re, im};
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mr = fmax(mr, __shfl_xor(mr, o));
  large = __any(large);
  if (l == 0) {
    ratio_red[w] = mr;
    mass_red[0][w] = large ? 1.0 : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PT / 64; ++q) {
    mr = fmax(mr, ratio_red[q]);
    large |= mass_red[0][q] != 0.0;
  }
  if (tid == 0) a.ratio[((int64_t)round * a.K + k) * (a.nb / 2) + pair] = (float)mr;
  if (mr < a.tol || (!large && negligible(sh.raw.h0, mass_red))) return;
  int row[8];
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) row[kk] = rows[4 * kk + (l >> 4)];
  RotTile x;
  if (w < rot.nx + (a.n1 + 31) / 32) rot_load(rot, w, row, x);
  jacobi32<PT, false>(sh.jac, PR, kInnerSweeps, 0.0, nullptr);
  rotate_rows(rot, sh.jac.V, rows, row, x);
}

__global__ void svt_conv_kernel(const float* __restrict__ ratio, int64_t K, int64_t k0, int64_t k1, int nrounds,
                                int npairs, double tol, int* conv) {
  const int64_t k = k0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= k1) return;
  if (conv[k]) return;
  float m = 0.f;
  for (int r = 0; r < nrounds; ++r)
#pragma unroll 8
    for (int p = 0; p < npairs; ++p) m = fmaxf(m, ratio[((int64_t)r * K + k) * npairs + p]);
  if (m < tol) conv[k] = 1;
}

// Number of slices whose sweeps ended without meeting the convergence test
// (conv[k] == 0), one workgroup, integer sums in a fixed order.
__global__ __launch_bounds__(256) void count_unconverged_kernel(const int* __restrict__ conv, int64_t K,
                                                                int32_t* __restrict__ out) {
  __shared__ int64_t red[256];
  int64_t c = 0;
  for (int64_t k = threadIdx.x; k < K; k += 256) c += conv[k] ? 0 : 1;
  red[threadIdx.x] = c;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = (int32_t)(red[0] < 0x7fffffff ? red[0] : 0x7fffffff);
}

__global__ void identity_kernel(float* re, float* im, int64_t K, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= K * n * n) return;
  const int64_t r = e % (n * n);
  re[e] = (r / n == r % n) ? 1.f : 0.f;
  im[e] = 0.f;
}

__global__ void zero_f32_kernel(float* p, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) p[e] = 0.f;
}

__global__ void zero_int_kernel(int* p, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) p[e] = 0;
}

// Row norms of X, shrink factors d_i = max(1 - tau / sigma_i, 0), X <- D X,
// and the number of sigma_i > tau per slice. Row norms at or below
// max(n1, n2) eps_32 sigma_max are rounding residue of rows that the
// rotations have emptied (a slice has at most min(n1, n2) nonzero singular
// values) and count as zero. Three passes over all slices at once: a
// wavefront per row sums it with consecutive lanes on consecutive columns;
// one workgroup per slice turns the norms into factors (sig, K x n1, holds
// the norms and then the factors); the scaling runs over every element.
__global__ __launch_bounds__(NT) void svt_rownorm_kernel(const float* __restrict__ xre, const float* __restrict__ xim,
                                                         int64_t K, int64_t n1, int64_t n2, int real_last,
                                                         double* __restrict__ sig) {
  const int64_t row = (int64_t)blockIdx.x * (NT / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= K * n1) return;
  const int64_t k = row / n1;
  const bool real = k == 0 || (real_last && k == K - 1);
  const float* re = xre + row * n2;
  const float* im = xim + row * n2;
  double s2 = 0.0;
  for (int64_t j = lane; j < n2; j += 64) {
    const double a = re[j], b = real ? 0.0 : im[j];
    s2 += a * a + b * b;
  }
  s2 = wave_sum(s2);
  if (lane == 0) sig[row] = sqrt(s2);
}

__global__ __launch_bounds__(NT) void svt_factor_kernel(int64_t n1, int64_t n2, double tau, double* sig,
                                                        int32_t* ranks) {
  __shared__ double red[NT];
  __shared__ int cnt[NT];
  const int64_t k = blockIdx.x;
  const int tid = threadIdx.x;
  double* sg = sig + k * n1;
  double mx = 0.0;
  for (int64_t i = tid; i < n1; i += NT) mx = fmax(mx, sg[i]);
  red[tid] = mx;
  __syncthreads();
  for (int w = NT / 2; w > 0; w >>= 1) {
    if (tid < w) red[tid] = fmax(red[tid], red[tid + w]);
    __syncthreads();
  }
  const double floor_ = (double)(n1 > n2 ? n1 : n2) * 1.1920928955078125e-07 * red[0];
  int mine = 0;
  for (int64_t i = tid; i < n1; i += NT) {
    const double sgi = sg[i];
    const bool kept = sgi > tau && sgi > floor_;
    if (kept) ++mine;
    sg[i] = kept ? 1.0 - tau / sgi : 0.0;
  }
  cnt[tid] = mine;
  __syncthreads();
  for (int w = NT / 2; w > 0; w >>= 1) {
    if (tid < w) cnt[tid] += cnt[tid + w];
    __syncthreads();
  }
  if (tid == 0 && ranks) ranks[k] = cnt[0];
}

__global__ void svt_scale_kernel(float* __restrict__ xre, float* __restrict__ xim, int64_t K, int64_t n1, int64_t n2,
                                 int real_last, const double* __restrict__ sig) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= K * n1 * n2) return;
  const int64_t row = e / n2, k = row / n1;
  const bool real = k == 0 || (real_last && k == K - 1);
  const double d = sig[row];
  xre[e] = (float)(d * xre[e]);
  if (!real) xim[e] = (float)(d * xim[e]);
}

// Leading singular (or eigen) vectors after the block Jacobi has made the m
// rows of X (row length ldx) orthogonal, X = Q Y with Q unitary. Row i of X
// is mu_i times a unit row and so mu_i = ||X_i||. Two uses:
//  * Y = G, a Hermitian positive semidefinite Gram matrix: q_i (row i of Q)
//    is a conjugated eigenvector and mu_i its eigenvalue, sigma = sqrt(mu);
//  * Y = a Fourier slice itself (m <= its row length): mu_i = sigma_i, rows
//    of Q are the conjugated left singular vectors and rows of X are sigma_i
//    times the conjugated right ones.
// For the r largest mu (descending, ties by index) column t of out (len x r
// planes per slice) is conj(row sel(t) of the source S (row length len))
// times 1, 1 / sqrt(mu) (mode 1) or 1 / mu (mode 2), and sv[k][t] =
// sqrt(mu) (sqrt_sv) or mu. One workgroup per slice. A mu at or below
// floor_rel times the slice's largest mu is rounding residue of a row the
// rotations have emptied (or of an eigenvalue that is zero): it is reported
// as 0 and its column is zero in every mode, so a rank-deficient slice gives
// the same zero columns whichever route produced X.
__global__ __launch_bounds__(NT) void tsvd_pick_kernel(const float* __restrict__ xre, const float* __restrict__ xim,
                                                       int64_t ldx, const float* __restrict__ sre,
                                                       const float* __restrict__ sim, int64_t len, int64_t K, int m,
                                                       int r, int real_last, int mode, int sqrt_sv, double floor_rel,
                                                       float* __restrict__ ore, float* __restrict__ oim,
                                                       double* __restrict__ sv) {
  __shared__ double red[NT];
  extern __shared__ double lam[];  // m row norms, then r selected rows (int)
  int* sel = reinterpret_cast<int*>(lam + m);
  const int64_t k = blockIdx.x;
  const bool real = k == 0 || (real_last && k == K - 1);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const float* xr = xre + k * m * ldx;
  const float* xi = xim + k * m * ldx;
  for (int i = wv; i < m; i += NT / 64) {
    double s2 = 0.0;
    for (int64_t j = lane; j < ldx; j += 64) {
      const double a = xr[(int64_t)i * ldx + j], b = real ? 0.0 : xi[(int64_t)i * ldx + j];
      s2 += a * a + b * b;
    }
    s2 = wave_sum(s2);
    if (lane == 0) lam[i] = sqrt(s2);
  }
  // every rank below r is taken exactly once for finite norms; the default
  // keeps a non-finite input in bounds
  for (int t = tid; t < r; t += NT) sel[t] = 0;
  __syncthreads();
  for (int i = tid; i < m; i += NT) {
    const double li = lam[i];
    int rank = 0;
    for (int j = 0; j < m; ++j) {
      const double lj = lam[j];
      rank += (lj > li || (lj == li && j < i)) ? 1 : 0;
    }
    if (rank < r) sel[rank] = i;
  }
  double mx = 0.0;
  for (int i = tid; i < m; i += NT) mx = fmax(mx, lam[i]);
  red[tid] = mx;
  __syncthreads();
  for (int w = NT / 2; w > 0; w >>= 1) {
    if (tid < w) red[tid] = fmax(red[tid], red[tid + w]);
    __syncthreads();
  }
  const double floor_ = floor_rel * red[0];
  const float* s_r = sre + k * m * len;
  const float* s_i = sim + k * m * len;
  float* o_r = ore + k * len * r;
  float* o_i = oim + k * len * r;
  for (int64_t e = tid; e < len * r; e += NT) {
    const int64_t j = e / r;
    const int t = (int)(e - j * r);
    const int row = sel[t];
    const double l = lam[row];
    const double sc = !(l > floor_) ? 0.0 : (mode == 0 ? 1.0 : (mode == 1 ? 1.0 / sqrt(l) : 1.0 / l));
    o_r[e] = (float)(sc * s_r[(int64_t)row * len + j]);
    o_i[e] = real ? 0.f : (float)(-sc * s_i[(int64_t)row * len + j]);
  }
  if (sv)
    for (int t = tid; t < r; t += NT) {
      const double l = lam[sel[t]];
      sv[k * r + t] = !(l > floor_) ? 0.0 : (sqrt_sv ? sqrt(l) : l);
    }
}

// t-transpose (Section 2.1): out (n2 x n1 x n3) with out[j][i][t] =
// in[i][j][(n3 - t) mod n3], i.e. every frontal slice transposed and slices
// 2..n3 in reverse order; its Fourier slices are the conjugate transposes
// of those of in.
template <typename T>
__global__ void ttranspose_kernel(const T* __restrict__ in, int64_t n1, int64_t n2, int64_t n3, T* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n1 * n2 * n3) return;
  const int64_t tube = e / n3, t = e - tube * n3;
  const int64_t j = tube / n1, i = tube - j * n1;
  const int64_t ts = t == 0 ? 0 : n3 - t;
  out[e] = in[(i * n2 + j) * n3 + ts];
}

// M = X - E - Y / mu (tube-major, elementwise)
__global__ void admm_pre_kernel(const float* __restrict__ x, const float* __restrict__ e,
                                const float* __restrict__ y, float inv_mu, int64_t n, float* __restrict__ m) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) m[i] = x[i] - e[i] - y[i] * inv_mu;
}

// E = P_unobserved(X - L - Y/mu); Y = Y + mu (L + E - X)
__global__ void admm_post_kernel(const float* __restrict__ x, const uint8_t* __restrict__ mask,
                                 const float* __restrict__ l, float mu, float inv_mu, int64_t n,
                                 float* __restrict__ e, float* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float xv = x[i], lv = l[i], yv = y[i];
  const float ev = mask[i] ? 0.f : (xv - lv - yv * inv_mu);
  e[i] = ev;
  y[i] = yv + mu * (lv + ev - xv);
}

// E = shrink(X - L - Y/mu, lam/mu), the prox of (lam/mu) ||.||_1 (robust
// PCA, eq. tlow7); Y = Y + mu (L + E - X)
__global__ void admm_post_soft_kernel(const float* __restrict__ x, const float* __restrict__ l, float mu,
                                      float inv_mu, float thr, int64_t n, float* __restrict__ e,
                                      float* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float xv = x[i], lv = l[i], yv = y[i];
  const float v = xv - lv - yv * inv_mu;
  const float ev = v > thr ? v - thr : (v < -thr ? v + thr : 0.f);
  e[i] = ev;
  y[i] = yv + mu * (lv + ev - xv);
}

// out[k][j][i] = conj(in[k][i][j]): the conjugate transpose of every
// Fourier slice (K x rows x cols planar in, K x cols x rows out). Reads are
// coalesced along j; the writes are strided.
__global__ void spec_conj_transpose_kernel(const float* __restrict__ re, const float* __restrict__ im, int64_t K,
                                           int64_t rows, int64_t cols, float* __restrict__ ore,
                                           float* __restrict__ oim) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t per = rows * cols;
  if (e >= K * per) return;
  const int64_t k = e / per, r = e - k * per, i = r / cols, j = r - i * cols;
  const int64_t o = k * per + j * rows + i;
  ore[o] = re[e];
  oim[o] = -im[e];
}

// The three quantities of Algorithm 7's convergence check for one
// iteration, reduced per workgroup: max |L - Lprev|, max |E - Eprev| and
// max |L + E - X| over the workgroup's elements (E the new iterate, read
// after the E-update; eprev a copy taken before it). One value triple per
// workgroup in part[3 * block + q]; the maxima are order independent.
__global__ __launch_bounds__(256) void admm_stop_partial_kernel(const float* __restrict__ x,
                                                                const float* __restrict__ l,
                                                                const float* __restrict__ lprev,
                                                                const float* __restrict__ e,
                                                                const float* __restrict__ eprev, int64_t n,
                                                                float* __restrict__ part) {
  __shared__ float red[3][256];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  float dl = 0.f, de = 0.f, rs = 0.f;
  if (i < n) {
    const float lv = l[i], ev = e[i];
    dl = fabsf(lv - lprev[i]);
    de = fabsf(ev - eprev[i]);
    rs = fabsf(lv + ev - x[i]);
  }
  red[0][threadIdx.x] = dl;
  red[1][threadIdx.x] = de;
  red[2][threadIdx.x] = rs;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
#pragma unroll
      for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = fmaxf(red[q][threadIdx.x], red[q][threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x < 3) part[3 * (int64_t)blockIdx.x + threadIdx.x] = red[threadIdx.x][0];
}

// out[q] = max over the nb partial triples (one workgroup)
__global__ __launch_bounds__(256) void admm_stop_reduce_kernel(const float* __restrict__ part, int64_t nb,
                                                               float* __restrict__ out) {
  __shared__ float red[3][256];
  float m[3] = {0.f, 0.f, 0.f};
  for (int64_t b = threadIdx.x; b < nb; b += 256)
#pragma unroll
    for (int q = 0; q < 3; ++q) m[q] = fmaxf(m[q], part[3 * b + q]);
#pragma unroll
  for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = m[q];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
#pragma unroll
      for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = fmaxf(red[q][threadIdx.x], red[q][threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x < 3) out[threadIdx.x] = red[threadIdx.x][0];
}

// out[a][b][t] = in[ra][cb][t] with ra = ridx ? ridx[a] : a and
// cb = cidx ? cidx[b] : b: picked lateral or horizontal slices of a
// tube-major tensor with in_cols lateral slices. Entries past the live pick
// count (*count, for the listed index) are written as zeros; a negative
// count (rejected weights) leaves every entry zero.
template <typename T>
__global__ void gather_slices_kernel(const T* __restrict__ in, int64_t in_cols, int64_t n3,
                                     const int32_t* __restrict__ ridx, const int32_t* __restrict__ cidx,
                                     const int64_t* __restrict__ count, int64_t rows, int64_t cols,
                                     T* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * cols * n3) return;
  const int64_t tube = i / n3, t = i - tube * n3;
  const int64_t a = tube / cols, b = tube - a * cols;
  const int64_t lim = count ? *count : INT64_MAX;
  if ((ridx && a >= lim) || (cidx && b >= lim)) {
    out[i] = T(0);
    return;
  }
  const int64_t ra = ridx ? (int64_t)ridx[a] : a;
  const int64_t cb = cidx ? (int64_t)cidx[b] : b;
  out[i] = in[(ra * in_cols + cb) * n3 + t];
}

unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

// The Jacobi sweeps use at most two streams: the caller's and the side
// stream (three or four streams measured slower than two).
constexpr int kSvtStreams = 2;

}  // namespace

size_t svt_ratio_count(int64_t K, int64_t n1) {
  const int nb = svt_blocks(n1);
  return size_t(nb - 1) * K * (nb / 2);
}

int svt_blocks(int64_t n1) {
  int nb = (int)((n1 + RB - 1) / RB);
  if (nb < 2) nb = 2;
  if (nb % 2) ++nb;
  return nb;
}

int zero_f32(float* p, int64_t n, hipStream_t st) {
  if (n == 0) return TP_OK;
  hipLaunchKernelGGL(zero_f32_kernel, dim3(nblk(n)), dim3(256), 0, st, p, n);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int svt_identity(float* ure, float* uim, int64_t K, int64_t n, hipStream_t st) {
  if (K * n * n == 0) return TP_OK;
  hipLaunchKernelGGL(identity_kernel, dim3(nblk(K * n * n)), dim3(256), 0, st, ure, uim, K, n);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int svt_count_unconverged(const int* conv, int64_t K, int32_t* out, hipStream_t st) {
  if (!out) return TP_OK;
  hipLaunchKernelGGL(count_unconverged_kernel, dim3(1), dim3(256), 0, st, conv, K, out);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int svt_jacobi(float* xre, float* xim, float* ure, float* uim, int64_t K, int64_t n1, int64_t n2, bool real_last,
               int max_sweeps, double tol, float* ratio, int* conv, hipStream_t st) {
  const int nb = svt_blocks(n1);
  hipLaunchKernelGGL(zero_int_kernel, dim3(nblk(K)), dim3(256), 0, st, conv, K);
  TP_LAUNCH_CHECK();
  PairArgs a{K, n1, n2, 0, xre, xim, ure, uim, nb, real_last ? 1 : 0, ratio, conv, tol};
  // slices [k0, k1) on stream s
  auto sweeps = [&](int64_t k0, int64_t k1, hipStream_t s) -> int {
    PairArgs g = a;
    for (int sweep = 0; sweep < max_sweeps; ++sweep) {
      for (int round = 0; round < nb - 1; ++round) {
        // the slices sit on a grid dimension of at most 65,535 values: longer
        // spectra take several launches per round
        for (int64_t c0 = k0; c0 < k1; c0 += 65535) {
          g.k0 = c0;
          const int64_t kc = k1 - c0 < 65535 ? k1 - c0 : 65535;
          hipLaunchKernelGGL(svt_pair_kernel, dim3(nb / 2, (unsigned)kc), dim3(PT), 0, s, g, round);
          TP_LAUNCH_CHECK();
        }
      }
      hipLaunchKernelGGL(svt_conv_kernel, dim3(nblk(k1 - k0)), dim3(256), 0, s, ratio, K, k0, k1, nb - 1, nb / 2,
                         tol, conv);
      TP_LAUNCH_CHECK();
    }
    return TP_OK;
  };
  // The slices are independent: when one launch would leave compute units
  // with a free pair-step slot (two fit per compute unit by registers) but has
  // more workgroups than compute units, the second half of the slices runs on
  // the side stream, so that one half's pair steps fill the units that the
  // other half's launch leaves idle. Six completion iterations on one / two
  // streams: 26 slices of 256 x 256 (208 pair steps per launch on 256 units)
  // 19.6 / 24.0 ms, 33 (264) 32.0 / 27.2, 51 (408) 35.6 / 32.3; 85 of 192 x 1140
  // (510, every slot taken) 60.1 / 62.2.
  int dev = 0, cus = 0;
  TP_HIP_CHECK(hipGetDevice(&dev));
  TP_HIP_CHECK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const int64_t w = K * (nb / 2);
  if (K < kSvtStreams || w <= cus || 8 * w > 7 * 2 * (int64_t)cus) return sweeps(0, K, st);
  SideStream* ss = nullptr;
  if (int rc = side_stream(&ss)) return rc;
  std::lock_guard<std::mutex> lk(ss->mu);
  const int64_t kh = K / 2;
  TP_HIP_CHECK(hipEventRecord(ss->fork, st));
  TP_HIP_CHECK(hipStreamWaitEvent(ss->s, ss->fork, 0));
  if (int rc = sweeps(kh, K, ss->s)) return rc;
  TP_HIP_CHECK(hipEventRecord(ss->join, ss->s));
  if (int rc = sweeps(0, kh, st)) return rc;
  TP_HIP_CHECK(hipStreamWaitEvent(st, ss->join, 0));
  return TP_OK;
}

int svt_shrink(float* xre, float* xim, int64_t K, int64_t n1, int64_t n2, double tau, bool real_last,
               double* sig, int32_t* ranks, hipStream_t st) {
  if (K * n1 == 0) return TP_OK;
  const int rl = real_last ? 1 : 0;
  const int64_t rows = K * n1;
  hipLaunchKernelGGL(svt_rownorm_kernel, dim3((unsigned)((rows + NT / 64 - 1) / (NT / 64))), dim3(NT), 0, st, xre,
                     xim, K, n1, n2, rl, sig);
  hipLaunchKernelGGL(svt_factor_kernel, dim3((unsigned)K), dim3(NT), 0, st, n1, n2, tau, sig, ranks);
  hipLaunchKernelGGL(svt_scale_kernel, dim3(nblk(K * n1 * n2)), dim3(256), 0, st, xre, xim, K, n1, n2, rl, sig);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int tsvd_pick(const float* xre, const float* xim, int64_t ldx, const float* sre, const float* sim, int64_t len,
              int64_t K, int64_t m, int64_t r, bool real_last, int mode, bool sqrt_sv, double floor_rel, float* ore,
              float* oim, double* sv, hipStream_t st) {
  if (K == 0 || r == 0) return TP_OK;
  if (m > kPickMax || r > m) return fail(TP_EUNSUPPORTED, "vector selection needs r <= m <= 4096");
  const size_t lds = size_t(m) * sizeof(double) + size_t(r) * sizeof(int);
  hipLaunchKernelGGL(tsvd_pick_kernel, dim3((unsigned)K), dim3(NT), lds, st, xre, xim, ldx, sre, sim, len, K, (int)m,
                     (int)r, real_last ? 1 : 0, mode, sqrt_sv ? 1 : 0, floor_rel, ore, oim, sv);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int admm_pre(const float* x, const float* e, const float* y, float inv_mu, int64_t n, float* m, hipStream_t st) {
  if (n == 0) return TP_OK;
  hipLaunchKernelGGL(admm_pre_kernel, dim3(nblk(n)), dim3(256), 0, st, x, e, y, inv_mu, n, m);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int admm_post(const float* x, const uint8_t* mask, const float* l, float mu, float inv_mu, int64_t n, float* e,
              float* y, hipStream_t st) {
  if (n == 0) return TP_OK;
  hipLaunchKernelGGL(admm_post_kernel, dim3(nblk(n)), dim3(256), 0, st, x, mask, l, mu, inv_mu, n, e, y);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int spec_conj_transpose(const float* re, const float* im, int64_t K, int64_t rows, int64_t cols, float* ore,
                        float* oim, hipStream_t st) {
  const int64_t n = K * rows * cols;
  if (n == 0) return TP_OK;
  hipLaunchKernelGGL(spec_conj_transpose_kernel, dim3(nblk(n)), dim3(256), 0, st, re, im, K, rows, cols, ore, oim);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

size_t admm_stop_floats(int64_t n) { return 3 * size_t(nblk(n)) + 4; }

int admm_stop(const float* x, const float* l, const float* lprev, const float* e, const float* eprev, int64_t n,
              float* part, float* out, hipStream_t st) {
  if (n == 0) return TP_OK;
  const unsigned nb = nblk(n);
  hipLaunchKernelGGL(admm_stop_partial_kernel, dim3(nb), dim3(256), 0, st, x, l, lprev, e, eprev, n, part);
  TP_LAUNCH_CHECK();
  hipLaunchKernelGGL(admm_stop_reduce_kernel, dim3(1), dim3(256), 0, st, part, (int64_t)nb, out);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int admm_post_soft(const float* x, const float* l, float mu, float inv_mu, float thr, int64_t n, float* e, float* y,
                   hipStream_t st) {
  if (n == 0) return TP_OK;
  hipLaunchKernelGGL(admm_post_soft_kernel, dim3(nblk(n)), dim3(256), 0, st, x, l, mu, inv_mu, thr, n, e, y);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int ttranspose(const void* in, int elem_bytes, int64_t n1, int64_t n2, int64_t n3, void* out, hipStream_t st) {
  const int64_t n = n1 * n2 * n3;
  if (n == 0) return TP_OK;
  if (elem_bytes == 4)
    hipLaunchKernelGGL(ttranspose_kernel<float>, dim3(nblk(n)), dim3(256), 0, st, (const float*)in, n1, n2, n3,
                       (float*)out);
  else if (elem_bytes == 1)
    hipLaunchKernelGGL(ttranspose_kernel<uint8_t>, dim3(nblk(n)), dim3(256), 0, st, (const uint8_t*)in, n1, n2, n3,
                       (uint8_t*)out);
  else
    return fail(TP_EUNSUPPORTED, "t-transpose supports 1- and 4-byte elements");
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int gather_slices(const void* in, int elem_bytes, int64_t in_cols, int64_t n3, const int32_t* ridx,
                  const int32_t* cidx, const int64_t* count, int64_t rows, int64_t cols, void* out, hipStream_t st) {
  const int64_t n = rows * cols * n3;
  if (n == 0) return TP_OK;
  if (elem_bytes == 4)
    hipLaunchKernelGGL(gather_slices_kernel<float>, dim3(nblk(n)), dim3(256), 0, st, (const float*)in, in_cols, n3,
                       ridx, cidx, count, rows, cols, (float*)out);
  else if (elem_bytes == 1)
    hipLaunchKernelGGL(gather_slices_kernel<uint8_t>, dim3(nblk(n)), dim3(256), 0, st, (const uint8_t*)in, in_cols,
                       n3, ridx, cidx, count, rows, cols, (uint8_t*)out);
  else
    return fail(TP_EUNSUPPORTED, "slice gather supports 1- and 4-byte elements");
  TP_LAUNCH_CHECK();
  return TP_OK;
}

}  // namespace tp
