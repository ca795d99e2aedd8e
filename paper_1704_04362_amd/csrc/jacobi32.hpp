// Hermitian Jacobi eigensolver for matrices of at most 32 x 32 (float64) on
// eight wavefronts. The rotations, their order and their arithmetic are those
// of jacobi.hpp (the round-robin tournament, smaller-root rotations); the
// layout is for short rounds. A round is bound by the issue of float64
// instructions (one in 8 cycles per SIMD) and its serial chain (LDS read, the
// rotation's roots and division, the update, LDS write, barrier):
//
// * Four wavefronts hold H: thread (u, v) updates the 2 x 2 block at the rows of
//   pair u and the columns of pair v. H lives in LDS twice and a round reads
//   one copy and writes the other, so a round has one barrier.
// * Every lane of these computes the rotation of its own column pair. The lanes
//   of a row of 16 take the column pairs from the row's own row pair on, so
//   the row pair's rotation is that of the row's first lane, one broadcast
//   within the row (DPP): rotations are not exchanged through LDS.
// * Four further wavefronts apply the rotations to V one round later, while the
//   first four are in the next round; a wavefront owns eight rows of V.
// * Complex entries are one 16-byte word, and the 16 lanes of a row of threads
//   touch 16 neighbouring ones.
#pragma once

#include <hip/hip_runtime.h>

namespace tp {

struct alignas(16) Cz {
  double x, y;
};

struct Jacobi32Shared {
  Cz H[2][32 * 32];  // row-major, row stride 32
  Cz V[32 * 32];
  Cz rot[2][16][2];  // (c, s), e of the pairs of a round and the one before
};

// Rotation of a pair p < q: rows (x, y) become (c x - s e y, s x + c e y),
// columns the same with conj(e)
struct Rot32 {
  double c, s, er, ei;
};

// 1 / sqrt(x), sqrt(x) and y / x from the hardware estimates (about 2^-24), for
// values whose squares neither overflow nor underflow. Zeros, infinities and NaN
// give NaN or infinity, which the caller's test rules out.
// 1 / sqrt: one step of third order, y (1 + e / 2 + 3 e^2 / 8) with e = 1 - x y^2.
// sqrt: a step of Goldschmidt's iteration on g ~ sqrt(x) and h ~ 1 / (2 sqrt(x)),
// then g + h (x - g^2), Newton's step in g, twice.
// Quotient: two Newton steps r + r (1 - x r) of the reciprocal, and the product
// y r corrected once by its residual.
__device__ __forceinline__ double j32_rsqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(y * -x, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ double j32_sqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double e = fma(-h, g, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  g = fma(fma(-g, g, x), h, g);
  return fma(fma(-g, g, x), h, g);
}
__device__ __forceinline__ double j32_div(double y, double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  r = fma(r, fma(-x, r, 1.0), r);
  const double q = y * r;
  return fma(fma(-x, q, y), r, q);
}

__device__ __forceinline__ Rot32 j32_rotation(double hpp, double hqq, Cz h) {
  const double h2 = fma(h.x, h.x, h.y * h.y), d = hqq - hpp;
  const double ih = j32_rsqrt(h2);
  const double root = j32_sqrt(fma(4.0, h2, d * d));
  const double habs = h2 * ih;
  const double t = j32_div((d >= 0.0 ? 2.0 : -2.0) * habs, fabs(d) + root);
  const double ct = j32_rsqrt(fma(t, t, 1.0));
  // rotate only entries that are not negligible (also rules out the
  // infinities of an underflowed h2)
  const bool on = h2 > 1e-300 && habs > 1e-18 * (fabs(hpp) + fabs(hqq));
  return Rot32{on ? ct : 1.0, on ? t * ct : 0.0, on ? h.x * ih : 1.0, on ? h.y * ih : 0.0};
}

// (the fused multiply-adds are written out, so that every use rounds alike)
__device__ __forceinline__ void j32_mix(const Rot32& r, double eyr, double eyi, Cz& x, Cz& y) {
  const Cz nx{fma(r.c, x.x, -(r.s * eyr)), fma(r.c, x.y, -(r.s * eyi))};
  y = Cz{fma(r.s, x.x, r.c * eyr), fma(r.s, x.y, r.c * eyi)};
  x = nx;
}
__device__ __forceinline__ void j32_rows(const Rot32& r, Cz& x, Cz& y) {
  j32_mix(r, fma(r.er, y.x, -(r.ei * y.y)), fma(r.ei, y.x, r.er * y.y), x, y);
}
__device__ __forceinline__ void j32_cols(const Rot32& r, Cz& x, Cz& y) {
  j32_mix(r, fma(r.er, y.x, r.ei * y.y), fma(r.er, y.y, -(r.ei * y.x)), x, y);
}

// the value of the first lane of the row of 16
__device__ __forceinline__ double j32_first(double v) {
  union {
    double d;
    int i[2];
  } a;
  a.d = v;
#pragma unroll
  for (int q = 0; q < 2; ++q) a.i[q] = __builtin_amdgcn_update_dpp(0, a.i[q], 0x150, 0xf, 0xf, false);
  return a.d;
}

// Diagonalises the n x n Hermitian matrix in sh.H[0] (n <= 32, both triangles
// filled; an odd n uses row and column n as an idle index) into sh.H[returned],
// the unitary into sh.V. Makes at most max_sweeps sweeps, stopping before one
// when the off-diagonal mass is below rel_tol^2 of the total (CHECK; red: 16
// doubles of LDS). Called by all NT >= 512 threads of the workgroup; starts
// and ends with a barrier.
template <int NT, bool CHECK>
__device__ int jacobi32(Jacobi32Shared& sh, int n, int max_sweeps, double rel_tol, double* red) {
  static_assert(NT >= 512, "eight wavefronts");
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = n + (n & 1), np = m >> 1;
  const bool hwork = w < 4, vwork = w >= 4 && w < 8;
  const int u = (4 * w + (lane >> 4)) & 15, v = hwork ? (lane + u) & 15 : lane & 15;
  __syncthreads();
  if ((n & 1) && tid <= n) {
    sh.H[0][tid * 32 + n] = Cz{0.0, 0.0};
    sh.H[0][n * 32 + tid] = Cz{0.0, 0.0};
  }
  for (int e = tid; e < 32 * 32; e += NT) sh.V[e] = Cz{(e >> 5) == (e & 31) ? 1.0 : 0.0, 0.0};
  __syncthreads();
  int cur = 0;
  // slot 0 of round rho holds (m - 1, rho), slot t ((rho + t), (rho - t)) mod m - 1
  const int a0 = v == 0 ? m - 1 : (v < np ? v : 1), b0 = v == 0 ? 0 : (v < np ? m - 1 - v : 0);
  const int c0 = u == 0 ? m - 1 : (u < np ? u : 1), d0 = u == 0 ? 0 : (u < np ? m - 1 - u : 0);
  const bool block = u < np && v < np;
  Cz* V0 = sh.V + 32 * (8 * (w & 3) + (lane >> 4));
  Cz* V1 = V0 + 32 * 4;
  auto step = [m](int x) { return x + 1 >= m - 1 ? x + 2 - m : x + 1; };
  for (int sweep = 0; sweep < max_sweeps; ++sweep) {
    if constexpr (CHECK) {
      double off = 0.0, tot = 0.0;
      if (w < 8) {
        for (int e = tid; e < n * 32; e += 512) {
          const int i = e >> 5, j = e & 31;
          const Cz z = sh.H[cur][e];
          const double q = j < n ? fma(z.x, z.x, z.y * z.y) : 0.0;
          tot += q;
          if (i != j) off += q;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          off += __shfl_xor(off, o);
          tot += __shfl_xor(tot, o);
        }
        if (lane == 0) {
          red[w] = off;
          red[8 + w] = tot;
        }
      }
      __syncthreads();
      double o = 0.0, t = 0.0;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        o += red[q];
        t += red[8 + q];
      }
      if (o <= rel_tol * rel_tol * t || t == 0.0) break;
    }
    int a = a0, b = b0, c = c0, d = d0;
    // round rho of H beside round rho - 1 of V
    for (int rho = 0; rho < m; ++rho) {
      if (hwork && rho < m - 1) {
        const int p = min(a, b), q = max(a, b), pu = 32 * min(c, d), qu = 32 * max(c, d);
        const Cz* H = sh.H[cur];
        const double hpp = H[p * 33].x, hqq = H[q * 33].x;
        const Cz hpq = H[p * 32 + q];
        Cz x00 = H[pu + p], x01 = H[pu + q], x10 = H[qu + p], x11 = H[qu + q];
        const Rot32 rv = j32_rotation(hpp, hqq, hpq);
        if (tid < 16) {
          sh.rot[rho & 1][v][0] = Cz{rv.c, rv.s};
          sh.rot[rho & 1][v][1] = Cz{rv.er, rv.ei};
        }
        const Rot32 ru{j32_first(rv.c), j32_first(rv.s), j32_first(rv.er), j32_first(rv.ei)};
        j32_rows(ru, x00, x10);
        j32_rows(ru, x01, x11);
        j32_cols(rv, x00, x01);
        j32_cols(rv, x10, x11);
        if (block) {
          Cz* O = sh.H[cur ^ 1];
          O[pu + p] = x00;
          O[pu + q] = x01;
          O[qu + p] = x10;
          O[qu + q] = x11;
        }
        if (v != 0) a = step(a);
        b = step(b);
        if (u != 0) c = step(c);
        d = step(d);
      }
      if (vwork && rho > 0) {
        const int p = min(a, b), q = max(a, b);
        const Cz cs = sh.rot[(rho & 1) ^ 1][v][0], e = sh.rot[(rho & 1) ^ 1][v][1];
        Cz y0 = V0[p], z0 = V0[q], y1 = V1[p], z1 = V1[q];
        const Rot32 rv{cs.x, cs.y, e.x, e.y};
        j32_cols(rv, y0, z0);
        j32_cols(rv, y1, z1);
        if (v < np) {
          V0[p] = y0;
          V0[q] = z0;
          V1[p] = y1;
          V1[q] = z1;
        }
        if (v != 0) a = step(a);
        b = step(b);
      }
      if (rho < m - 1) cur ^= 1;
      __syncthreads();
    }
  }
  return cur;
}

}  // namespace tp
