// Tubes beyond the LDS transforms: a four-step transform through HBM, with the
// caller's output as the only intermediate storage. The real tube x of even
// length n is packed as z[m] = x[2m] + i x[2m+1], m < N = n/2, and with
// N = N1 N2, m = j1 + N1 j2, k = k2 + N2 k1 its DFT factors as
//   Z[k2 + N2 k1] = sum_j1 W_N1^{j1 k1} W_N^{j1 k2} sum_j2 z[j1 + N1 j2] W_N2^{j2 k2}
// (W_L = exp(-2 pi i / L)). Forward:
//   tube pass: per block of tubes and of j1 the inner length-N2 transforms over
//     j2 and the twiddle W_N^{j1 k2}, written to spectrum slice k2 + N2 j1 of
//     that tube's slot;
//   slice pass: per block of slots and pair {k2, N2 - k2} the outer length-N1
//     transforms over j1 (the partner Z[N - k] of every Z[k] of the pair is
//     in the pair), then X[k] = E[k] + W_n^k O[k] and X[N-k] = conj(E[k] -
//     W_n^k O[k]), E[k] = (Z[k] + conj Z[N-k]) / 2, O[k] = (Z[k] - conj Z[N-k]) / 2i,
//     written to slices k and N - k: exactly the slices the pair's intermediate
//     values occupy (and N for k = 0), so each workgroup overwrites only what
//     it has read.
// Inverse (the steps reversed, conjugated, into the output tensor):
//   slice pass: per block of slots and pair {k2, N2 - k2}, Z[k] = E[k] + i O[k]
//     from the half spectrum (E = (X[k] + conj X[N-k]) / 2, O = (X[k] -
//     conj X[N-k]) W_n^-k / 2), the inverse transform over k1 and the twiddle
//     W_N^{-j1 k2}, written into the tube at packed position j1 + N1 k2;
//   tube pass: per block of tubes and of j1 the inverse transform over k2, 1/N,
//     and the real and imaginary parts as x[2m], x[2m+1] at the positions it
//     read.
// Both short transforms run in LDS in the stages of fft_stages.hpp. Twiddles
// W_N^{j1 k2} come from two short tables per factor that is fixed in a
// workgroup (the root of a sum of exponents as a product of two), and so does
// W_n^k over k1. Float tubes have float butterflies (every root rounded once
// from float64) and float64 twiddles and separations.
//
// A pass moves the tensor once each way (450 us at 576 tubes x 500,000 float32
// and the 5.1 TB/s of a large copy). Bound: the stages between, at ~45 % of the
// vector issue slots, behind barriers. So 128 KB tiles (runs of 32 to 64 bytes
// on either side; half of it and two workgroups a CU measured the same, with
// padded rows 1.5x slower), one persistent workgroup a CU that loads the next
// tile while the stages of this one run (forward 1.97 -> 1.79 ms, inverse 1.79
// -> 1.70), tables of all roots, built once. 576 x 500,000: forward 5.05 ->
// 1.78 ms, inverse 5.11 -> 1.69; 3e7 float32 values as tubes of 10,000: 1589 /
// 2561 -> 187 / 187 us, of 65,536: 722 / 877 -> 168 / 151; float64 6043 / 10899
// -> 362 / 351 and 1843 / 2964 -> 309 / 283 (replaced: radices up to 13, 64 KB of
// split re / im tiles with integer divisions and a sincospi per butterfly
// input).
#include "fft_stages.hpp"
#include "fft_tubes.hpp"

#include <algorithm>

namespace tp {
namespace {

using lfft::Cx;

constexpr int kMaxN2 = 256, kMaxN1 = 1024, kLogNT = 10, kNT = 1 << kLogNT;
constexpr int kMaxLV = 4;  // at most 16 values of j1 a workgroup

// Rows of its sequence that a thread of a pass holds: 2^17 bytes of sequences a workgroup
template <typename T>
constexpr int kRows = 128 / (2 * sizeof(T));

// Float passes load the next tile while the stages of this one run; double ones,
// whose butterflies take the registers, load where the values are needed.
template <typename T>
constexpr bool kAhead = sizeof(T) == 4;

// the value, hidden from loop-invariant code motion: the addresses of a tile's
// rows are formed where they are used instead of held in registers
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

struct FourPlan {
  int N1, N2;
  // tube pass: 2^lu slots x 2^lv values of j1 a workgroup, slice pass: 2^ls slots x the pair
  int lu, lv, ls;
  int ldt, lds;  // elements between LDS rows
  lfft::Plan p1, p2;  // of lengths N1 and N2
};

// Taylor coefficients of cos y and sin(y) / y in y^2
__constant__ const double kCos[9] = {1.0, -1.0 / 2, 1.0 / 24, -1.0 / 720, 1.0 / 40320, -1.0 / 3628800, 1.0 / 479001600,
                                     -1.0 / 87178291200, 1.0 / 20922789888000};
__constant__ const double kSin[9] = {1.0, -1.0 / 6, 1.0 / 120, -1.0 / 5040, 1.0 / 362880, -1.0 / 39916800,
                                     1.0 / 6227020800, -1.0 / 1307674368000, 1.0 / 355687428096000};
// exp(-2 pi i b / L), 0 <= b <= L < 2^20: the angle to the nearest quarter turn, exact
// as an integer, |y| <= pi / 4, where the series end below 1e-17. A loop over
// loaded coefficients: a library call inlined in the passes' tile loops has
// its constants hoisted into registers that the prefetched tile needs.
__device__ __forceinline__ Cx<double> turn(int b, int L) {
  const int q = (int)rint(4.0 * (double)b / (double)L);
  const double y = (double)(4 * b - q * L) / (double)L * 1.5707963267948966, y2 = y * y;
  double c = 0.0, s = 0.0;
#pragma unroll 1
  for (int k = 8; k >= 0; --k) {
    c = fma(c, y2, kCos[k]);
    s = fma(s, y2, kSin[k]);
  }
  s *= y;
  const double u = q & 1 ? -s : c, v = q & 1 ? -c : -s;
  return q & 2 ? Cx<double>{-u, -v} : Cx<double>{u, v};
}

// W_L^{o + a b}, 0 <= b < LO HI, as the product of W_L^{a (b mod LO)} (fixed for a
// thread that steps by LO) and W_L^{o + a LO (b / LO)}; LO values, then HI
__device__ __forceinline__ void fill_powers(Cx<double>* w, int LO, int HI, int o, int a, int L, int tid, int nt) {
  for (int e = tid; e < LO + HI; e += nt) {
    const int b = e < LO ? a * e : o + a * LO * (e - LO);
    w[e] = turn(b, L);
  }
}
__device__ __forceinline__ Cx<double> times(Cx<double> a, Cx<double> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}

// dynamic LDS: powers, roots of the stages, sequences, positions
template <typename T>
struct FourLds {
  Cx<double>* pw;
  Cx<T>* tab;
  Cx<T>* buf;
  uint16_t* pos;
  size_t bytes;
  __host__ __device__ FourLds(int npw, int n, int ld, unsigned char* base) {
    size_t o = 0;
    pw = (Cx<double>*)(base + o);
    o += sizeof(Cx<double>) * npw;
    tab = (Cx<T>*)(base + o);
    o += (sizeof(Cx<T>) * n + 15) / 16 * 16;
    buf = (Cx<T>*)(base + o);
    o += (sizeof(Cx<T>) * n * ld + 15) / 16 * 16;
    pos = (uint16_t*)(base + o);
    o += 2 * size_t(n);
    bytes = o;
  }
};
// the powers' sizes: per j1 of a tube pass, of the pair's twiddles (each) and
// separation of a slice pass
__host__ __device__ __forceinline__ int ceil_div(int a, int b) { return (a + b - 1) / b; }
__host__ __device__ __forceinline__ int tube_powers(const FourPlan& f) {
  const int rows = kNT >> (f.lu + f.lv);
  return rows + ceil_div(f.N2, rows) + 1;  // (odd row length: other banks for every j1)
}
__host__ __device__ __forceinline__ int pair_powers(const FourPlan& f) {
  const int rows = kNT >> (f.ls + 1);
  return rows + ceil_div(f.N1, rows);
}
__host__ __device__ __forceinline__ int half_powers(const FourPlan& f) {
  const int rows = kNT >> f.ls;
  return rows + ceil_div(f.N1, rows);
}

// Tiles of the tube passes: 4 x 4 groups of (slot block, j1 block), j1 groups
// fastest, so that reads (contiguous in j1) and writes (contiguous in slots)
// both share lines within a group
struct TubeTiles {
  uint32_t nsb, nj, ngj;
  XcdWalk walk;
  __device__ TubeTiles(int64_t ks, const FourPlan& f)
      : nsb((uint32_t)((ks + (1 << f.lu) - 1) >> f.lu)),
        nj((uint32_t)((f.N1 + (1 << f.lv) - 1) >> f.lv)),
        ngj((nj + 3) / 4),
        walk((int64_t)ngj * ((nsb + 3) / 4) * 16) {}
  __device__ bool next(int64_t& sb, int& jb) {
    int64_t G;
    while (walk.next(G)) {
      const uint32_t g = (uint32_t)(G / 16), w = (uint32_t)G % 16, gs = g / ngj;
      jb = (int)((g - gs * ngj) * 4 + w % 4);
      sb = (int64_t)gs * 4 + w / 4;
      if (jb < (int)nj && sb < (int64_t)nsb) return true;
    }
    return false;
  }
};
// tiles of the slice passes: (pair, slot block), slot blocks fastest
struct SliceTiles {
  uint32_t nsb;
  XcdWalk walk;
  __device__ SliceTiles(int64_t ks, const FourPlan& f)
      : nsb((uint32_t)((ks + (1 << f.ls) - 1) >> f.ls)), walk((int64_t)nsb * (f.N2 / 2 + 1)) {}
  __device__ bool next(int64_t& sb, int& ka) {
    int64_t G;
    if (!walk.next(G)) return false;
    ka = (int)((uint32_t)G / nsb);
    sb = (int64_t)((uint32_t)G - (uint32_t)ka * nsb);
    return true;
  }
};

template <typename T>
struct alignas(sizeof(T)) Two {
  T x, y;
};
template <typename T>
__device__ __forceinline__ Two<T> load_two(const T* p) {
  Two<T> r;
  __builtin_memcpy(&r, p, sizeof(r));
  return r;
}
template <typename T>
__device__ __forceinline__ void store_two(T* p, T x, T y) {
  const Two<T> r{x, y};
  __builtin_memcpy(p, &r, sizeof(r));
}

// forward tube pass
template <typename T>
__global__ __launch_bounds__(kNT, 4) void four_fwd_tube_kernel(const T* __restrict__ x, FwdArgs a, FourPlan fs,
                                                               T* __restrict__ ore, T* __restrict__ oim) {
  constexpr int R = kRows<T>;
  extern __shared__ __align__(16) unsigned char four_lds[];
  const int N1 = fs.N1, N2 = fs.N2, N = N1 * N2, tid = threadIdx.x;
  const int LU = fs.lu, LV = fs.lv, LG = LU + LV, TB = 1 << LU, JB = 1 << LV, rows = kNT >> LG, npw = tube_powers(fs);
  const FourLds<T> l(npw << LV, N2, fs.ldt, four_lds);
  const int64_t ks = a.ntubes;
  TubeTiles tiles(ks, fs);
  lfft::fill_all_roots(N2, l.tab);
  lfft::fill_positions(fs.p2, l.pos);
  // z[j1 + N1 j2] of sequence (u, v): lanes on consecutive j1 read, on consecutive
  // slots write; the column u ^ v keeps both on different banks
  Two<T> z[R];
  double sc = 1.0;
  bool ok = false;
  const auto load = [&](int64_t sb, int jb) {
    const int td = opaque(tid);
    const int64_t t = (sb << LU) + ((td >> LV) & (TB - 1));
    const int j1 = (jb << LV) + (td & (JB - 1));
    int64_t src = 0;
    sc = 1.0;
    ok = t < ks && j1 < N1 && tube_source(a, t, src, sc);
    const T* p = x + (ok ? src * (int64_t)(2 * N) + 2 * (int64_t)j1 : 0);
    const int last = ok ? N2 - 1 : 0, r = td >> LG;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int j2 = r + q * rows;
      z[q] = load_two(p + 2 * ((int64_t)N1 * (j2 < last ? j2 : last)));
    }
  };
  int64_t sb, nsb;
  int jb, njb;
  bool more = tiles.next(sb, jb);
  if (kAhead<T> && more) load(sb, jb);
  while (more) {
    if (!kAhead<T>) load(sb, jb);
    {
      const int td = opaque(tid), v = td & (JB - 1), u = (td >> LV) & (TB - 1), r = td >> LG;
      Cx<T>* w = l.buf + (v << LU) + (u ^ (v & (TB - 1)));
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const int j2 = r + q * rows;
        if (j2 >= N2) continue;
        T zr = z[q].x, zi = z[q].y;
        if (sc != 1.0) {
          zr = (T)((double)zr * sc);
          zi = (T)((double)zi * sc);
        }
        w[j2 * fs.ldt] = ok ? Cx<T>{zr, zi} : Cx<T>{T(0), T(0)};
      }
    }
    const int lp = kLogNT - LV, v0 = opaque(tid) >> lp;
    fill_powers(l.pw + v0 * npw, rows, npw - rows - 1, 0, (jb << LV) + v0, N, tid & ((1 << lp) - 1), 1 << lp);
    __syncthreads();
    more = tiles.next(nsb, njb);
    if (kAhead<T> && more) load(nsb, njb);
    lfft::stages<T, true, true>(fs.p2, l.buf, LG, fs.ldt, lfft::AllRoots<T>{l.tab});
    // twiddle W_N^{j1 k2}; value (t, j1, k2) goes to slice k2 + N2 j1 of slot t
    const int td = opaque(tid), u = td & (TB - 1), v = (td >> LU) & (JB - 1), r0 = td >> LG;
    const int64_t t = (sb << LU) + u;
    const int j1 = (jb << LV) + v;
    if (t < ks && j1 < N1) {
      const Cx<T>* w = l.buf + (v << LU) + (u ^ (v & (TB - 1)));
      const Cx<double>* pw = l.pw + v * npw;
      const Cx<double> lo = pw[r0];
      const int64_t o = (int64_t)N2 * j1 * ks + t;
#pragma unroll 4
      for (int k2 = r0, i = rows; k2 < N2; k2 += rows, ++i) {
        const Cx<T> y = w[(int)l.pos[k2] * fs.ldt];
        const Cx<double> r = times(times(lo, pw[i]), Cx<double>{(double)y.x, (double)y.y});
        ore[o + k2 * ks] = (T)r.x;
        oim[o + k2 * ks] = (T)r.y;
      }
    }
    __syncthreads();
    sb = nsb;
    jb = njb;
  }
}

// The k1 of the partner N - k of k = k2 + N2 k1 (in the other sequence of the
// pair, or in the same one where k2 = N2 - k2 mod N2)
__device__ __forceinline__ int partner(int k2, int k1, int N1) { return k2 == 0 ? (k1 ? N1 - k1 : 0) : N1 - 1 - k1; }

// forward slice pass, sequence h 2^ls + u
template <typename T>
__global__ __launch_bounds__(kNT, 4) void four_fwd_slice_kernel(FourPlan fs, int64_t ks, T* ore, T* oim) {
  constexpr int R = kRows<T>;
  extern __shared__ __align__(16) unsigned char four_lds[];
  const int N1 = fs.N1, N2 = fs.N2, N = N1 * N2, tid = threadIdx.x;
  const int LS = fs.ls, LG = LS + 1, SB = 1 << LS, rows = kNT >> LG, pairs = kNT >> LS, npn = half_powers(fs);
  const FourLds<T> l(npn, N1, fs.lds, four_lds);
  SliceTiles tiles(ks, fs);
  lfft::fill_all_roots(N1, l.tab);
  lfft::fill_positions(fs.p1, l.pos);
  const int64_t step = (int64_t)N2 * ks;
  T zr[R], zi[R];
  const auto load = [&](int64_t sb, int ka) {
    const int td = opaque(tid), h = (td >> LS) & 1;
    const int64_t t = (sb << LS) + (td & (SB - 1));
    const bool ok = t < ks;
    const int64_t o = ok ? (int64_t)(h && ka ? N2 - ka : ka) * ks + t : 0;
    const int last = ok ? N1 - 1 : 0, r = td >> LG;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int j1 = r + q * rows;
      const int64_t oo = o + (j1 < last ? j1 : last) * step;
      zr[q] = ore[oo];
      zi[q] = oim[oo];
    }
  };
  int64_t sb, nsb;
  int ka, nka;
  bool more = tiles.next(sb, ka);
  if (kAhead<T> && more) load(sb, ka);
  while (more) {
    if (!kAhead<T>) load(sb, ka);
    {
      const int td = opaque(tid), r = td >> LG;
      Cx<T>* w = l.buf + (td & ((1 << LG) - 1));
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const int j1 = r + q * rows;
        if (j1 < N1) w[j1 * fs.lds] = Cx<T>{zr[q], zi[q]};
      }
    }
    fill_powers(l.pw, pairs, npn - pairs, ka, N2, 2 * N, tid, kNT);  // W_n^k, k = ka + N2 k1
    // (every value of the pair is in LDS before the first is overwritten)
    __syncthreads();
    more = tiles.next(nsb, nka);
    if (kAhead<T> && more) load(nsb, nka);
    lfft::stages<T, true, true>(fs.p1, l.buf, LG, fs.lds, lfft::AllRoots<T>{l.tab});
    const int td = opaque(tid), u = td & (SB - 1), rs = td >> LS;
    const int64_t t = (sb << LS) + u;
    if (t < ks) {
      const bool two = ka != 0 && 2 * ka != N2;
      const Cx<double> lo = l.pw[rs];
      const Cx<T>*wa = l.buf + u, *wb = l.buf + (two ? SB : 0) + u;
      T *fr = ore + t, *fi = oim + t;
#pragma unroll 2
      for (int k1 = rs, i = pairs; k1 < N1; k1 += pairs, ++i) {
        const int p1 = partner(ka, k1, N1);
        if (!two && k1 > p1) continue;
        const Cx<T> za = wa[(int)l.pos[k1] * fs.lds], zb = wb[(int)l.pos[p1] * fs.lds];
        const int k = ka + N2 * k1;
        const double xr = (double)za.x, xi = (double)za.y, yr = (double)zb.x, yi = (double)zb.y;
        if (k == 0) {
          fr[0] = (T)(xr + xi);
          fi[0] = T(0);
          fr[(int64_t)N * ks] = (T)(xr - xi);
          fi[(int64_t)N * ks] = T(0);
          continue;
        }
        const double er = 0.5 * (xr + yr), ei = 0.5 * (xi - yi);
        const Cx<double> p = times(times(lo, l.pw[i]), Cx<double>{0.5 * (xi + yi), 0.5 * (yr - xr)});
        fr[k * ks] = (T)(er + p.x);
        fi[k * ks] = (T)(ei + p.y);
        if (two || k1 < p1) {
          fr[(N - k) * ks] = (T)(er - p.x);
          fi[(N - k) * ks] = (T)(p.y - ei);
        }
      }
    }
    __syncthreads();
    sb = nsb;
    ka = nka;
  }
}

// inverse slice pass, sequence h 2^ls + u
template <typename T>
__global__ __launch_bounds__(kNT, 4) void four_inv_slice_kernel(const T* __restrict__ xre, const T* __restrict__ xim,
                                                                int64_t ks, FourPlan fs, T* __restrict__ y) {
  constexpr int R = kRows<T> / 2;
  extern __shared__ __align__(16) unsigned char four_lds[];
  const int N1 = fs.N1, N2 = fs.N2, N = N1 * N2, tid = threadIdx.x;
  const int LS = fs.ls, LG = LS + 1, SB = 1 << LS, rows = kNT >> LG, pairs = kNT >> LS;
  const int npw = pair_powers(fs), npn = half_powers(fs);
  const FourLds<T> l(2 * npw + npn, N1, fs.lds, four_lds);
  const Cx<double>* pn = l.pw + 2 * npw;  // W_n^k, k = ka + N2 k1
  SliceTiles tiles(ks, fs);
  lfft::fill_all_roots(N1, l.tab);
  lfft::fill_positions(fs.p1, l.pos);
  T ar[R], ai[R], br[R], bi[R];
  const auto load = [&](int64_t sb, int ka) {
    const int td = opaque(tid);
    const int64_t t = (sb << LS) + (td & (SB - 1)), tt = t < ks ? t : 0;
    const T *fr = xre + tt, *fi = xim + tt;
    const int last = t < ks ? N1 - 1 : 0, r = td >> LS;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int k1 = r + q * pairs;
      const int64_t k = ka + N2 * (k1 < last ? k1 : last);
      ar[q] = fr[k * ks];
      ai[q] = fi[k * ks];
      br[q] = fr[(N - k) * ks];
      bi[q] = fi[(N - k) * ks];
    }
  };
  int64_t sb, nsb;
  int ka, nka;
  bool more = tiles.next(sb, ka);
  if (kAhead<T> && more) load(sb, ka);
  while (more) {
    if (!kAhead<T>) load(sb, ka);
    const bool two = ka != 0 && 2 * ka != N2;
    const int kb = ka ? N2 - ka : 0;
    fill_powers(l.pw + 2 * npw, pairs, npn - pairs, ka, N2, 2 * N, tid, kNT);
    fill_powers(l.pw + (tid < kNT / 2 ? 0 : npw), rows, npw - rows, 0, tid < kNT / 2 ? ka : kb, N, tid % (kNT / 2),
                kNT / 2);  // W_N^{j1 k2} of either k2
    __syncthreads();
    // conj Z: the forward stages of the conjugate give the conjugate of the inverse
    {
      const int td = opaque(tid), u = td & (SB - 1), r = td >> LS;
      const Cx<double> lo = pn[r];
      Cx<T>*wa = l.buf + u, *wb = l.buf + SB + u;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const int k1 = r + q * pairs;
        if (k1 >= N1) continue;
        const bool first = ka == 0 && k1 == 0;
        const double xr = (double)ar[q], xi = first ? 0.0 : (double)ai[q];
        const double yr = (double)br[q], yi = first ? 0.0 : (double)bi[q];
        const double er = 0.5 * (xr + yr), ei = 0.5 * (xi - yi);
        const Cx<double> w = times(lo, pn[pairs + q]);
        const Cx<double> d = times(Cx<double>{w.x, -w.y}, Cx<double>{0.5 * (xr - yr), 0.5 * (xi + yi)});
        wa[(int)l.pos[k1] * fs.lds] = Cx<T>{(T)(er - d.y), (T)(-(ei + d.x))};
        if (two) wb[(int)l.pos[partner(ka, k1, N1)] * fs.lds] = Cx<T>{(T)(er + d.y), (T)(ei - d.x)};
      }
    }
    __syncthreads();
    more = tiles.next(nsb, nka);
    if (kAhead<T> && more) load(nsb, nka);
    lfft::stages<T, false, true>(fs.p1, l.buf, LG, fs.lds, lfft::AllRoots<T>{l.tab});
    // u[j1] = conj(stage result) W_N^{-j1 k2} = conj(result W_N^{j1 k2}), stored at
    // packed position j1 + N1 k2 of the slot's tube, lanes on consecutive j1
    const int td = opaque(tid), s = td >> (kLogNT - LG), h = s >> LS, r0 = td & (rows - 1);
    const int64_t t = (sb << LS) + (s & (SB - 1));
    if (t < ks && !(h && !two)) {
      const Cx<T>* w = l.buf + s;
      const Cx<double>* pw = l.pw + h * npw;
      const Cx<double> lo = pw[r0];
      T* row = y + t * (int64_t)(2 * N) + 2 * (int64_t)N1 * (h ? kb : ka);
#pragma unroll 4
      for (int j1 = r0, i = rows; j1 < N1; j1 += rows, ++i) {
        const Cx<T> z = w[j1 * fs.lds];
        const Cx<double> r = times(times(lo, pw[i]), Cx<double>{(double)z.x, (double)z.y});
        store_two(row + 2 * j1, (T)r.x, (T)-r.y);
      }
    }
    __syncthreads();
    sb = nsb;
    ka = nka;
  }
}

// inverse tube pass, in place in y
template <typename T>
__global__ __launch_bounds__(kNT, 4) void four_inv_tube_kernel(int64_t ks, FourPlan fs, T* y) {
  constexpr int R = kRows<T>;
  extern __shared__ __align__(16) unsigned char four_lds[];
  const int N1 = fs.N1, N2 = fs.N2, N = N1 * N2, tid = threadIdx.x;
  const int LU = fs.lu, LV = fs.lv, LG = LU + LV, rows = kNT >> LG;
  const FourLds<T> l(0, N2, fs.ldt, four_lds);
  TubeTiles tiles(ks, fs);
  lfft::fill_all_roots(N2, l.tab);
  lfft::fill_positions(fs.p2, l.pos);
  const int v = tid & ((1 << LV) - 1), u = (tid >> LV) & ((1 << LU) - 1), r0 = tid >> LG;
  Cx<T>* w = l.buf + (tid & ((1 << LG) - 1));
  Two<T> z[R];
  T *p = y, *np = y;
  bool ok = false, nok = false;
  const auto load = [&](int64_t sb, int jb) {
    const int64_t t = (sb << LU) + u;
    const int j1 = (jb << LV) + v;
    nok = t < ks && j1 < N1;
    np = y + (nok ? t * (int64_t)(2 * N) + 2 * j1 : 0);
    const int last = nok ? N2 - 1 : 0, r = opaque(r0);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int k2 = r + q * rows;
      z[q] = load_two(np + 2 * ((int64_t)N1 * (k2 < last ? k2 : last)));
    }
  };
  const double inv = 1.0 / (double)N;
  int64_t sb;
  int jb;
  bool more = tiles.next(sb, jb);
  if (kAhead<T> && more) load(sb, jb);
  while (more) {
    if (!kAhead<T>) load(sb, jb);
    p = np;
    ok = nok;
    const int r = opaque(r0);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int k2 = r + q * rows;
      if (k2 < N2) w[k2 * fs.ldt] = Cx<T>{z[q].x, (T)-z[q].y};  // conjugate in, conjugate out
    }
    __syncthreads();
    more = tiles.next(sb, jb);
    if (kAhead<T> && more) load(sb, jb);
    lfft::stages<T, true, true>(fs.p2, l.buf, LG, fs.ldt, lfft::AllRoots<T>{l.tab});
    if (ok) {
#pragma unroll 4
      for (int j2 = opaque(r0); j2 < N2; j2 += rows) {
        const Cx<T> c = w[(int)l.pos[j2] * fs.ldt];
        store_two(p + 2 * ((int64_t)N1 * j2), (T)((double)c.x * inv), (T)(-(double)c.y * inv));
      }
    }
    __syncthreads();
  }
}

// Four-step plan of an even n: N = n/2 = N1 N2 with N2 the largest divisor
// <= kMaxN2 that leaves N1 <= kMaxN1, both without prime factors above 13; where
// there is none, the smallest divisor above kMaxN2 and up to kMaxN1 that does
// (375 x 625), else the same with N1 <= 2 kMaxN1 (1331 x 121): so every n up to
// 2 kMaxN1 kMaxN2 whose half has no prime factor above 13.
bool four_plan(int64_t n, FourPlan& fs) {
  if (n % 2 || n < 4) return false;
  const int64_t N = n / 2;
  if (N > (int64_t)kMaxN1 * kMaxN2) return false;
  const auto take = [&](int64_t n2, int64_t most) {
    if (N % n2 || N / n2 > most) return false;
    fs.N1 = (int)(N / n2);
    fs.N2 = (int)n2;
    return lfft::radix_plan(fs.N1, fs.p1) && lfft::radix_plan(fs.N2, fs.p2);
  };
  for (const int64_t most : {kMaxN1, 2 * kMaxN1}) {
    for (int64_t n2 = kMaxN2 < N ? kMaxN2 : N; n2 >= 1 && N / n2 <= most; --n2)
      if (take(n2, most)) return true;
    for (int64_t n2 = kMaxN2 + 1; n2 <= kMaxN1 && n2 <= N; ++n2)
      if (take(n2, most)) return true;
  }
  return false;
}

int log2_ceil(int64_t n) {
  int l = 0;
  while ((int64_t(1) << l) < n) ++l;
  return l;
}

// Tiles: as many sequences as kRows rows a thread hold; of a tube pass eight
// slots (fewer if there are fewer) and up to 16 values of j1.
template <typename T>
void set_geometry(int64_t ntubes, FourPlan& f) {
  const int most = kNT * kRows<T>;
  const int kt = log2_ceil(ntubes);
  f.lu = std::min(3, kt);
  f.lv = std::min(kMaxLV, log2_ceil(f.N1));
  while ((f.N2 << (f.lu + f.lv)) > most) --f.lv;
  f.ls = 0;
  while (f.ls < std::min(8, kt) && (f.N1 << (f.ls + 2)) <= most) ++f.ls;
  f.ldt = (1 << (f.lu + f.lv)) + (sizeof(T) == 4);
  f.lds = (2 << f.ls) + (sizeof(T) == 4);
}

template <typename T>
struct Grids {
  int64_t tube, slice;
  size_t lft, lfs, lis, lit;  // LDS of the passes
  bool fit;
  Grids(int64_t ntubes, const FourPlan& f) {
    const int64_t nsb = (ntubes + (1 << f.lu) - 1) >> f.lu, nj = (f.N1 + (1 << f.lv) - 1) >> f.lv;
    tube = (nj + 3) / 4 * ((nsb + 3) / 4) * 16;
    slice = ((ntubes + (1 << f.ls) - 1) >> f.ls) * (f.N2 / 2 + 1);
    fit = tube <= 0x7fffffffLL && slice <= 0x7fffffffLL;
    // one workgroup a CU
    tube = xcd_grid(std::min<int64_t>(tube, 256));
    slice = xcd_grid(std::min<int64_t>(slice, 256));
    lft = FourLds<T>(tube_powers(f) << f.lv, f.N2, f.ldt, nullptr).bytes;
    lit = FourLds<T>(0, f.N2, f.ldt, nullptr).bytes;
    lfs = FourLds<T>(half_powers(f), f.N1, f.lds, nullptr).bytes;
    lis = FourLds<T>(half_powers(f) + 2 * pair_powers(f), f.N1, f.lds, nullptr).bytes;
  }
};

template <typename T>
int forward(const T* x, const FwdArgs& a, FourPlan& fs, T* re, T* im, hipStream_t st) {
  set_geometry<T>(a.ntubes, fs);
  const Grids<T> g(a.ntubes, fs);
  if (!g.fit) return fail(TP_EUNSUPPORTED, "too many tubes");
  hipLaunchKernelGGL(four_fwd_tube_kernel<T>, dim3((unsigned)g.tube), dim3(kNT), g.lft, st, x, a, fs, re, im);
  TP_LAUNCH_CHECK();
  hipLaunchKernelGGL(four_fwd_slice_kernel<T>, dim3((unsigned)g.slice), dim3(kNT), g.lfs, st, fs, a.ntubes, re, im);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

template <typename T>
int inverse(const T* re, const T* im, int64_t ntubes, FourPlan& fs, T* y, hipStream_t st) {
  set_geometry<T>(ntubes, fs);
  const Grids<T> g(ntubes, fs);
  if (!g.fit) return fail(TP_EUNSUPPORTED, "too many tubes");
  hipLaunchKernelGGL(four_inv_slice_kernel<T>, dim3((unsigned)g.slice), dim3(kNT), g.lis, st, re, im, ntubes, fs, y);
  TP_LAUNCH_CHECK();
  hipLaunchKernelGGL(four_inv_tube_kernel<T>, dim3((unsigned)g.tube), dim3(kNT), g.lit, st, ntubes, fs, y);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

}  // namespace

int four_forward(const void* x, int dtype, int64_t n3, const FwdArgs& a, void* re, void* im, hipStream_t st,
                 bool* handled) {
  FourPlan fs;
  *handled = four_plan(n3, fs);
  if (!*handled) return TP_OK;
  return dtype == TP_F64 ? forward<double>((const double*)x, a, fs, (double*)re, (double*)im, st)
                         : forward<float>((const float*)x, a, fs, (float*)re, (float*)im, st);
}

int four_inverse(const void* re, const void* im, int dtype, int64_t n3, int64_t ntubes, void* y, hipStream_t st,
                 bool* handled) {
  FourPlan fs;
  *handled = four_plan(n3, fs);
  if (!*handled) return TP_OK;
  return dtype == TP_F64 ? inverse<double>((const double*)re, (const double*)im, ntubes, fs, (double*)y, st)
                         : inverse<float>((const float*)re, (const float*)im, ntubes, fs, (float*)y, st);
}

}  // namespace tp
