// Tube transforms of the lengths without prime factors above 13 that LDS holds
// and that have no register kernel: 2^lg tubes per workgroup.
//
// A real tube of even length n is packed as N = n/2 complex values
// z[m] = x[2m] + i x[2m+1]; an odd one takes N = n complex values with zero
// imaginary part. The N-point transforms run in place through LDS in the
// mixed-radix stages of fft_stages.hpp. Lengths whose N has a prime factor
// above 13 take the dense products of fft_dense.hip.
//
// What bounds it: HBM, then the LDS round trips of the stages. Several tubes
// per workgroup make the spectrum side of the transform, slice-major, runs of
// 2^lg neighbouring values instead of single ones, and spread the roots and
// the index table over that many tubes; XCD-contiguous
// launch order lets neighbouring workgroups complete each other's cache lines
// in one L2. Stages of radix up to 16 in registers (three for n = 2000), with
// float64 butterflies (see fft_stages.hpp).
// Measured (3e7 values, us forward / inverse, against the transforms these
// replaced: one workgroup per tube with a run-time radix for n > 256, a direct
// sum per tube below): float32 n = 80 1374 / 1901 -> 112 / 80, n = 256
// 2677 / 11831 -> 112 / 80, n = 2000 1656 / 1641 -> 118 / 98; float64 n = 60 1779 / 2197 -> 132 / 117,
// n = 2000 1626 / 1697 -> 194 / 188. A copy of the same bytes takes 46 (92) us:
// the rest is the vector work of the stages, whose LDS round trips and
// twiddles take about as long as the bytes.
#include <algorithm>
#include <cmath>

#include "fft_stages.hpp"
#include "fft_tubes.hpp"

namespace tp {
namespace lfft {

namespace {

struct Radix {
  int p;
  float cost;  // of a stage, per element: its LDS round trip and its butterfly
};
// (14 only where a 7 and a 2 would be left)
constexpr Radix kRadices[] = {{16, 25}, {15, 26}, {14, 35}, {13, 35}, {12, 23}, {11, 33}, {10, 23}, {9, 24},
                              {8, 21},  {7, 27},  {6, 21},  {5, 21},  {4, 18},  {3, 19},  {2, 16}};

void search(int n, int first, float cost, int depth, int* cur, float& best, int* out, int& nout) {
  if (cost >= best) return;
  if (n == 1) {
    best = cost;
    nout = depth;
    for (int i = 0; i < depth; ++i) out[i] = cur[i];
    return;
  }
  if (depth == kMaxStages) return;
  for (int i = first; i < (int)(sizeof(kRadices) / sizeof(Radix)); ++i) {
    if (n % kRadices[i].p) continue;
    cur[depth] = kRadices[i].p;
    search(n / kRadices[i].p, i, cost + kRadices[i].cost, depth + 1, cur, best, out, nout);
  }
}

}  // namespace

bool radix_plan(int64_t n, Plan& pl) {
  int64_t r = n;
  for (int p : {2, 3, 5, 7, 11, 13})
    while (r % p == 0) r /= p;
  if (n < 1 || r != 1 || n >= (1 << 16)) return false;
  int cur[kMaxStages];
  float best = 1e30f;
  pl.n = (int)n;
  pl.nst = 0;
  search((int)n, 0, 0.0f, 0, cur, best, pl.rad, pl.nst);
  if (n > 1 && pl.nst == 0) return false;
  int m = 1;
  for (int q = 0; q < pl.nst; ++q) {
    pl.m[q] = m;
    pl.mag[q] = m > 1 ? (uint32_t)(((uint64_t(1) << 32) + m - 1) / m) : 0;
    pl.rmag[q] = (uint32_t)(((uint64_t(1) << 32) + pl.rad[q] - 1) / pl.rad[q]);
    m *= pl.rad[q];
    pl.w[q] = (int)n / m;
  }
  return true;
}

}  // namespace lfft

namespace {

using lfft::Cx;

constexpr int kMaxNT = 512;
constexpr int64_t kLdsMax = 160 * 1024;  // per workgroup (and per CU)

struct LdsPlan {
  int n, N, lg;  // tube length, complex length, log2 of the tubes per workgroup
  lfft::Plan pl; // length N
};

// dynamic LDS, in order: roots of the stages; data; tube sources and scales;
// positions
template <typename S>
struct Layout {
  Cx<double>* tab;
  Cx<S>* buf;
  int64_t* src;  // [2][tubes]: of this block and the next
  double* scl;
  uint16_t* pos;
  size_t bytes;
  __host__ __device__ Layout(const LdsPlan& p, unsigned char* base) {
    size_t o = 0;
    tab = (Cx<double>*)(base + o);
    o += sizeof(Cx<double>) * (p.N / 2 + 1);
    buf = (Cx<S>*)(base + o);
    o += (sizeof(Cx<S>) * p.N) << p.lg;
    src = (int64_t*)(base + o);
    o += size_t(16) << p.lg;
    scl = (double*)(base + o);
    o += size_t(16) << p.lg;
    pos = (uint16_t*)(base + o);
    o += 2 * size_t(p.N);
    bytes = o;
  }
};

// E consecutive values from an address aligned to one value
template <typename T, int E>
struct Run {
  T v[E];
};
template <typename T, int E>
__device__ __forceinline__ Run<T, E> load_run(const T* p) {
  Run<T, E> r;
  __builtin_memcpy(&r, p, sizeof(r));
  return r;
}
template <typename T, int E>
__device__ __forceinline__ void store_run(T* p, const Run<T, E>& r) {
  __builtin_memcpy(p, &r, sizeof(r));
}

// element k of the transform of the sequence `u` (after the stages)
template <typename S>
__device__ __forceinline__ void result(const LdsPlan& p, const Layout<S>& l, int k, int u, double& r, double& i) {
  const Cx<S> v = l.buf[((int)l.pos[k] << p.lg) + u];
  r = (double)v.x;
  i = (double)v.y;
}

// Tube-major side: pieces of E values, 2^plog consecutive pieces of a tube
// (64 to 128 bytes) per run of lanes, then the next tube, then the next run.
// f -> (piece, tube)
struct Pieces {
  int nv, plog, total;
  __device__ Pieces(int nv_, int lg) : nv(nv_) {
    plog = 0;
    while ((1 << plog) < nv && plog < 3) ++plog;
    total = (((nv + (1 << plog) - 1) >> plog) << plog) << lg;
  }
  __device__ __forceinline__ void at(int f, int lg, int& piece, int& u) const {
    u = (f >> plog) & ((1 << lg) - 1);
    piece = ((f >> (plog + lg)) << plog) + (f & ((1 << plog) - 1));
  }
};

constexpr int kBatch = 8;  // pieces whose loads a thread keeps in flight

// Reads the tubes into buf in natural order. E values make E/2 complex
// elements (even n), or one with zero imaginary part (E = 1, odd n).
template <typename T, typename S, int E>
__device__ void load_tubes(const T* x, const int64_t* src, const double* scl, const LdsPlan& p,
                           const Layout<S>& l) {
  const Pieces pc(p.n / E, p.lg);
  for (int f0 = threadIdx.x; f0 < pc.total; f0 += kBatch * blockDim.x) {
    Run<T, E> v[kBatch];
    // unconditional loads from clamped addresses, so that all stay in flight
#pragma unroll
    for (int q = 0; q < kBatch; ++q) {
      const int f = f0 + q * blockDim.x;
      int piece, u;
      pc.at(f, p.lg, piece, u);
      const bool ok = f < pc.total && piece < pc.nv && src[u] >= 0;
      v[q] = load_run<T, E>(x + (ok ? src[u] * p.n + (int64_t)piece * E : 0));
    }
#pragma unroll
    for (int q = 0; q < kBatch; ++q) {
      const int f = f0 + q * blockDim.x;
      int piece, u;
      pc.at(f, p.lg, piece, u);
      if (f >= pc.total || piece >= pc.nv) continue;
      const bool live = src[u] >= 0;
      const double s = scl[u];
      T w[E];
#pragma unroll
      for (int e = 0; e < E; ++e) w[e] = !live ? T(0) : (s == 1.0) ? v[q].v[e] : (T)((double)v[q].v[e] * s);
      constexpr int C = E > 1 ? E / 2 : 1;
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const int m = piece * C + c;
        const double zr = (double)w[E > 1 ? 2 * c : 0], zi = E > 1 ? (double)w[E > 1 ? 2 * c + 1 : 0] : 0.0;
        l.buf[(m << p.lg) + u] = Cx<S>{(S)zr, (S)zi};
      }
    }
  }
}

// Inverse transforms are divided by their length in float64: where they are read
// if float32 values lie between the stages, which round the last stage's, else
// where they are written
template <typename S>
constexpr bool kDivideFirst = sizeof(S) == 4;

// Writes the tubes: element m of the transformed conjugate, conjugated, is the
// tube's values 2m and 2m+1 (odd n: value m)
template <typename T, typename S, int E>
__device__ void store_tubes(T* y, int64_t t0, int64_t ntubes, const LdsPlan& p, const Layout<S>& l) {
  const Pieces pc(p.n / E, p.lg);
  const double inv = kDivideFirst<S> ? 1.0 : 1.0 / (double)p.N;
  for (int f = threadIdx.x; f < pc.total; f += blockDim.x) {
    int piece, u;
    pc.at(f, p.lg, piece, u);
    const int64_t t = t0 + u;
    if (piece >= pc.nv || t >= ntubes) continue;
    constexpr int C = E > 1 ? E / 2 : 1;
    Run<T, E> v;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int m = piece * C + c;
      const Cx<S> w = l.buf[(m << p.lg) + u];
      v.v[E > 1 ? 2 * c : 0] = (T)((double)w.x * inv);
      if constexpr (E > 1) v.v[2 * c + 1] = (T)(-(double)w.y * inv);
    }
    store_run<T, E>(y + t * p.n + (int64_t)piece * E, v);
  }
}

template <typename T, typename S>
__global__ __launch_bounds__(kMaxNT, 4) void rfft_lds_kernel(const T* __restrict__ x, FwdArgs a, LdsPlan p,
                                                          T* __restrict__ ore, T* __restrict__ oim) {
  constexpr bool EXACT = sizeof(T) == 8;
  extern __shared__ __align__(16) unsigned char lfft_lds[];
  const Layout<S> l(p, lfft_lds);
  const int TB = 1 << p.lg, N = p.N;
  const int64_t ks = a.ntubes;
  auto sources = [&](int64_t G, int half) {
    for (int u = threadIdx.x; u < TB; u += blockDim.x) {
      const int64_t t = (G << p.lg) + u;
      int64_t src = -1;
      double s = 0.0;
      if (!(t < ks && tube_source(a, t, src, s))) src = -1;
      l.src[half * TB + u] = src;
      l.scl[half * TB + u] = s;
    }
  };
  XcdWalk walk((ks + TB - 1) >> p.lg);
  int64_t G, next;
  bool more = walk.next(G);
  if (!more) return;
  sources(G, 0);
  lfft::fill_roots(N, l.tab);
  lfft::fill_positions(p.pl, l.pos);
  __syncthreads();
  for (int half = 0; more; half ^= 1, G = next) {
    const int64_t t0 = G << p.lg;
    const int64_t* src = l.src + half * TB;
    const double* scl = l.scl + half * TB;
    if (p.n % 2)
      load_tubes<T, S, 1>(x, src, scl, p, l);
    else if (sizeof(T) == 4 && p.n % 4 == 0)
      load_tubes<T, S, sizeof(T) == 4 ? 4 : 2>(x, src, scl, p, l);
    else
      load_tubes<T, S, 2>(x, src, scl, p, l);
    more = walk.next(next);
    if (more) sources(next, half ^ 1);
    __syncthreads();
    lfft::stages<S, true, EXACT>(p.pl, l.buf, p.lg, l.tab);
    if (p.n % 2) {
      for (int e = threadIdx.x; e < ((p.n / 2 + 1) << p.lg); e += blockDim.x) {
        const int k = e >> p.lg, u = e & (TB - 1);
        const int64_t t = t0 + u;
        if (t >= ks) continue;
        double r, i;
        result<S>(p, l, k, u, r, i);
        ore[(int64_t)k * ks + t] = (T)r;
        oim[(int64_t)k * ks + t] = k == 0 ? T(0) : (T)i;
      }
      __syncthreads();
      continue;
    }
    // X[k] = E[k] + W_n^k O[k] for the pair (k, N - k), E[k] = (Z[k] + conj Z[N-k]) / 2,
    // O[k] = (Z[k] - conj Z[N-k]) / 2i; W_n^{N-k} = -conj W_n^k
    for (int e = threadIdx.x; e < ((N / 2 + 1) << p.lg); e += blockDim.x) {
      const int k = e >> p.lg, u = e & (TB - 1);
      const int64_t t = t0 + u;
      if (t >= ks) continue;
      double zr, zi, wr, wi;
      result<S>(p, l, k, u, zr, zi);
      if (k == 0) {
        ore[t] = (T)(zr + zi);
        oim[t] = T(0);
        ore[(int64_t)N * ks + t] = (T)(zr - zi);
        oim[(int64_t)N * ks + t] = T(0);
        continue;
      }
      result<S>(p, l, N - k, u, wr, wi);
      const double er = 0.5 * (zr + wr), ei = 0.5 * (zi - wi);
      const double dr = 0.5 * (zi + wi), di = 0.5 * (wr - zr);
      const Cx<double> w = l.tab[k];
      const double pr = dr * w.x - di * w.y, pi = dr * w.y + di * w.x;
      ore[(int64_t)k * ks + t] = (T)(er + pr);
      oim[(int64_t)k * ks + t] = (T)(ei + pi);
      if (2 * k < N) {
        ore[(int64_t)(N - k) * ks + t] = (T)(er - pr);
        oim[(int64_t)(N - k) * ks + t] = (T)(pi - ei);
      }
    }
    __syncthreads();
  }
}

constexpr int kInvBatch = 4;  // (k, N - k) pairs whose loads a thread keeps in flight

template <typename T, typename S>
__global__ __launch_bounds__(kMaxNT, 4) void irfft_lds_kernel(const T* __restrict__ xre, const T* __restrict__ xim,
                                                           int64_t ks, LdsPlan p, T* __restrict__ y) {
  constexpr bool EXACT = sizeof(T) == 8;
  extern __shared__ __align__(16) unsigned char lfft_lds[];
  const Layout<S> l(p, lfft_lds);
  const int TB = 1 << p.lg, N = p.N;
  lfft::fill_roots(N, l.tab);
  lfft::fill_positions(p.pl, l.pos);
  __syncthreads();
  const double inv = kDivideFirst<S> ? 1.0 / (double)N : 1.0;
  XcdWalk walk((ks + TB - 1) >> p.lg);
  for (int64_t G; walk.next(G);) {
    const int64_t t0 = G << p.lg;
    // conj Z into buf: the forward transform of the conjugate is the conjugate
    // of the inverse
    auto put = [&](int k, int u, double zr, double zi) {
      l.buf[((int)l.pos[k] << p.lg) + u] = Cx<S>{(S)(zr * inv), (S)(zi * inv)};
    };
    const bool odd = p.n % 2;
    const int total = (N / 2 + 1) << p.lg;
    for (int e0 = threadIdx.x; e0 < total; e0 += kInvBatch * blockDim.x) {
      T ar[kInvBatch], ai[kInvBatch], br[kInvBatch], bi[kInvBatch];
#pragma unroll
      for (int q = 0; q < kInvBatch; ++q) {
        const int e = e0 + q * blockDim.x;
        const int k = e < total ? e >> p.lg : 0, u = e & (TB - 1);
        const int64_t t = t0 + u < ks ? t0 + u : ks - 1;
        const int64_t oa = (int64_t)k * ks + t, ob = odd ? oa : (int64_t)(N - k) * ks + t;
        ar[q] = xre[oa];
        ai[q] = xim[oa];
        br[q] = xre[ob];
        bi[q] = xim[ob];
      }
#pragma unroll
      for (int q = 0; q < kInvBatch; ++q) {
        const int e = e0 + q * blockDim.x;
        if (e >= total) continue;
        const int k = e >> p.lg, u = e & (TB - 1);
        const double xr = (double)ar[q], xi = k == 0 ? 0.0 : (double)ai[q];
        if (odd) {
          // Z[n - k] = conj Z[k]
          put(k, u, xr, -xi);
          if (k > 0) put(N - k, u, xr, xi);
          continue;
        }
        // Z[k] = E + i O, E = (X[k] + conj X[N-k]) / 2, O = (X[k] - conj X[N-k]) conj(W_n^k) / 2,
        // Z[N-k] = conj E + i conj O
        const double yr = (double)br[q], yi = k == 0 ? 0.0 : (double)bi[q];
        const double er = 0.5 * (xr + yr), ei = 0.5 * (xi - yi);
        const double dr = 0.5 * (xr - yr), di = 0.5 * (xi + yi);
        const Cx<double> w = l.tab[k];
        const double qr = dr * w.x + di * w.y, qi = di * w.x - dr * w.y;
        put(k, u, er - qi, -(ei + qr));
        if (k > 0 && 2 * k < N) put(N - k, u, er + qi, ei - qr);
      }
    }
    __syncthreads();
    lfft::stages<S, false, EXACT>(p.pl, l.buf, p.lg, l.tab);
    if (odd)
      store_tubes<T, S, 1>(y, t0, ks, p, l);
    else if (sizeof(T) == 4 && p.n % 4 == 0)
      store_tubes<T, S, sizeof(T) == 4 ? 4 : 2>(y, t0, ks, p, l);
    else
      store_tubes<T, S, 2>(y, t0, ks, p, l);
    __syncthreads();
  }
}

// Tubes per workgroup and threads (256 where three workgroups fit a CU: n = 80
// 112 us against 137 with 512; 512 otherwise: n = 2048 117 against 133). As many tubes (a power of two) as leave
// two workgroups per CU (half of the LDS each), or eight if one fills it;
// fewer when there are too few tubes for two workgroups per CU.
template <typename S>
bool lds_fit(LdsPlan& p, int64_t ntubes, size_t& bytes, int& nt) {
  auto need = [&](int lg) {
    LdsPlan q = p;
    q.lg = lg;
    return (int64_t)Layout<S>(q, nullptr).bytes;
  };
  if (need(0) > kLdsMax) return false;
  p.lg = 0;
  while (p.lg < 8 && ((int64_t)p.pl.n << (p.lg + 1)) <= 8192 && (ntubes >> p.lg) > 512 &&
         (need(p.lg + 1) <= kLdsMax / 2 || (p.lg < 3 && need(p.lg + 1) <= kLdsMax)))
    ++p.lg;
  bytes = (size_t)need(p.lg);
  // 256 threads where LDS holds three workgroups per CU, 512 otherwise, and
  // no more than the stages' butterflies
  int most = p.pl.n;
  for (int q = 0; q < p.pl.nst; ++q) most = std::min(most, p.pl.rad[q]);
  nt = bytes * 3 <= (size_t)kLdsMax ? 256 : kMaxNT;
  const int items = std::max(1, p.pl.n / std::max(1, most)) << p.lg;
  nt = std::max(64, std::min(nt, (items + 63) / 64 * 64));
  return true;
}

// Workgroups of a launch over `blocks` tube blocks: as many as the GPU's 256
// CUs hold at once, each walking several blocks, so that the roots, tables and
// filter are made once per workgroup.
int64_t lds_grid(int64_t blocks, size_t bytes, int nt) {
  const int64_t per_cu = std::min<int64_t>(kLdsMax / (int64_t)bytes, 1024 / nt);
  return xcd_grid(std::min<int64_t>(blocks, 256 * std::max<int64_t>(per_cu, 1)));
}

bool lds_plan(int64_t n, LdsPlan& p) {
  p.n = (int)n;
  p.N = n % 2 ? (int)n : (int)(n / 2);
  return lfft::radix_plan(p.N, p.pl);
}

template <typename T, typename S>
int launch_fwd(LdsPlan p, const T* x, const FwdArgs& a, T* re, T* im, hipStream_t st, bool* handled) {
  size_t bytes;
  int nt;
  if (!lds_fit<S>(p, a.ntubes, bytes, nt)) return TP_OK;
  *handled = true;
  const int64_t grid = lds_grid((a.ntubes + (1 << p.lg) - 1) >> p.lg, bytes, nt);
  hipLaunchKernelGGL((rfft_lds_kernel<T, S>), dim3((unsigned)grid), dim3(nt), bytes, st, x, a, p, re, im);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

template <typename T, typename S>
int launch_inv(LdsPlan p, const T* re, const T* im, int64_t ntubes, T* y, hipStream_t st, bool* handled) {
  size_t bytes;
  int nt;
  if (!lds_fit<S>(p, ntubes, bytes, nt)) return TP_OK;
  *handled = true;
  const int64_t grid = lds_grid((ntubes + (1 << p.lg) - 1) >> p.lg, bytes, nt);
  hipLaunchKernelGGL((irfft_lds_kernel<T, S>), dim3((unsigned)grid), dim3(nt), bytes, st, re, im, ntubes, p, y);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

// float32 tubes up to this length are kept in float64 between the stages, and so
// are those of 4 11^a 13^b, whose stages (of 11, of 13, and of the 2 left over)
// would round once more often than the sums of 4, 11 and 13 that a transform of
// the unpacked tube takes (n = 484, float32 between: error 5.2e-8 / 5.6e-8, so
// 2.5e-8 / 1.7e-8; 1.5e6 values 18 / 15 us, so 19 / 16)
constexpr int64_t kWideMax = 256;
bool wide(const LdsPlan& p) {
  int r = p.N % 2 ? 0 : p.N / 2;
  for (int q : {11, 13})
    while (r && r % q == 0) r /= q;
  return p.n <= kWideMax || (r == 1 && p.n % 2 == 0);
}
// lengths that LDS could hold at all
constexpr int64_t kLdsLenMax = 8192;

}  // namespace

int lds_forward(const void* x, int dtype, int64_t n3, const FwdArgs& a, void* re, void* im, hipStream_t st,
                bool* handled) {
  *handled = false;
  LdsPlan p;
  if (n3 < 2 || n3 > kLdsLenMax || !lds_plan(n3, p)) return TP_OK;
  if (dtype == TP_F64)
    return launch_fwd<double, double>(p, (const double*)x, a, (double*)re, (double*)im, st, handled);
  const float* xf = (const float*)x;
  float *fr = (float*)re, *fi = (float*)im;
  return wide(p) ? launch_fwd<float, double>(p, xf, a, fr, fi, st, handled)
                 : launch_fwd<float, float>(p, xf, a, fr, fi, st, handled);
}

int lds_inverse(const void* re, const void* im, int dtype, int64_t n3, int64_t ntubes, void* y, hipStream_t st,
                bool* handled) {
  *handled = false;
  LdsPlan p;
  if (n3 < 2 || n3 > kLdsLenMax || !lds_plan(n3, p)) return TP_OK;
  if (dtype == TP_F64)
    return launch_inv<double, double>(p, (const double*)re, (const double*)im, ntubes, (double*)y, st, handled);
  const float *fr = (const float*)re, *fi = (const float*)im;
  float* yf = (float*)y;
  return wide(p) ? launch_inv<float, double>(p, fr, fi, ntubes, yf, st, handled)
                 : launch_inv<float, float>(p, fr, fi, ntubes, yf, st, handled);
}

}  // namespace tp
