// Tube transforms along the third mode (Section 2.1 "Operators": fft/ifft
// along mode 3, MATLAB convention; the transforms that open and close
// Algorithm 1).
//
// Layout: the tensor is tube-major (each tube X_{ij:} is n3 contiguous
// values); the spectrum is slice-major planar, re[k][tube] / im[k][tube],
// holding the K = n3/2 + 1 non-redundant slices.
//
// Forward kernel (one wavefront = 64 tubes):
//   1. the 64 tubes are read with 16-byte loads, consecutive lanes reading
//      consecutive pieces of a tube, and staged in LDS with a row stride of
//      n3 + 1 words so that the transposed read below is conflict free;
//      gathers of picked slices and their scales are applied here;
//   2. every lane packs its real tube as z[m] = x[2m] + i x[2m+1] and runs a
//      length-n3/2 complex FFT in registers (radix 4/2/5/3 Cooley-Tukey and
//      a direct DFT for other prime factors, fully unrolled, twiddles from a
//      per-device constant table);
//   3. the half spectrum of the real tube is separated from Z by conjugate
//      symmetry, X[k] = (Z[k] + conj Z[M-k])/2 + W_n3^k (Z[k] - conj Z[M-k])/2i,
//      and each slice k is written with one coalesced store per wavefront.
// The inverse kernel runs these steps backwards. Short lengths without a
// packed kernel run one tube per thread (rfft_small_kernel); other lengths
// that LDS holds take the transforms of fft_lds.hip, or of fft_dense.hip where
// there is a prime factor above 13; even ones beyond it (up to 2^19) a
// four-step transform through HBM; the rest a direct O(n3^2) transform.
#include <cmath>
#include <mutex>
#include <vector>

#include "fft_stages.hpp"
#include "fft_tubes.hpp"

namespace tp {
namespace {

// --------------------------------------------------------------------------
// Twiddle tables: W_L^e = exp(-2 pi i e / L) for the lengths below, stored
// back to back (re, im interleaved), computed on the host in long double.
// --------------------------------------------------------------------------
constexpr int kTwLens[] = {1, 2, 4, 8, 16, 32, 64, 128, 256, 5, 10, 20, 25, 50, 100, 200, 7, 21, 84, 168};
constexpr int kTwCount = sizeof(kTwLens) / sizeof(int);

constexpr int tw_offset(int L) {
  int off = 0;
  for (int i = 0; i < kTwCount; ++i) {
    if (kTwLens[i] == L) return off;
    off += kTwLens[i];
  }
  return -1;
}
constexpr int kTwTotal = tw_offset(168) + 168;

__constant__ double g_tw64[2 * kTwTotal];
__constant__ float g_tw32[2 * kTwTotal];

template <typename T>
__device__ __forceinline__ T tw_re(int L, int e);
template <typename T>
__device__ __forceinline__ T tw_im(int L, int e);
template <>
__device__ __forceinline__ double tw_re<double>(int L, int e) { return g_tw64[2 * (tw_offset(L) + e)]; }
template <>
__device__ __forceinline__ double tw_im<double>(int L, int e) { return g_tw64[2 * (tw_offset(L) + e) + 1]; }
template <>
__device__ __forceinline__ float tw_re<float>(int L, int e) { return g_tw32[2 * (tw_offset(L) + e)]; }
template <>
__device__ __forceinline__ float tw_im<float>(int L, int e) { return g_tw32[2 * (tw_offset(L) + e) + 1]; }

std::mutex g_tw_mutex;
std::vector<int> g_tw_ready;  // per device

int ensure_twiddles() {
  int dev = 0;
  TP_HIP_CHECK(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(g_tw_mutex);
  if (dev < (int)g_tw_ready.size() && g_tw_ready[dev]) return TP_OK;
  std::vector<double> t64(2 * kTwTotal);
  std::vector<float> t32(2 * kTwTotal);
  const long double two_pi = 6.283185307179586476925286766559005768L;
  for (int i = 0; i < kTwCount; ++i) {
    int L = kTwLens[i], off = tw_offset(L);
    for (int e = 0; e < L; ++e) {
      long double ang = two_pi * (long double)e / (long double)L;
      long double c = cosl(ang), s = -sinl(ang);
      // exact values where the angle is a multiple of pi/2
      if ((4 * e) % L == 0) {
        int q = (4 * e) / L;
        c = (q == 0) ? 1.0L : (q == 2 ? -1.0L : 0.0L);
        s = (q == 1) ? -1.0L : (q == 3 ? 1.0L : 0.0L);
      }
      t64[2 * (off + e)] = (double)c;
      t64[2 * (off + e) + 1] = (double)s;
      t32[2 * (off + e)] = (float)c;
      t32[2 * (off + e) + 1] = (float)s;
    }
  }
  TP_HIP_CHECK(hipMemcpyToSymbol(HIP_SYMBOL(g_tw64), t64.data(), t64.size() * sizeof(double)));
  TP_HIP_CHECK(hipMemcpyToSymbol(HIP_SYMBOL(g_tw32), t32.data(), t32.size() * sizeof(float)));
  if (dev >= (int)g_tw_ready.size()) g_tw_ready.resize(dev + 1, 0);
  g_tw_ready[dev] = 1;
  return TP_OK;
}

// --------------------------------------------------------------------------
// In-register complex FFT of length M (decimation in time).
// --------------------------------------------------------------------------
constexpr int radix_of(int M) {
  return (M % 4 == 0) ? 4 : (M % 2 == 0) ? 2 : (M % 5 == 0) ? 5 : (M % 3 == 0) ? 3 : M;
}

template <typename T, int M>
__device__ __forceinline__ void cfft(T (&re)[M], T (&im)[M]) {
  if constexpr (M > 1) {
    static_assert(tw_offset(M) >= 0, "no twiddle table for this transform length");
    constexpr int p = radix_of(M);
    constexpr int Q = M / p;
    T sr[p][Q], si[p][Q];
#pragma unroll
    for (int r = 0; r < p; ++r)
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        sr[r][q] = re[q * p + r];
        si[r][q] = im[q * p + r];
      }
#pragma unroll
    for (int r = 0; r < p; ++r) cfft<T, Q>(sr[r], si[r]);
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      T tr[p], ti[p];
#pragma unroll
      for (int r = 0; r < p; ++r) {
        const int e = (r * k) % M;
        if (e == 0) {
          tr[r] = sr[r][k];
          ti[r] = si[r][k];
        } else {
          const T wr = tw_re<T>(M, e), wi = tw_im<T>(M, e);
          tr[r] = sr[r][k] * wr - si[r][k] * wi;
          ti[r] = sr[r][k] * wi + si[r][k] * wr;
        }
      }
      if constexpr (p == 2) {
        re[k] = tr[0] + tr[1];
        im[k] = ti[0] + ti[1];
        re[k + Q] = tr[0] - tr[1];
        im[k + Q] = ti[0] - ti[1];
      } else if constexpr (p == 4) {
        const T ar = tr[0] + tr[2], ai = ti[0] + ti[2];
        const T br = tr[0] - tr[2], bi = ti[0] - ti[2];
        const T cr = tr[1] + tr[3], ci = ti[1] + ti[3];
        // (t1 - t3) * (-i)
        const T dr = ti[1] - ti[3], di = tr[3] - tr[1];
        re[k] = ar + cr;
        im[k] = ai + ci;
        re[k + 2 * Q] = ar - cr;
        im[k + 2 * Q] = ai - ci;
        re[k + Q] = br + dr;
        im[k + Q] = bi + di;
        re[k + 3 * Q] = br - dr;
        im[k + 3 * Q] = bi - di;
      } else {
        // generic p-point DFT with W_p^{rs} = W_M^{r s Q}
#pragma unroll
        for (int s = 0; s < p; ++s) {
          T accr = tr[0], acci = ti[0];
#pragma unroll
          for (int r = 1; r < p; ++r) {
            const int e = (r * s * Q) % M;
            if (e == 0) {
              accr += tr[r];
              acci += ti[r];
            } else {
              const T wr = tw_re<T>(M, e), wi = tw_im<T>(M, e);
              accr += tr[r] * wr - ti[r] * wi;
              acci += tr[r] * wi + ti[r] * wr;
            }
          }
          re[k + s * Q] = accr;
          im[k + s * Q] = acci;
        }
      }
    }
  }
}

template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
  using type = float4;
  static constexpr int n = 4;
};
template <>
struct Vec16<double> {
  using type = double2;
  static constexpr int n = 2;
};

constexpr int kTile = 64;  // tubes per workgroup (one wavefront)

// Output of one spectrum value: planar float (re, im planes [k][slot]) or,
// with SPLIT, four bf16 planes [p][k][slot] = hi(re), lo(re), hi(im), lo(im)
// (hi = round-to-nearest-even bf16 of x, lo = bf16 of x - hi), the operand
// format of the matrix-core products.
template <typename T, bool SPLIT>
__device__ __forceinline__ void emit(T* ore, T* oim, int64_t K, int64_t ks, int64_t k, int64_t t, T vr, T vi) {
  if constexpr (SPLIT) {
    __bf16* b = reinterpret_cast<__bf16*>(ore);
    const __bf16 hr = (__bf16)vr, hi = (__bf16)vi;
    const int64_t ps = K * ks, o = k * ks + t;
    b[o] = hr;
    b[ps + o] = (__bf16)(vr - (float)hr);
    b[2 * ps + o] = hi;
    b[3 * ps + o] = (__bf16)(vi - (float)hi);
  } else {
    ore[k * ks + t] = vr;
    oim[k * ks + t] = vi;
  }
}

// Long tubes are staged through LDS in two halves (HALF): half the LDS per
// workgroup, so twice as many wavefronts fit on a compute unit to hide the
// memory latency of this HBM-bound kernel; each lane picks its half tube out
// of LDS between the two stagings.
template <typename T, int N, bool SPLIT = false>
__global__ __launch_bounds__(kTile) void rfft_kernel(const T* __restrict__ x, FwdArgs a, T* __restrict__ ore,
                                                     T* __restrict__ oim) {
  const int64_t b = blockIdx.x;
#include "fft_packed.inc"
}

// One operand of a launch that transforms two: a product's first step is two
// transforms that do not depend on each other, each shorter than its launch
// where the product is small (64 x 48 times 48 x 32, n3 = 16, float64: 24.8 ->
// 21.6 us the whole t-product).
template <typename T>
struct Operand {
  const T* x;
  FwdArgs a;
  T *re, *im;
};
// (a uniform choice of arguments, no second copy of the code)
template <typename T>
__device__ __forceinline__ Operand<T> choose(const Operand<T>& p, const Operand<T>& q, int64_t np, int64_t& b) {
  b = blockIdx.x;
  const bool second = b >= np;
  if (second) b -= np;
  return second ? q : p;
}

template <typename T, int N>
__global__ __launch_bounds__(kTile) void rfft_pair_kernel(Operand<T> p, int64_t np, Operand<T> q) {
  constexpr bool SPLIT = false;
  int64_t b;
  const Operand<T> o = choose(p, q, np, b);
  const T* __restrict__ x = o.x;
  const FwdArgs a = o.a;
  T* __restrict__ ore = o.re;
  T* __restrict__ oim = o.im;
#include "fft_packed.inc"
}

// Short lengths without a packed kernel: one tube per thread, the length-N
// transform of fft_stages.hpp in float64 registers with a zero imaginary part
// (folded away by the compiler), each thread reading its whole tube at once.
// Bound by HBM: 3e7 values of n = 5 float32 tubes take 40 us forward and 38
// back (6.6 TB/s; a direct sum per output 86 / 85, the LDS stages 176 / 129).
template <typename T, int N>
struct Tube {
  T v[N];
};
constexpr int kSmallNT = 256;

template <typename T, int N>
__device__ __forceinline__ void rfft_small_body(const T* __restrict__ x, const FwdArgs& a, T* __restrict__ ore,
                                                T* __restrict__ oim, int64_t b) {
  const int64_t t = b * kSmallNT + threadIdx.x, ks = a.ntubes;
  if (t >= ks) return;
  int64_t src;
  double s;
  double r[N], i[N];
  const bool live = tube_source(a, t, src, s);
  Tube<T, N> w = {};
  if (live) __builtin_memcpy(&w, x + src * N, sizeof(w));
#pragma unroll
  for (int e = 0; e < N; ++e) {
    r[e] = (!live || s == 1.0) ? (double)w.v[e] : (double)(T)((double)w.v[e] * s);
    i[e] = 0.0;
  }
  lfft::dft<N>(r, i);
#pragma unroll
  for (int k = 0; k <= N / 2; ++k) {
    ore[k * ks + t] = (T)r[k];
    oim[k * ks + t] = (k == 0 || 2 * k == N) ? T(0) : (T)i[k];
  }
}

template <typename T, int N>
__global__ __launch_bounds__(kSmallNT) void rfft_small_kernel(const T* __restrict__ x, FwdArgs a, T* __restrict__ ore,
                                                              T* __restrict__ oim) {
  rfft_small_body<T, N>(x, a, ore, oim, blockIdx.x);
}

template <typename T, int N>
__global__ __launch_bounds__(kSmallNT) void rfft_small_pair_kernel(Operand<T> p, int64_t np, Operand<T> q) {
  int64_t b;
  const Operand<T> o = choose(p, q, np, b);
  rfft_small_body<T, N>(o.x, o.a, o.re, o.im, b);
}

template <typename T, int N>
__global__ __launch_bounds__(kSmallNT) void irfft_small_kernel(const T* __restrict__ xre, const T* __restrict__ xim,
                                                               int64_t ks, T* __restrict__ y) {
  const int64_t t = (int64_t)blockIdx.x * kSmallNT + threadIdx.x;
  if (t >= ks) return;
  // the forward transform of the conjugated Hermitian extension is real
  double r[N], i[N];
#pragma unroll
  for (int k = 0; k <= N / 2; ++k) {
    const bool real = k == 0 || 2 * k == N;
    r[k] = (double)xre[k * ks + t];
    i[k] = real ? 0.0 : -(double)xim[k * ks + t];
    if (!real) {
      r[N - k] = r[k];
      i[N - k] = -i[k];
    }
  }
  lfft::dft<N>(r, i);
  Tube<T, N> w;
#pragma unroll
  for (int e = 0; e < N; ++e) w.v[e] = (T)(r[e] / (double)N);
  __builtin_memcpy(y + t * N, &w, sizeof(w));
}

// Output staging of the inverse transform: the 64 tubes of a workgroup are
// transposed through LDS in NH pieces of N / NH entries (two for the longer
// tubes, which halves the LDS a workgroup holds and doubles the workgroups
// that fit on a CU).
template <int N>
struct InvStage {
  static constexpr int VN = 4;
  static constexpr int NH = (N >= 64 && N % (2 * VN) == 0) ? 2 : 1;
  static constexpr int SPAN = N / NH;
  static constexpr int PAD = SPAN + 1;
};

template <typename T, int N>
__global__ __launch_bounds__(kTile) void irfft_kernel(const T* __restrict__ xre, const T* __restrict__ xim,
                                                      int64_t ntubes, T* __restrict__ y) {
  constexpr int M = N / 2;
  static_assert(N <= 2 || tw_offset(N) >= 0, "no twiddle table for this tube length");
  using ST = InvStage<N>;
  constexpr int NH = ST::NH, SPAN = ST::SPAN, PAD = ST::PAD;
  constexpr int VN = Vec16<T>::n;
  using V = typename Vec16<T>::type;
  __shared__ T lds[kTile * PAD];
  const int lane = threadIdx.x;
  const int64_t tile0 = (int64_t)blockIdx.x * kTile;
  const int64_t t = tile0 + lane;
  const int64_t ks = ntubes;
  // the time-domain tube of this lane: y[2 m] = zr[m], y[2 m + 1] = zi[m]
  // once the transform is done (y[0] = zr[0] for N = 1)
  constexpr int MZ = M > 0 ? M : 1;
  T zr[MZ], zi[MZ];
  if (t < ntubes) {
    if constexpr (N == 1) {
      zr[0] = xre[t];
    } else {
      // the half spectrum is read into zr / zi and turned into conj(Z),
      // Z[k] = E[k] + i O[k], in place: slot k takes X[k] for k < M and
      // X[M] is held apart; the pair (k, M - k) is rewritten together
#pragma unroll
      for (int k = 0; k < M; ++k) {
        zr[k] = xre[(int64_t)k * ks + t];
        zi[k] = k == 0 ? T(0) : xim[(int64_t)k * ks + t];
      }
      const T xmr = xre[(int64_t)M * ks + t];
      auto zpart = [&](int k, T xkr, T xki, T xjr, T xji, T& outr, T& outi) {
        const T er = (xkr + xjr) * T(0.5), ei = (xki - xji) * T(0.5);
        const T dr = (xkr - xjr) * T(0.5), di = (xki + xji) * T(0.5);
        // O = d * conj(W_N^k); Z = E + i O; store conj(Z)
        const T wr = tw_re<T>(N, k), wi = -tw_im<T>(N, k);
        const T orr = dr * wr - di * wi, oi = dr * wi + di * wr;
        outr = er - oi;
        outi = -(ei + orr);
      };
      {
        // k = 0 pairs with X[M] (imaginary parts of both are dropped)
        T o0r, o0i;
        zpart(0, zr[0], T(0), xmr, T(0), o0r, o0i);
        zr[0] = o0r;
        zi[0] = o0i;
      }
#pragma unroll
      for (int k = 1; k <= M / 2; ++k) {
        const int j = M - k;
        const T xkr = zr[k], xki = zi[k], xjr = zr[j], xji = zi[j];
        T okr, oki, ojr, oji;
        zpart(k, xkr, xki, xjr, xji, okr, oki);
        zpart(j, xjr, xji, xkr, xki, ojr, oji);
        zr[k] = okr;
        zi[k] = oki;
        zr[j] = ojr;
        zi[j] = oji;
      }
      cfft<T, M>(zr, zi);
      const T inv = T(1) / T(M);
#pragma unroll
      for (int m = 0; m < M; ++m) {
        zr[m] = zr[m] * inv;
        zi[m] = -zi[m] * inv;
      }
    }
  }
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    if (h > 0) __syncthreads();
    if (t < ntubes) {
#pragma unroll
      for (int e = 0; e < SPAN; ++e) {
        const int g = h * SPAN + e;  // entry of the tube
        lds[lane * PAD + e] = (g & 1) ? zi[g >> 1] : zr[g >> 1];
      }
    }
    __syncthreads();
    if constexpr (SPAN % VN == 0) {
      constexpr int CH = SPAN / VN;
#pragma unroll
      for (int it = 0; it < CH; ++it) {
        const int f = it * kTile + lane;
        const int tl = f / CH, part = f - tl * CH;
        const int64_t tt = tile0 + tl;
        if (tt < ntubes) {
          V w;
          T* wp = reinterpret_cast<T*>(&w);
#pragma unroll
          for (int e = 0; e < VN; ++e) wp[e] = lds[tl * PAD + part * VN + e];
          *reinterpret_cast<V*>(y + tt * N + h * SPAN + part * VN) = w;
        }
      }
    } else {
      for (int it = 0; it < SPAN; ++it) {
        const int f = it * kTile + lane;
        const int tl = f / SPAN, e = f - tl * SPAN;
        const int64_t tt = tile0 + tl;
        if (tt < ntubes) y[tt * N + h * SPAN + e] = lds[tl * PAD + e];
      }
    }
  }
}

// Direct transforms for lengths without a specialised kernel. Every term
// uses a root exp(-2 pi i m / N) with m = k n mod N; up to kDirectTable
// points the N roots are evaluated once per workgroup into LDS (the same
// sincospi values the direct formula takes), beyond that per term.
constexpr int kDirectTable = 2048;

template <bool TABLE>
__device__ __forceinline__ void direct_root(const double* tw, int m, int N, double& sn, double& cs) {
  if (TABLE) {
    cs = tw[m];
    sn = tw[N + m];
  } else {
    sincospi(2.0 * (double)m / (double)N, &sn, &cs);
  }
}

__device__ __forceinline__ void direct_table(double* tw, int N) {
  for (int m = threadIdx.x; m < N; m += blockDim.x) {
    double sn, cs;
    sincospi(2.0 * (double)m / (double)N, &sn, &cs);
    tw[m] = cs;
    tw[N + m] = sn;
  }
  __syncthreads();
}

template <typename T, bool TABLE>
__global__ void rdft_direct_kernel(const T* __restrict__ x, int N, FwdArgs a, T* __restrict__ ore,
                                   T* __restrict__ oim) {
  extern __shared__ double tw[];  // TABLE: cos, then sin, of 2 pi m / N
  if (TABLE) direct_table(tw, N);
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= a.ntubes) return;
  const int K = N / 2 + 1;
  int64_t src;
  double s;
  const bool live = tube_source(a, t, src, s);
  for (int k = 0; k < K; ++k) {
    double accr = 0, acci = 0;
    if (live) {
      int m = 0;  // k n mod N
      for (int n = 0; n < N; ++n) {
        double sn, cs;
        direct_root<TABLE>(tw, m, N, sn, cs);
        const double v = (double)(T)((double)x[src * N + n] * s);
        accr += v * cs;
        acci -= v * sn;
        m += k;
        m = m >= N ? m - N : m;
      }
    }
    ore[(int64_t)k * a.ntubes + t] = (T)accr;
    oim[(int64_t)k * a.ntubes + t] = (k == 0 || 2 * k == N) ? T(0) : (T)acci;
  }
}

template <typename T, bool TABLE>
__global__ void irdft_direct_kernel(const T* __restrict__ xre, const T* __restrict__ xim, int N, int64_t ntubes,
                                    T* __restrict__ y) {
  extern __shared__ double tw[];
  if (TABLE) direct_table(tw, N);
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ntubes) return;
  const int K = N / 2 + 1;
  for (int n = 0; n < N; ++n) {
    double acc = 0;
    int m = 0;  // k n mod N
    for (int k = 0; k < K; ++k) {
      const double wk = (k == 0 || 2 * k == N) ? 1.0 : 2.0;
      double sn, cs;
      direct_root<TABLE>(tw, m, N, sn, cs);
      const double xr = (double)xre[(int64_t)k * ntubes + t];
      const double xi = (k == 0 || 2 * k == N) ? 0.0 : (double)xim[(int64_t)k * ntubes + t];
      acc += wk * (xr * cs - xi * sn);
      m += n;
      m = m >= N ? m - N : m;
    }
    y[t * N + n] = (T)(acc / N);
  }
}

// shortest length that the four-step transform takes
constexpr int64_t kLongMin = 257;

template <typename T>
using FwdKernel = void (*)(const T*, FwdArgs, T*, T*);
template <typename T>
using PairKernel = void (*)(Operand<T>, int64_t, Operand<T>);
template <typename T>
using InvKernel = void (*)(const T*, const T*, int64_t, T*);

template <typename T>
FwdKernel<T> pick_fwd(int64_t n) {
  switch (n) {
    case 1: return rfft_kernel<T, 1>;
    case 2: return rfft_kernel<T, 2>;
    case 4: return rfft_kernel<T, 4>;
    case 8: return rfft_kernel<T, 8>;
    case 16: return rfft_kernel<T, 16>;
    case 32: return rfft_kernel<T, 32>;
    case 64: return rfft_kernel<T, 64>;
    case 128: return rfft_kernel<T, 128>;
    case 10: return rfft_kernel<T, 10>;
    case 20: return rfft_kernel<T, 20>;
    case 50: return rfft_kernel<T, 50>;
    case 100: return rfft_kernel<T, 100>;
    case 168: return rfft_kernel<T, 168>;
    default: return nullptr;
  }
}

template <typename T>
InvKernel<T> pick_inv(int64_t n) {
  switch (n) {
    case 1: return irfft_kernel<T, 1>;
    case 2: return irfft_kernel<T, 2>;
    case 4: return irfft_kernel<T, 4>;
    case 8: return irfft_kernel<T, 8>;
    case 16: return irfft_kernel<T, 16>;
    case 32: return irfft_kernel<T, 32>;
    case 64: return irfft_kernel<T, 64>;
    case 128: return irfft_kernel<T, 128>;
    case 10: return irfft_kernel<T, 10>;
    case 20: return irfft_kernel<T, 20>;
    case 50: return irfft_kernel<T, 50>;
    case 100: return irfft_kernel<T, 100>;
    case 168: return irfft_kernel<T, 168>;
    default: return nullptr;
  }
}

template <typename T>
FwdKernel<T> pick_small_fwd(int64_t n) {
  switch (n) {
    case 3: return rfft_small_kernel<T, 3>;
    case 5: return rfft_small_kernel<T, 5>;
    case 6: return rfft_small_kernel<T, 6>;
    case 7: return rfft_small_kernel<T, 7>;
    case 9: return rfft_small_kernel<T, 9>;
    case 11: return rfft_small_kernel<T, 11>;
    case 12: return rfft_small_kernel<T, 12>;
    case 13: return rfft_small_kernel<T, 13>;
    case 14: return rfft_small_kernel<T, 14>;
    case 15: return rfft_small_kernel<T, 15>;
    case 17: return rfft_small_kernel<T, 17>;
    case 19: return rfft_small_kernel<T, 19>;
    case 23: return rfft_small_kernel<T, 23>;
    default: return nullptr;
  }
}

template <typename T>
PairKernel<T> pick_pair(int64_t n) {
  switch (n) {
    case 1: return rfft_pair_kernel<T, 1>;
    case 2: return rfft_pair_kernel<T, 2>;
    case 4: return rfft_pair_kernel<T, 4>;
    case 8: return rfft_pair_kernel<T, 8>;
    case 16: return rfft_pair_kernel<T, 16>;
    case 32: return rfft_pair_kernel<T, 32>;
    case 64: return rfft_pair_kernel<T, 64>;
    case 128: return rfft_pair_kernel<T, 128>;
    case 10: return rfft_pair_kernel<T, 10>;
    case 20: return rfft_pair_kernel<T, 20>;
    case 50: return rfft_pair_kernel<T, 50>;
    case 100: return rfft_pair_kernel<T, 100>;
    case 168: return rfft_pair_kernel<T, 168>;
    default: return nullptr;
  }
}

template <typename T>
PairKernel<T> pick_small_pair(int64_t n) {
  switch (n) {
    case 3: return rfft_small_pair_kernel<T, 3>;
    case 5: return rfft_small_pair_kernel<T, 5>;
    case 6: return rfft_small_pair_kernel<T, 6>;
    case 7: return rfft_small_pair_kernel<T, 7>;
    case 9: return rfft_small_pair_kernel<T, 9>;
    case 11: return rfft_small_pair_kernel<T, 11>;
    case 12: return rfft_small_pair_kernel<T, 12>;
    case 13: return rfft_small_pair_kernel<T, 13>;
    case 14: return rfft_small_pair_kernel<T, 14>;
    case 15: return rfft_small_pair_kernel<T, 15>;
    case 17: return rfft_small_pair_kernel<T, 17>;
    case 19: return rfft_small_pair_kernel<T, 19>;
    case 23: return rfft_small_pair_kernel<T, 23>;
    default: return nullptr;
  }
}

template <typename T>
InvKernel<T> pick_small_inv(int64_t n) {
  switch (n) {
    case 3: return irfft_small_kernel<T, 3>;
    case 5: return irfft_small_kernel<T, 5>;
    case 6: return irfft_small_kernel<T, 6>;
    case 7: return irfft_small_kernel<T, 7>;
    case 9: return irfft_small_kernel<T, 9>;
    case 11: return irfft_small_kernel<T, 11>;
    case 12: return irfft_small_kernel<T, 12>;
    case 13: return irfft_small_kernel<T, 13>;
    case 14: return irfft_small_kernel<T, 14>;
    case 15: return irfft_small_kernel<T, 15>;
    case 17: return irfft_small_kernel<T, 17>;
    case 19: return irfft_small_kernel<T, 19>;
    case 23: return irfft_small_kernel<T, 23>;
    default: return nullptr;
  }
}

template <typename T>
struct TypeOf;
template <>
struct TypeOf<float> {
  static constexpr int dtype = TP_F32;
};
template <>
struct TypeOf<double> {
  static constexpr int dtype = TP_F64;
};

// longest tube of fft_lds.hip and fft_dense.hip
template <typename T>
constexpr int64_t lds_max() {
  return 32768 / (int64_t)sizeof(T);
}

FwdArgs planar_args(const TubeGather& g) {
  return {g.rows, g.cols, g.in_cols, g.rows * g.cols, g.row_idx, g.col_idx, g.row_scale, g.col_scale, g.count,
          g.cols, 0, 0};
}

// Both operands in one launch, for the lengths whose kernel gives a tube to a
// thread; *handled is false for the others.
template <typename T>
int pair_impl(const T* x, const TubeGather& g, T* re, T* im, const T* y, const TubeGather& h, T* yre, T* yim,
              int64_t n3, hipStream_t st, bool* handled) {
  const Operand<T> p{x, planar_args(g), re, im}, q{y, planar_args(h), yre, yim};
  const bool packed = pick_pair<T>(n3) != nullptr;
  const auto k = packed ? pick_pair<T>(n3) : pick_small_pair<T>(n3);
  const int64_t nt = packed ? kTile : kSmallNT, np = (p.a.ntubes + nt - 1) / nt, nq = (q.a.ntubes + nt - 1) / nt;
  // (a launch holds 2^32 work-items: beyond, each operand has its own)
  *handled = k && np + nq > 0 && (np + nq) * nt < int64_t(1) << 32;
  if (!*handled) return TP_OK;
  hipLaunchKernelGGL(k, dim3((unsigned)(np + nq)), dim3((unsigned)nt), 0, st, p, np, q);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

template <typename T>
int fwd_impl(const T* x, int64_t n3, const TubeGather& g, T* re, T* im, hipStream_t st, bool sums) {
  const FwdArgs a = planar_args(g);
  if (a.ntubes == 0) return TP_OK;
  sums = sums && n3 < kLongMin;
  if (auto k = pick_fwd<T>(n3)) {
    const int64_t blocks = (a.ntubes + kTile - 1) / kTile;
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(kTile), 0, st, x, a, re, im);
  } else if (auto k = pick_small_fwd<T>(n3); k && !sums) {
    const int64_t blocks = (a.ntubes + kSmallNT - 1) / kSmallNT;
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(kSmallNT), 0, st, x, a, re, im);
  } else {
    bool handled = false;
    if (n3 <= lds_max<T>() && !sums) {
      if (int rc = lds_forward(x, TypeOf<T>::dtype, n3, a, re, im, st, &handled)) return rc;
      return handled ? TP_OK : dense_forward(x, TypeOf<T>::dtype, n3, a, re, im, st);
    }
    if (n3 >= kLongMin)
      if (int rc = four_forward(x, TypeOf<T>::dtype, n3, a, re, im, st, &handled)) return rc;
    if (handled) return TP_OK;
    const int64_t blocks = (a.ntubes + 127) / 128;
    if (n3 <= kDirectTable)
      hipLaunchKernelGGL((rdft_direct_kernel<T, true>), dim3((unsigned)blocks), dim3(128), 2 * n3 * sizeof(double), st,
                         x, (int)n3, a, re, im);
    else
      hipLaunchKernelGGL((rdft_direct_kernel<T, false>), dim3((unsigned)blocks), dim3(128), 0, st, x, (int)n3, a, re,
                         im);
  }
  TP_LAUNCH_CHECK();
  return TP_OK;
}

template <typename T>
int inv_impl(const T* re, const T* im, int64_t n3, int64_t ntubes, T* y, hipStream_t st, bool sums) {
  if (ntubes == 0) return TP_OK;
  sums = sums && n3 < kLongMin;
  if (auto k = pick_inv<T>(n3)) {
    const int64_t blocks = (ntubes + kTile - 1) / kTile;
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(kTile), 0, st, re, im, ntubes, y);
  } else if (auto k = pick_small_inv<T>(n3); k && !sums) {
    const int64_t blocks = (ntubes + kSmallNT - 1) / kSmallNT;
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(kSmallNT), 0, st, re, im, ntubes, y);
  } else {
    bool handled = false;
    if (n3 <= lds_max<T>() && !sums) {
      if (int rc = lds_inverse(re, im, TypeOf<T>::dtype, n3, ntubes, y, st, &handled)) return rc;
      return handled ? TP_OK : dense_inverse(re, im, TypeOf<T>::dtype, n3, ntubes, y, st);
    }
    if (n3 >= kLongMin)
      if (int rc = four_inverse(re, im, TypeOf<T>::dtype, n3, ntubes, y, st, &handled)) return rc;
    if (handled) return TP_OK;
    const int64_t blocks = (ntubes + 127) / 128;
    if (n3 <= kDirectTable)
      hipLaunchKernelGGL((irdft_direct_kernel<T, true>), dim3((unsigned)blocks), dim3(128), 2 * n3 * sizeof(double),
                         st, re, im, (int)n3, ntubes, y);
    else
      hipLaunchKernelGGL((irdft_direct_kernel<T, false>), dim3((unsigned)blocks), dim3(128), 0, st, re, im, (int)n3,
                         ntubes, y);
  }
  TP_LAUNCH_CHECK();
  return TP_OK;
}

template <bool SPLIT>
FwdKernel<float> pick_fwd_split(int64_t n) {
  switch (n) {
    case 1: return rfft_kernel<float, 1, true>;
    case 2: return rfft_kernel<float, 2, true>;
    case 4: return rfft_kernel<float, 4, true>;
    case 8: return rfft_kernel<float, 8, true>;
    case 16: return rfft_kernel<float, 16, true>;
    case 32: return rfft_kernel<float, 32, true>;
    case 64: return rfft_kernel<float, 64, true>;
    case 128: return rfft_kernel<float, 128, true>;
    case 10: return rfft_kernel<float, 10, true>;
    case 20: return rfft_kernel<float, 20, true>;
    case 50: return rfft_kernel<float, 50, true>;
    case 100: return rfft_kernel<float, 100, true>;
    default: return nullptr;
  }
}

}  // namespace

bool fft_supported(int64_t n3) { return pick_fwd<float>(n3) != nullptr; }

bool fft_split_supported(int64_t n3) { return pick_fwd_split<true>(n3) != nullptr; }

int fft_forward_split(const float* x, int64_t n3, const TubeGather& g, bool colmajor, int64_t ld, void* planes,
                      hipStream_t st) {
  if (int rc = ensure_twiddles()) return rc;
  auto k = pick_fwd_split<true>(n3);
  if (!k) return fail(TP_EUNSUPPORTED, "no split-output transform for this tube length");
  if (ld < (colmajor ? g.rows : g.cols)) return fail(TP_EINVAL, "split spectrum stride below its extent");
  FwdArgs a{g.rows, g.cols, g.in_cols, (colmajor ? g.cols : g.rows) * ld, g.row_idx, g.col_idx, g.row_scale,
            g.col_scale, g.count, ld, colmajor ? 1 : 0, (colmajor && ld % kTile == 0) ? g.cols : 0};
  if (a.ntubes == 0) return TP_OK;
  const int64_t blocks = (a.ntubes + kTile - 1) / kTile;
  if (blocks > 0x7fffffffLL) return fail(TP_EUNSUPPORTED, "too many tubes");
  hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(kTile), 0, st, x, a, (float*)planes, (float*)nullptr);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int fft_forward(const void* x, int dtype, int64_t n3, const TubeGather& g, void* re, void* im, hipStream_t st,
                bool sums) {
  if (int rc = ensure_twiddles()) return rc;
  if ((g.rows * g.cols + kTile - 1) / kTile > 0x7fffffffLL) return fail(TP_EUNSUPPORTED, "too many tubes");
  if (dtype == TP_F64)
    return fwd_impl<double>((const double*)x, n3, g, (double*)re, (double*)im, st, sums);
  return fwd_impl<float>((const float*)x, n3, g, (float*)re, (float*)im, st, sums);
}

int fft_forward_pair(const void* x, const TubeGather& g, void* re, void* im, const void* y, const TubeGather& h,
                     void* yre, void* yim, int dtype, int64_t n3, hipStream_t st) {
  if (int rc = ensure_twiddles()) return rc;
  bool handled = false;
  if (dtype == TP_F64) {
    if (int rc = pair_impl<double>((const double*)x, g, (double*)re, (double*)im, (const double*)y, h, (double*)yre,
                                   (double*)yim, n3, st, &handled))
      return rc;
  } else {
    if (int rc = pair_impl<float>((const float*)x, g, (float*)re, (float*)im, (const float*)y, h, (float*)yre,
                                  (float*)yim, n3, st, &handled))
      return rc;
  }
  if (handled) return TP_OK;
  if (int rc = fft_forward(x, dtype, n3, g, re, im, st)) return rc;
  return fft_forward(y, dtype, n3, h, yre, yim, st);
}

int fft_inverse(const void* re, const void* im, int dtype, int64_t n3, int64_t rows, int64_t cols, void* x,
                hipStream_t st, bool sums) {
  if (int rc = ensure_twiddles()) return rc;
  if (dtype == TP_F64)
    return inv_impl<double>((const double*)re, (const double*)im, n3, rows * cols, (double*)x, st, sums);
  return inv_impl<float>((const float*)re, (const float*)im, n3, rows * cols, (float*)x, st, sums);
}

}  // namespace tp
