// Tube transforms of lengths that have a prime factor above 13 (in n, or n / 2 of
// an even n), up to what fft_lds.hip takes otherwise: dense products with the
// roots of unity on the float64 matrix cores.
//
// An odd length is one sequence (R = 1) of N = n values, an even one two (R = 2) of
// N = n / 2, the even and the odd values. With H = N / 2 + 1 and a sequence folded
// about its middle, P[u] = x[u] + x[N-u], Q[u] = x[u] - x[N-u] (u < H; at u = 0 and
// N / 2 the value alone and 0), its transform is
//   Y[k] = sum_u P[u] cos(2 pi u k / N) - i sum_u Q[u] sin(2 pi u k / N), k < H,
// and with P[k] = 2 Re Y[k], Q[k] = 2 Im Y[k] (at k = 0, N / 2 the value alone and 0)
//   N x[m], N x[N-m] = sum_k P[k] cos(2 pi k m / N) -+ sum_k Q[k] sin(2 pi k m / N).
// Either way two real H x H matrices. Two sequences' transforms E, O make
// X[k], conj X[N-k] = E[k] +- W_n^k O[k], and 2 E[k] = X[k] + conj X[N-k],
// 2 O[k] = (X[k] - conj X[N-k]) W_n^-k.
//
// Four wavefronts own 16 WO outputs of 16 TT (4 / WO) tubes, each 16 outputs of TT
// blocks of 16 tubes. P and Q come in chunks of CC, loaded one chunk ahead into
// registers and folded into one of two LDS buffers; a lane reads its root, of index
// u k mod N, from a table of half a turn. Products are summed in blocks of 32 and
// the blocks one by one, so that the rounding of long sums stays small: relative
// error of float64 tubes 1.5e-16 (n = 29) to 2.8e-16 (2033), a direct sum's 2.4e-16
// (29) to 5.5e-16 (251), Bluestein's chirp-z transform in LDS 3.9e-16 to 6.1e-16.
//
// Bound: HBM up to n of about 150, then the float64 matrix cores (n^2 operations a
// tube, half of that in two sequences; 58 TFLOP/s from registers, 34 here at n =
// 997). 1.5e6 float64 values, us forward / inverse, direct sum and Bluestein /
// here: n = 29 40 / 66 and 115 / 110 -> 14 / 13, 127 642 / 943 and 92 / 87 -> 14 / 14,
// 254 1670 / 3542 and 66 / 64 -> 16 / 15, 1013 Bluestein 158 / 150 -> 58 / 56; 14640
// float32 tubes of 997, Bluestein 912 / 887 -> 424 / 384, of 2039 1880 / 1893 -> 1532 /
// 1375.
#include <algorithm>

#include "fft_stages.hpp"
#include "fft_tubes.hpp"

namespace tp {
namespace {

using lfft::Cx;

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int NT = 256;
constexpr int kBlock = 8;  // matrix instructions, of four terms each, a block of a sum
constexpr int64_t kLds = 160 * 1024;

template <int R, int WO, int TT>
struct Shape {
  static constexpr int TB = 16 * TT * (4 / WO);  // tubes a workgroup
  // terms a chunk: few tubes bring few products to hide a chunk's loads behind
  static constexpr int CC = TB == 16 ? 64 / R : 16;
  static constexpr int E = CC * TB / NT;  // a thread's
  // (rows of 1 mod 16 doubles: writes of neighbouring terms or tubes and the
  // fragment reads, 4 rows x 16 columns, spread evenly over the banks)
  struct Lds {
    double p[2][R][CC][TB + 1], q[2][R][CC][TB + 1];
    int64_t src[TB];
    double scl[TB];
  };
};

template <typename T>
struct DenseArgs {
  const T *x, *xim;  // tubes, or the spectrum's planes
  FwdArgs a;         // (forward)
  int64_t ks;        // tubes
  int n;
  T *y, *yim;  // the spectrum's planes, or tubes
};

template <typename T, int R>
struct Vals {
  T v[R];
};

template <typename T, int R, int WO, int TT, bool INV>
__global__ __launch_bounds__(NT, 2) void dense_kernel(DenseArgs<T> g) {
  using S = Shape<R, WO, TT>;
  constexpr int TB = S::TB, CC = S::CC, E = S::E;
  extern __shared__ __align__(16) unsigned char dense_lds[];
  typename S::Lds& sh = *reinterpret_cast<typename S::Lds*>(dense_lds);
  Cx<double>* tab = reinterpret_cast<Cx<double>*>(dense_lds + sizeof(typename S::Lds));
  const int n = g.n, N = n / R, H = N / 2 + 1, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int gr = lane >> 4, j = lane & 15;
  const int nob = (H + 16 * WO - 1) / (16 * WO), nch = (H + CC - 1) / CC;
  lfft::fill_roots(N, tab);  // exp(-2 pi i k / 2N), k < H
  XcdWalk walk((g.ks + TB - 1) / TB * nob);
  for (int64_t G; walk.next(G);) {
    const int64_t t0 = G / nob * TB;
    const int o0 = (int)(G % nob) * 16 * WO + 16 * (w % WO), tw = 16 * TT * (w / WO);
    if constexpr (!INV) {
      if (tid < TB) {
        int64_t src = 0;
        double s = 1.0;
        const bool ok = t0 + tid < g.ks && tube_source(g.a, t0 + tid, src, s);
        sh.src[tid] = ok ? src : -1;
        sh.scl[tid] = s;
      }
    }
    __syncthreads();
    // term c and tube t of a thread's value e: forward, lanes on a tube's
    // consecutive values; inverse, on a slice's consecutive tubes
    const auto place = [&](int e, int& c, int& t) {
      const int f = tid + e * NT;
      c = INV ? f / TB : f % CC;
      t = INV ? f % TB : f / CC;
    };
    // terms c and N - c as they are stored: R values each of a tube, or (re, im)
    // of slices c and, for R = 2, N - c (unconditional loads, clamped)
    Vals<T, 2> za[E], zb[E];
    const auto load = [&](int ch) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        int c, t;
        place(e, c, t);
        c += ch * CC;
        c = c < H ? c : H - 1;
        if constexpr (INV) {
          const int64_t tube = t0 + t < g.ks ? t0 + t : g.ks - 1, o = c * g.ks + tube, o2 = (N - c) * g.ks + tube;
          za[e] = {g.x[o], g.xim[o]};
          if (R == 2) zb[e] = {g.x[o2], g.xim[o2]};
        } else {
          const T* p = g.x + (sh.src[t] < 0 ? 0 : sh.src[t] * n);
          __builtin_memcpy(za[e].v, p + R * c, R * sizeof(T));
          __builtin_memcpy(zb[e].v, p + (c ? R * (N - c) : 0), R * sizeof(T));
        }
      }
    };
    const auto fold = [&](int ch) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        int row, t;
        place(e, row, t);
        const int c = row + ch * CC, b = ch & 1;
        const bool alone = c == 0 || 2 * c == N;
        double p[R], q[R];
        bool live = c < H;
        if constexpr (INV) {
          live = live && t0 + t < g.ks;
          const double xr = (double)za[e].v[0], xi = c == 0 ? 0.0 : (double)za[e].v[1];
          if constexpr (R == 1) {
            p[0] = alone ? xr : 2.0 * xr;
            q[0] = alone ? 0.0 : 2.0 * xi;
          } else {
            const double yr = (double)zb[e].v[0], yi = c == 0 ? 0.0 : (double)zb[e].v[1], h = alone ? 0.5 : 1.0;
            const Cx<double> r = tab[c < H ? c : H - 1];
            const double dr = h * (xr - yr), di = h * (xi + yi);
            p[0] = h * (xr + yr);
            q[0] = alone ? 0.0 : xi - yi;
            p[1] = dr * r.x + di * r.y;
            q[1] = alone ? 0.0 : di * r.x - dr * r.y;
          }
        } else {
          live = live && sh.src[t] >= 0;
          const double s = sh.scl[t];
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const double a = (double)za[e].v[r], z = (double)zb[e].v[r];
            const double x = s == 1.0 ? a : a * s, y = s == 1.0 ? z : z * s;
            p[r] = alone ? x : x + y;
            q[r] = alone ? 0.0 : x - y;
          }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          sh.p[b][r][row][t] = live ? p[r] : 0.0;
          sh.q[b][r][row][t] = live ? q[r] : 0.0;
        }
      }
    };
    const bool work = o0 < H;
    // the root's index of successive terms gr, gr + 4, gr + 8 ..
    const int oj = o0 + j < H ? o0 + j : H - 1, de = 4 * oj % N;
    int e = gr * oj % N;
    d4 cs[R][TT], sn[R][TT], ct[R][TT], st[R][TT];  // a block's sums, and the blocks'
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int t = 0; t < TT; ++t) cs[r][t] = sn[r][t] = ct[r][t] = st[r][t] = d4{0.0, 0.0, 0.0, 0.0};
    const auto close = [&]() {
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          ct[r][t] += cs[r][t];
          st[r][t] += sn[r][t];
          cs[r][t] = sn[r][t] = d4{0.0, 0.0, 0.0, 0.0};
        }
    };
    load(0);
    for (int ch = 0; ch < nch; ++ch) {
      fold(ch);
      // (this buffer's readers of two chunks ago have passed the last chunk's barrier)
      __syncthreads();
      if (ch + 1 < nch) load(ch + 1);
      if (!work) continue;
#pragma unroll
      for (int kk = 0; kk < CC / 4; ++kk) {
        double c, s;
        lfft::root_at(tab, N, e, c, s);
        e += de;
        e = e >= N ? e - N : e;
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const double p = sh.p[ch & 1][r][4 * kk + gr][tw + 16 * t + j];
            const double q = sh.q[ch & 1][r][4 * kk + gr][tw + 16 * t + j];
            cs[r][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(INV ? p : c, INV ? c : p, cs[r][t], 0, 0, 0);
            sn[r][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(INV ? q : s, INV ? s : q, sn[r][t], 0, 0, 0);
          }
        if (kk % kBlock == kBlock - 1) close();
      }
      if (CC / 4 < kBlock && (ch % (4 * kBlock / CC) == 4 * kBlock / CC - 1 || ch + 1 == nch)) close();
    }
    // lane: rows 4 v + gr of the first operand, column j of the second
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int o = o0 + (INV ? j : 4 * v + gr);
        const int64_t tube = t0 + tw + 16 * t + (INV ? 4 * v + gr : j);
        if (o >= H || tube >= g.ks) continue;
        const bool alone = o == 0 || 2 * o == N;
        if constexpr (INV) {
          T* y = g.y + tube * n;
          Vals<T, R> a, b;
#pragma unroll
          for (int r = 0; r < R; ++r) {
            a.v[r] = (T)((ct[r][t][v] + st[r][t][v]) / (double)N);
            b.v[r] = (T)((ct[r][t][v] - st[r][t][v]) / (double)N);
          }
          __builtin_memcpy(y + R * o, a.v, sizeof(a));
          if (!alone) __builtin_memcpy(y + R * (N - o), b.v, sizeof(b));
        } else if constexpr (R == 1) {
          g.y[o * g.ks + tube] = (T)ct[0][t][v];
          g.yim[o * g.ks + tube] = alone ? T(0) : (T)st[0][t][v];
        } else {
          const Cx<double> r = tab[o];
          const double er = ct[0][t][v], ei = alone ? 0.0 : st[0][t][v];
          const double zr = ct[1][t][v], zi = alone ? 0.0 : st[1][t][v];
          const double pr = zr * r.x - zi * r.y, pi = zr * r.y + zi * r.x;
          g.y[o * g.ks + tube] = (T)(er + pr);
          g.yim[o * g.ks + tube] = o == 0 ? T(0) : (T)(ei + pi);
          if (2 * o != N) {
            g.y[(N - o) * g.ks + tube] = (T)(er - pr);
            g.yim[(N - o) * g.ks + tube] = o == 0 ? T(0) : (T)(pi - ei);
          }
        }
      }
    // before the next tile's chunk 0 and sources overwrite what a slower
    // wavefront of this one still reads
    __syncthreads();
  }
}

template <typename T, int R, int WO, int TT, bool INV>
int launch_dense(const DenseArgs<T>& g, hipStream_t st) {
  using S = Shape<R, WO, TT>;
  const int H = g.n / R / 2 + 1;
  const size_t lds = sizeof(typename S::Lds) + sizeof(Cx<double>) * H;
  const int64_t tiles = (g.ks + S::TB - 1) / S::TB * ((H + 16 * WO - 1) / (16 * WO));
  const int64_t per_cu = std::min<int64_t>(kLds / (int64_t)lds, R * TT >= 4 ? 2 : 4);
  hipLaunchKernelGGL((dense_kernel<T, R, WO, TT, INV>), dim3((unsigned)xcd_grid(std::min(tiles, 256 * per_cu))),
                     dim3(NT), lds, st, g);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

// Blocks of outputs by their number, and 64 (two sequences: 32) tubes a workgroup,
// or 16, whose products share a root and the folded values among fewer (about 1.15
// times the time per product), where that leaves fewer rounds over the 256 CUs, or
// 64 not more than one workgroup a CU: float64 tubes of 2039, 1100 of them 214 us
// with 64 and 148 with 16, 2000 221 and 233; of 509, 2000 42 and 24.
template <typename T, bool INV>
int dense(const DenseArgs<T>& g, hipStream_t st) {
  const bool even = g.n % 2 == 0;
  const int H = g.n / (even ? 4 : 2) + 1;
  const int64_t tubes = even ? 32 : 64, blocks = (H + 63) / 64;
  const int64_t wide = (g.ks + tubes - 1) / tubes * blocks, narrow = (g.ks + 15) / 16 * blocks;
  const bool few = wide <= 256 || 23 * ((narrow + 255) / 256) < 20 * (tubes / 16) * ((wide + 255) / 256);
  if (even) {
    if (H <= 32) return launch_dense<T, 2, 2, 1, INV>(g, st);
    return few ? launch_dense<T, 2, 4, 1, INV>(g, st) : launch_dense<T, 2, 4, 2, INV>(g, st);
  }
  if (H <= 16) return launch_dense<T, 1, 1, 1, INV>(g, st);
  if (H <= 32) return launch_dense<T, 1, 2, 2, INV>(g, st);
  return few ? launch_dense<T, 1, 4, 1, INV>(g, st) : launch_dense<T, 1, 4, 4, INV>(g, st);
}

}  // namespace

int dense_forward(const void* x, int dtype, int64_t n3, const FwdArgs& a, void* re, void* im, hipStream_t st) {
  if (dtype == TP_F64)
    return dense<double, false>({(const double*)x, nullptr, a, a.ntubes, (int)n3, (double*)re, (double*)im}, st);
  return dense<float, false>({(const float*)x, nullptr, a, a.ntubes, (int)n3, (float*)re, (float*)im}, st);
}

int dense_inverse(const void* re, const void* im, int dtype, int64_t n3, int64_t ntubes, void* y, hipStream_t st) {
  if (dtype == TP_F64)
    return dense<double, true>({(const double*)re, (const double*)im, {}, ntubes, (int)n3, (double*)y, nullptr}, st);
  return dense<float, true>({(const float*)re, (const float*)im, {}, ntubes, (int)n3, (float*)y, nullptr}, st);
}

}  // namespace tp
