// Short complex transforms in registers and the mixed-radix transform of
// many sequences in LDS built on them (used by the tube transforms of
// fft_lds.hip and by the four-step transform of fft_four.hip).
//
// The butterflies' type is that of the root table: float64 for the tubes in
// LDS, also float ones, which then round only where a stage stores; the tube's
// own type in the four-step passes, whose registers hold the next tile too.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace tp {
namespace lfft {

// cos and sin of 2 pi k / P
template <int P>
struct Root;
template <>
struct Root<3> {
  static constexpr double c[3] = {1.0, -0.5, -0.5};
  static constexpr double s[3] = {0.0, 0.8660254037844386, -0.8660254037844386};
};
template <>
struct Root<5> {
  static constexpr double c[5] = {
      1.0, 0.30901699437494745, -0.8090169943749475, -0.8090169943749475, 0.30901699437494745};
  static constexpr double s[5] = {
      0.0, 0.9510565162951535, 0.5877852522924731, -0.5877852522924731, -0.9510565162951535};
};
template <>
struct Root<7> {
  static constexpr double c[7] = {
      1.0, 0.6234898018587335, -0.2225209339563144, -0.9009688679024191, -0.9009688679024191, -0.2225209339563144,
      0.6234898018587335};
  static constexpr double s[7] = {
      0.0, 0.7818314824680298, 0.9749279121818236, 0.4338837391175581, -0.4338837391175581, -0.9749279121818236,
      -0.7818314824680298};
};
template <>
struct Root<11> {
  static constexpr double c[11] = {
      1.0, 0.8412535328311812, 0.41541501300188644, -0.14231483827328514, -0.6548607339452851,
      -0.9594929736144974, -0.9594929736144974, -0.6548607339452851, -0.14231483827328514, 0.41541501300188644,
      0.8412535328311812};
  static constexpr double s[11] = {
      0.0, 0.5406408174555976, 0.9096319953545183, 0.9898214418809327, 0.7557495743542583, 0.28173255684142967,
      -0.28173255684142967, -0.7557495743542583, -0.9898214418809327, -0.9096319953545183, -0.5406408174555976};
};
template <>
struct Root<13> {
  static constexpr double c[13] = {
      1.0, 0.8854560256532099, 0.5680647467311558, 0.12053668025532305, -0.3546048870425356, -0.7485107481711011,
      -0.970941817426052, -0.970941817426052, -0.7485107481711011, -0.3546048870425356, 0.12053668025532305,
      0.5680647467311558, 0.8854560256532099};
  static constexpr double s[13] = {
      0.0, 0.46472317204376856, 0.8229838658936564, 0.992708874098054, 0.9350162426854148, 0.6631226582407952,
      0.23931566428755777, -0.23931566428755777, -0.6631226582407952, -0.9350162426854148, -0.992708874098054,
      -0.8229838658936564, -0.46472317204376856};
};
template <>
struct Root<17> {
  static constexpr double c[17] = {
      1.0, 0.9324722294043558, 0.7390089172206591, 0.44573835577653825, 0.092268359463302, -0.2736629900720829,
      -0.6026346363792564, -0.8502171357296141, -0.9829730996839018, -0.9829730996839018, -0.8502171357296141,
      -0.6026346363792564, -0.2736629900720829, 0.092268359463302, 0.44573835577653825, 0.7390089172206591,
      0.9324722294043558};
  static constexpr double s[17] = {
      0.0, 0.3612416661871529, 0.6736956436465572, 0.8951632913550623, 0.9957341762950345, 0.961825643172819,
      0.7980172272802395, 0.5264321628773558, 0.18374951781657034, -0.18374951781657034, -0.5264321628773558,
      -0.7980172272802395, -0.961825643172819, -0.9957341762950345, -0.8951632913550623, -0.6736956436465572,
      -0.3612416661871529};
};
template <>
struct Root<19> {
  static constexpr double c[19] = {
      1.0, 0.9458172417006346, 0.7891405093963936, 0.5469481581224269, 0.24548548714079915, -0.08257934547233232,
      -0.4016954246529695, -0.6772815716257411, -0.8794737512064891, -0.9863613034027223, -0.9863613034027223,
      -0.8794737512064891, -0.6772815716257411, -0.4016954246529695, -0.08257934547233232, 0.24548548714079915,
      0.5469481581224269, 0.7891405093963936, 0.9458172417006346};
  static constexpr double s[19] = {
      0.0, 0.3246994692046835, 0.6142127126896678, 0.8371664782625285, 0.9694002659393304, 0.9965844930066698,
      0.9157733266550574, 0.7357239106731316, 0.47594739303707356, 0.1645945902807339, -0.1645945902807339,
      -0.47594739303707356, -0.7357239106731316, -0.9157733266550574, -0.9965844930066698, -0.9694002659393304,
      -0.8371664782625285, -0.6142127126896678, -0.3246994692046835};
};
template <>
struct Root<23> {
  static constexpr double c[23] = {
      1.0, 0.9629172873477992, 0.8544194045464886, 0.6825531432186541, 0.46006503773115215, 0.20345601305263378,
      -0.06824241336467098, -0.33487961217098616, -0.5766803221148672, -0.7757112907044198, -0.917211301505453,
      -0.9906859460363308, -0.9906859460363308, -0.917211301505453, -0.7757112907044198, -0.5766803221148672,
      -0.33487961217098616, -0.06824241336467098, 0.20345601305263378, 0.46006503773115215, 0.6825531432186541,
      0.8544194045464886, 0.9629172873477992};
  static constexpr double s[23] = {
      0.0, 0.2697967711570243, 0.5195839500354336, 0.7308359642781241, 0.8878852184023752, 0.9790840876823229,
      0.9976687691905392, 0.9422609221188205, 0.816969893010442, 0.6310879443260528, 0.39840108984624145,
      0.1361666490962466, -0.1361666490962466, -0.39840108984624145, -0.6310879443260528, -0.816969893010442,
      -0.9422609221188205, -0.9976687691905392, -0.9790840876823229, -0.8878852184023752, -0.7308359642781241,
      -0.5195839500354336, -0.2697967711570243};
};
template <>
struct Root<8> {
  static constexpr double c[8] = {
      1.0, 0.7071067811865476, 0.0, -0.7071067811865476, -1.0, -0.7071067811865476, 0.0, 0.7071067811865476};
  static constexpr double s[8] = {
      0.0, 0.7071067811865476, 1.0, 0.7071067811865476, 0.0, -0.7071067811865476, -1.0, -0.7071067811865476};
};
template <>
struct Root<9> {
  static constexpr double c[9] = {
      1.0, 0.766044443118978, 0.17364817766693036, -0.5, -0.9396926207859084, -0.9396926207859084, -0.5,
      0.17364817766693036, 0.766044443118978};
  static constexpr double s[9] = {
      0.0, 0.6427876096865394, 0.984807753012208, 0.8660254037844386, 0.3420201433256687, -0.3420201433256687,
      -0.8660254037844386, -0.984807753012208, -0.6427876096865394};
};
template <>
struct Root<16> {
  static constexpr double c[16] = {
      1.0, 0.9238795325112867, 0.7071067811865476, 0.3826834323650898, 0.0, -0.3826834323650898,
      -0.7071067811865476, -0.9238795325112867, -1.0, -0.9238795325112867, -0.7071067811865476,
      -0.3826834323650898, 0.0, 0.3826834323650898, 0.7071067811865476, 0.9238795325112867};
  static constexpr double s[16] = {
      0.0, 0.3826834323650898, 0.7071067811865476, 0.9238795325112867, 1.0, 0.9238795325112867,
      0.7071067811865476, 0.3826834323650898, 0.0, -0.3826834323650898, -0.7071067811865476, -0.9238795325112867,
      -1.0, -0.9238795325112867, -0.7071067811865476, -0.3826834323650898};
};
template <int P, typename R>
__device__ __forceinline__ void dft(R (&r)[P], R (&i)[P]);

template <typename R>
__device__ __forceinline__ void dft2(R& ar, R& ai, R& br, R& bi) {
  const R xr = ar - br, xi = ai - bi;
  ar += br;
  ai += bi;
  br = xr;
  bi = xi;
}

template <typename R>
__device__ __forceinline__ void dft4(R (&r)[4], R (&i)[4]) {
  const R ar = r[0] + r[2], ai = i[0] + i[2], br = r[0] - r[2], bi = i[0] - i[2];
  const R cr = r[1] + r[3], ci = i[1] + i[3], dr = i[1] - i[3], di = r[3] - r[1];  // (x1 - x3)(-i)
  r[0] = ar + cr;
  i[0] = ai + ci;
  r[1] = br + dr;
  i[1] = bi + di;
  r[2] = ar - cr;
  i[2] = ai - ci;
  r[3] = br - dr;
  i[3] = bi - di;
}

// odd prime P: with t_u = x_u + x_{P-u}, d_u = x_u - x_{P-u},
// X_{k}, X_{P-k} = (x_0 + sum_u t_u cos) -+ i sum_u d_u sin
template <int P, typename R>
__device__ __forceinline__ void dft_prime(R (&r)[P], R (&i)[P]) {
  constexpr int H = (P - 1) / 2;
  R tr[H], ti[H], dr[H], di[H];
#pragma unroll
  for (int u = 0; u < H; ++u) {
    tr[u] = r[u + 1] + r[P - 1 - u];
    ti[u] = i[u + 1] + i[P - 1 - u];
    dr[u] = r[u + 1] - r[P - 1 - u];
    di[u] = i[u + 1] - i[P - 1 - u];
  }
  const R x0r = r[0], x0i = i[0];
#pragma unroll
  for (int u = 0; u < H; ++u) {
    r[0] += tr[u];
    i[0] += ti[u];
  }
#pragma unroll
  for (int k = 1; k <= H; ++k) {
    R ar = x0r, ai = x0i, br = R(0), bi = R(0);
#pragma unroll
    for (int u = 0; u < H; ++u) {
      const int e = (k * (u + 1)) % P;
      ar += R(Root<P>::c[e]) * tr[u];
      ai += R(Root<P>::c[e]) * ti[u];
      br += R(Root<P>::s[e]) * di[u];
      bi += R(Root<P>::s[e]) * dr[u];
    }
    r[k] = ar + br;
    i[k] = ai - bi;
    r[P - k] = ar - br;
    i[P - k] = ai + bi;
  }
}

// P = A B, Cooley-Tukey: A transforms of length B, twiddles, B of length A
template <int A, int B, typename R>
__device__ __forceinline__ void dft_ct(R (&r)[A * B], R (&i)[A * B]) {
  constexpr int P = A * B;
  R yr[A][B], yi[A][B];
#pragma unroll
  for (int a = 0; a < A; ++a) {
#pragma unroll
    for (int b = 0; b < B; ++b) {
      yr[a][b] = r[a + A * b];
      yi[a][b] = i[a + A * b];
    }
    dft<B>(yr[a], yi[a]);
  }
#pragma unroll
  for (int k = 0; k < B; ++k) {
    R tr[A], ti[A];
#pragma unroll
    for (int a = 0; a < A; ++a) {
      const int e = a * k;
      if (e == 0) {
        tr[a] = yr[a][k];
        ti[a] = yi[a][k];
      } else {
        const R c = R(Root<P>::c[e]), s = R(Root<P>::s[e]);
        tr[a] = yr[a][k] * c + yi[a][k] * s;
        ti[a] = yi[a][k] * c - yr[a][k] * s;
      }
    }
    dft<A>(tr, ti);
#pragma unroll
    for (int a = 0; a < A; ++a) {
      r[k + B * a] = tr[a];
      i[k + B * a] = ti[a];
    }
  }
}

// P = A B with A, B coprime, no twiddles (Good-Thomas): input B a + A b,
// output k with k = ka mod A, k = kb mod B
template <int A, int B, typename R>
__device__ __forceinline__ void dft_pfa(R (&r)[A * B], R (&i)[A * B]) {
  constexpr int P = A * B;
  R yr[A][B], yi[A][B];
#pragma unroll
  for (int a = 0; a < A; ++a) {
#pragma unroll
    for (int b = 0; b < B; ++b) {
      yr[a][b] = r[(B * a + A * b) % P];
      yi[a][b] = i[(B * a + A * b) % P];
    }
    dft<B>(yr[a], yi[a]);
  }
#pragma unroll
  for (int b = 0; b < B; ++b) {
    R tr[A], ti[A];
#pragma unroll
    for (int a = 0; a < A; ++a) {
      tr[a] = yr[a][b];
      ti[a] = yi[a][b];
    }
    dft<A>(tr, ti);
#pragma unroll
    for (int a = 0; a < A; ++a) {
      int k = a;  // k = a mod A and b mod B (folded at compile time)
#pragma unroll
      for (int q = 0; q < B; ++q)
        if ((a + q * A) % B == b) k = a + q * A;
      r[k] = tr[a];
      i[k] = ti[a];
    }
  }
}

template <int P, typename R>
__device__ __forceinline__ void dft(R (&r)[P], R (&i)[P]) {
  if constexpr (P == 2)
    dft2(r[0], i[0], r[1], i[1]);
  else if constexpr (P == 4)
    dft4(r, i);
  else if constexpr (P == 6)
    dft_pfa<2, 3>(r, i);
  else if constexpr (P == 8)
    dft_ct<2, 4>(r, i);
  else if constexpr (P == 9)
    dft_ct<3, 3>(r, i);
  else if constexpr (P == 10)
    dft_pfa<2, 5>(r, i);
  else if constexpr (P == 12)
    dft_pfa<4, 3>(r, i);
  else if constexpr (P == 14)
    dft_pfa<2, 7>(r, i);
  else if constexpr (P == 15)
    dft_pfa<3, 5>(r, i);
  else if constexpr (P == 16)
    dft_ct<4, 4>(r, i);
  else if constexpr (P > 1)
    dft_prime<P>(r, i);
}

// --------------------------------------------------------------------------
// Mixed-radix transforms of 2^lg sequences of length N in LDS, element
// (pos, sequence u) at pos 2^lg + u: the lanes of a wavefront take
// neighbouring sequences of a few positions, so every access is a run of
// consecutive words whatever the stage's span.
// --------------------------------------------------------------------------
constexpr int kMaxStages = 12;

struct Plan {
  int n = 0, nst = 0;
  int rad[kMaxStages];
  int m[kMaxStages];        // product of the earlier radices
  int w[kMaxStages];        // product of the later radices
  // ceil(2^32 / d) for d = m and d = rad: x / d = umulhi(x, mag) for x, d < 2^16, d > 1
  uint32_t mag[kMaxStages], rmag[kMaxStages];
};

template <typename S>
struct alignas(2 * sizeof(S)) Cx {
  S x, y;
};

// exp(-2 pi i e / N), 0 <= e < N, from a table of exp(-2 pi i k / 2N),
// k <= N / 2, by the symmetries of the circle
template <typename R>
__device__ __forceinline__ void root_at(const Cx<R>* tab, int N, int e, R& c, R& s) {
  int a = 2 * e;
  const bool neg = a >= N;  // half a turn further
  a = neg ? a - N : a;
  const bool mir = 2 * a > N;  // mirrored on the imaginary axis
  a = mir ? N - a : a;
  const Cx<R> w = tab[a];
  c = neg != mir ? -w.x : w.x;
  s = neg ? -w.y : w.y;
}

// the same from a table of all exp(-2 pi i e / N)
template <typename R>
struct AllRoots {
  const Cx<R>* w;
};
template <typename R>
__device__ __forceinline__ void root_at(AllRoots<R> tab, int, int e, R& c, R& s) {
  const Cx<R> w = tab.w[e];
  c = w.x;
  s = w.y;
}
template <typename R>
__device__ R root_type(const Cx<R>*);
template <typename R>
__device__ R root_type(AllRoots<R>);

// x_t *= W^t, t = 1 .. P-1, W = exp(-2 pi i e1 / N). Float tubes (EXACT false)
// form the powers by two running products in float64 (odd and even t), far
// below the rounding of their storage; double ones read every root.
template <int P, bool EXACT, typename Tab, typename R>
__device__ __forceinline__ void twiddle(Tab tab, int N, int e1, R (&r)[P], R (&i)[P]) {
  R cr[2], ci[2];  // the running powers of odd and even t
  root_at(tab, N, e1, cr[1], ci[1]);
  const R sr = cr[1] * cr[1] - ci[1] * ci[1], si = R(2) * cr[1] * ci[1];
  cr[0] = sr;
  ci[0] = si;
#pragma unroll
  for (int t = 1; t < P; ++t) {
    R &wr = cr[t & 1], &wi = ci[t & 1];
    if (EXACT ? t > 1 : t > 2) {
      if constexpr (EXACT) {
        root_at(tab, N, e1 * t, wr, wi);
      } else {
        const R x = wr;
        wr = x * sr - wi * si;
        wi = x * si + wi * sr;
      }
    }
    const R x = r[t];
    r[t] = x * wr - i[t] * wi;
    i[t] = x * wi + i[t] * wr;
  }
}

// One stage in place: radix P, butterfly (group g, j < m) over the positions
// g m P + j + t m, `ld` elements apart. Decimation in time (DIF false): twiddle W_{mP}^{j t}, then the
// P-point transform; decimation in frequency: the transform, then the twiddle.
template <typename S, int P, bool DIF, bool EXACT, typename Tab>
__device__ __forceinline__ void stage(Cx<S>* buf, int lg, int ld, int N, int m, uint32_t mag, Tab tab) {
  using R = decltype(root_type(tab));
  const int mask = (1 << lg) - 1, per = N / P, total = per << lg;
  for (int b = threadIdx.x; b < total; b += blockDim.x) {
    const int u = b & mask, c = b >> lg;
    int g = c, j = 0;
    if (m > 1) {
      g = (int)__umulhi((uint32_t)c, mag);
      j = c - g * m;
    }
    Cx<S>* p = buf + (g * (m * P) + j) * ld + u;
    const int step = m * ld;
    R r[P], i[P];
#pragma unroll
    for (int t = 0; t < P; ++t) {
      const Cx<S> v = p[t * step];
      r[t] = (R)v.x;
      i[t] = (R)v.y;
    }
    const int e1 = j * (N / (m * P));
    if (!DIF && m > 1) twiddle<P, EXACT>(tab, N, e1, r, i);
    dft<P>(r, i);
    if (DIF && m > 1) twiddle<P, EXACT>(tab, N, e1, r, i);
#pragma unroll
    for (int t = 0; t < P; ++t) p[t * step] = Cx<S>{(S)r[t], (S)i[t]};
  }
}

// All stages. DIF: natural order in, element k of the result at position
// pos(k) (see fill_positions); otherwise input element e at pos(e), natural
// order out. Ends with a barrier.
template <typename S, bool DIF, bool EXACT, typename Tab>
__device__ void stages(const Plan& pl, Cx<S>* buf, int lg, int ld, Tab tab) {
  for (int q = 0; q < pl.nst; ++q) {
    const int z = DIF ? pl.nst - 1 - q : q;
    const int m = pl.m[z];
    const uint32_t mag = pl.mag[z];
    switch (pl.rad[z]) {
      case 2: stage<S, 2, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 3: stage<S, 3, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 4: stage<S, 4, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 5: stage<S, 5, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 6: stage<S, 6, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 7: stage<S, 7, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 8: stage<S, 8, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 9: stage<S, 9, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 10: stage<S, 10, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 11: stage<S, 11, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 12: stage<S, 12, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 13: stage<S, 13, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 14: stage<S, 14, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      case 15: stage<S, 15, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
      default: stage<S, 16, DIF, EXACT>(buf, lg, ld, pl.n, m, mag, tab); break;
    }
    __syncthreads();
  }
}
template <typename S, bool DIF, bool EXACT>
__device__ __forceinline__ void stages(const Plan& pl, Cx<S>* buf, int lg, const Cx<double>* tab) {
  stages<S, DIF, EXACT>(pl, buf, lg, 1 << lg, tab);
}

// pos[k], k < N: where the in-place stages keep element k of the transform
__device__ __forceinline__ void fill_positions(const Plan& pl, uint16_t* pos) {
  for (int p = threadIdx.x; p < pl.n; p += blockDim.x) {
    int rest = p, k = 0;
    for (int q = 0; q < pl.nst; ++q) {
      const int next = (int)__umulhi((uint32_t)rest, pl.rmag[q]);
      k += (rest - next * pl.rad[q]) * pl.w[q];
      rest = next;
    }
    pos[k] = (uint16_t)p;
  }
}

// exp(-2 pi i k / 2N), k <= N / 2
__device__ __forceinline__ void fill_roots(int N, Cx<double>* tab) {
  for (int k = threadIdx.x; k <= N / 2; k += blockDim.x) {
    double s, c;
    sincospi(-(double)k / (double)N, &s, &c);
    tab[k] = Cx<double>{c, s};
  }
}

// exp(-2 pi i k / N), k < N, rounded once to the butterflies' type
template <typename R>
__device__ __forceinline__ void fill_all_roots(int N, Cx<R>* tab) {
  for (int k = threadIdx.x; k < N; k += blockDim.x) {
    double s, c;
    sincospi(-2.0 * (double)k / (double)N, &s, &c);
    tab[k] = Cx<R>{(R)c, (R)s};
  }
}

// Radix plan of a length without prime factors above 13 with the fewest
// stages, larger radices last (their twiddles are the longest); false for
// other lengths.
bool radix_plan(int64_t n, Plan& pl);

}  // namespace lfft
}  // namespace tp
