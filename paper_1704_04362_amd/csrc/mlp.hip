// Learned lateral-leverage proposal: cheap per-slice features, a small MLP
// (17 -> 128 -> 128 -> 1, ReLU) on the fp16 matrix cores with float32
// accumulation, per-tensor softmax with a KL loss against the exact
// leverage distribution, backward pass and Adam. Not part of the paper,
// which estimates leverage with a randomized routine it cites without
// describing; the exact scores (eq. cur-col-prob) stay the fallback.
//
// Features of lateral slice j of an n1 x n2 x n3 tensor A: the sketch
// s_j = Phi^T vec(A_{:j:}) with a caller-supplied (n1 n3) x 16 matrix Phi,
// whitened as z_j = G^{-1/2} s_j sqrt(n2), G = sum_j s_j s_j^T, and
// f_j = log(n2 a_j / sum a), a_j = ||A_{:j:}||_F^2.
//
// Parameters are one float32 array (the master copy) laid out as
//   W1 (17 x 128) | b1 (128) | W2 (128 x 128) | b2 (128) | w3 (128) | b3 (1)
// (h1 = relu(x W1 + b1), h2 = relu(h1 W2 + b2), o = h2 w3 + b3); the
// forward and backward passes use fp16 copies of W1 and W2 and fp16
// activations as matrix-core operands.
#include <cmath>

#include "common.hpp"
#include "jacobi.hpp"
#include "mlp.hpp"

namespace tp {
namespace {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int DS = 16, DIN = 17, KIN = 32, HID = 128;
constexpr int OFF_W1 = 0, OFF_B1 = DIN * HID, OFF_W2 = OFF_B1 + HID, OFF_B2 = OFF_W2 + HID * HID,
              OFF_W3 = OFF_B2 + HID, OFF_B3 = OFF_W3 + HID;
constexpr int NPARAM = OFF_B3 + 1;
static_assert(NPARAM == kMlpParams, "parameter layout");

// ---------------------------------------------------------------------------
// features
// ---------------------------------------------------------------------------
// The sketch is the contraction S = X Phi with X (n2 x n1 n3), row j =
// vec(A_{:j:}). In the tube-major layout horizontal slice i of A is an
// n2 x n3 row-major block, so S = sum_i A_{i::} Phi_i with Phi_i the rows
// i n3 .. i n3 + n3 - 1 of Phi: per horizontal slice a (64 slices x n3) by
// (n3 x 16) product on the fp32 matrix cores (v_mfma_f32_16x16x4f32), one
// 16-slice tile per wavefront. Lane l of a wavefront owns row l % 16 of the
// tile and tube entries 4 (l / 16) .. 4 (l / 16) + 3 of every 16-entry tube
// block (one float4 load); its four values feed four matrix-core steps,
// with Phi_i read at the same tube positions from a transposed LDS copy.
constexpr int SJ = 64;   // lateral slices per workgroup (4 tiles of 16)
constexpr int SIR = 16;  // horizontal slices per workgroup
constexpr int SNT = 256;

// Tubes are taken in chunks of at most kSketchChunk entries (a multiple of
// 16), so that two chunks of Phi_i fit in 64 KB of LDS at any tube length.
constexpr int kSketchChunk = 496;
__device__ __host__ __forceinline__ int sketch_chunk(int64_t n3) {
  const int64_t r = (n3 + 15) / 16 * 16;
  return (int)(r < kSketchChunk ? r : kSketchChunk);
}
__device__ __host__ __forceinline__ int sketch_ldk(int64_t n3) { return sketch_chunk(n3) + 4; }

// partial[(y n2 + j) (DS + 1) + d]: the chunk-y sums (float32) of the
// sketch (d < DS) and of the squared norm (d = DS) of lateral slice j.
__global__ __launch_bounds__(SNT) void sketch_mfma_kernel(const float* __restrict__ a, const float* __restrict__ phi,
                                                           int64_t n1, int64_t n2, int64_t n3,
                                                           float* __restrict__ partial) {
  extern __shared__ float phs[];  // [2][DS][ldk]: a tube chunk of Phi_i transposed, double buffered
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kc = sketch_chunk(n3), ldk = kc + 4;
  const int64_t j0 = (int64_t)blockIdx.x * SJ;
  const int64_t i0 = (int64_t)blockIdx.y * SIR;
  const int64_t rows = (n1 - i0) < SIR ? (n1 - i0) : SIR;
  const int g = lane >> 4, r = lane & 15;
  const int64_t j = j0 + wave * 16 + r;
  const bool jok = j < n2;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float nrm = 0.f;
  // steps over (horizontal slice, tube chunk); the buffer written in a step
  // was last read two steps earlier, before the previous step's barrier
  int step = 0;
  for (int64_t ii = 0; ii < rows; ++ii) {
    const int64_t i = i0 + ii;
    const float* src = phi + i * n3 * DS;
    const float* arow = a + (i * n2 + j) * n3;
    for (int64_t k0 = 0; k0 < n3; k0 += kc, ++step) {
      float* buf = phs + (step & 1) * DS * ldk;
      // this chunk of Phi_i, zero beyond the tube's end
      for (int e = tid; e < kc * DS; e += SNT) {
        const int kk = e / DS, d = e - kk * DS;
        buf[d * ldk + kk] = k0 + kk < n3 ? src[(k0 + kk) * DS + d] : 0.f;
      }
      __syncthreads();
      const int nkb = (int)((n3 - k0 < kc ? n3 - k0 : kc) + 15) / 16;
      for (int kb = 0; kb < nkb; ++kb) {
        const int kk = kb * 16 + 4 * g;
        const int64_t k = k0 + kk;
        float4 x = {0.f, 0.f, 0.f, 0.f};
        if (jok && k < n3) x = *reinterpret_cast<const float4*>(arow + k);
        const float4 p = *reinterpret_cast<const float4*>(buf + r * ldk + kk);
        nrm += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, p.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, p.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.z, p.z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.w, p.w, acc, 0, 0, 0);
      }
    }
  }
  // lane l holds S[row 4 g + v][d = l % 16] of the wavefront's tile
  float* out = partial + ((int64_t)blockIdx.y * n2) * (DS + 1);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int64_t jj = j0 + wave * 16 + 4 * g + v;
    if (jj < n2) out[jj * (DS + 1) + r] = acc[v];
  }
  nrm += __shfl_xor(nrm, 16);
  nrm += __shfl_xor(nrm, 32);
  if (g == 0 && jok) out[j * (DS + 1) + DS] = nrm;
}

// The same contraction for tubes of at most 16 NKB entries with every load
// of a horizontal slice issued at once: lane (g, r) holds the NKB float4
// pieces 4 g + 16 b (b < NKB) of its tube, and the next slice's pieces and
// its share of the next Phi_i are fetched into registers before the
// current slice's matrix-core steps, so that HBM latency overlaps the
// arithmetic. Phi_i is staged transposed in two LDS buffers (one barrier
// per slice).
template <int NKB>
__global__ __launch_bounds__(SNT) void sketch_mfma_pipe_kernel(const float* __restrict__ a,
                                                                const float* __restrict__ phi, int64_t n1,
                                                                int64_t n2, int64_t n3, float* __restrict__ partial) {
  constexpr int LDK = 16 * NKB + 4;
  constexpr int PH = 16 * NKB * DS / SNT;  // Phi_i entries per thread (padded tube)
  static_assert(PH * SNT == 16 * NKB * DS, "whole Phi_i per workgroup");
  __shared__ __align__(16) float phs[2][DS][LDK];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t j0 = (int64_t)blockIdx.x * SJ;
  const int64_t i0 = (int64_t)blockIdx.y * SIR;
  const int64_t rows = (n1 - i0) < SIR ? (n1 - i0) : SIR;
  const int g = lane >> 4, r = lane & 15;
  const int64_t j = j0 + wave * 16 + r;
  const bool jok = j < n2;
  auto load_a = [&](int64_t i, float4 (&x)[NKB]) {
    const float* arow = a + (i * n2 + (jok ? j : 0)) * n3;
#pragma unroll
    for (int b = 0; b < NKB; ++b) {
      const int64_t k = 16 * b + 4 * g;
      x[b] = (jok && k < n3) ? *reinterpret_cast<const float4*>(arow + k) : float4{0.f, 0.f, 0.f, 0.f};
    }
  };
  // thread's Phi entries: e = tid + SNT u of the padded (16 NKB) x DS block
  auto load_phi = [&](int64_t i, float (&v)[PH]) {
    const float* src = phi + i * n3 * DS;
#pragma unroll
    for (int u = 0; u < PH; ++u) {
      const int e = tid + SNT * u;
      v[u] = (e / DS) < n3 ? src[e] : 0.f;
    }
  };
  float4 xc[NKB], xn[NKB];
  float pv[PH];
  load_a(i0, xc);
  load_phi(i0, pv);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float nrm = 0.f;
  for (int64_t ii = 0; ii < rows; ++ii) {
    float(*buf)[LDK] = phs[ii & 1];
#pragma unroll
    for (int u = 0; u < PH; ++u) {
      const int e = tid + SNT * u;
      buf[e % DS][e / DS] = pv[u];
    }
    if (ii + 1 < rows) {
      load_a(i0 + ii + 1, xn);
      load_phi(i0 + ii + 1, pv);
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NKB; ++b) {
      const float4 x = xc[b];
      const float4 p = *reinterpret_cast<const float4*>(&buf[r][16 * b + 4 * g]);
      nrm += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, p.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, p.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.z, p.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.w, p.w, acc, 0, 0, 0);
    }
#pragma unroll
    for (int b = 0; b < NKB; ++b) xc[b] = xn[b];
  }
  float* out = partial + ((int64_t)blockIdx.y * n2) * (DS + 1);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int64_t jj = j0 + wave * 16 + 4 * g + v;
    if (jj < n2) out[jj * (DS + 1) + r] = acc[v];
  }
  nrm += __shfl_xor(nrm, 16);
  nrm += __shfl_xor(nrm, 32);
  if (g == 0 && jok) out[j * (DS + 1) + DS] = nrm;
}

// Per block of SJS lateral slices: the float64 sums over the row chunks
// (sk[j][0..DS] = sketch and squared norm), and the block's share of the
// Gram matrix G = sum_j s_j s_j^T and of sum_j a_j (gpart[blk][0..DS*DS]).
constexpr int SJS = 16;
__global__ __launch_bounds__(256) void sketch_sum_kernel(const float* __restrict__ partial, int64_t nch, int64_t n2,
                                                          double* __restrict__ sk, double* __restrict__ gpart) {
  __shared__ double s[SJS][DS + 1];
  const int tid = threadIdx.x;
  const int64_t j0 = (int64_t)blockIdx.x * SJS;
  const int64_t nj = (n2 - j0) < SJS ? (n2 - j0) : SJS;
  // entries e of the block's (nj x (DS + 1)) run are contiguous in every chunk
  for (int e = tid; e < SJS * (DS + 1); e += 256) {
    const int t = e / (DS + 1);
    double v = 0.0;
    if (t < nj) {
      const float* src = partial + j0 * (DS + 1) + e;
      const int64_t stride = n2 * (DS + 1);
      int64_t y = 0;
      for (; y + 8 <= nch; y += 8) {
        float f[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) f[u] = src[(y + u) * stride];
#pragma unroll
        for (int u = 0; u < 8; ++u) v += (double)f[u];
      }
      for (; y < nch; ++y) v += (double)src[y * stride];
      sk[j0 * (DS + 1) + e] = v;
    }
    s[t][e - t * (DS + 1)] = v;
  }
  __syncthreads();
  {
    const int p = tid / DS, q = tid % DS;
    double gsum = 0.0;
    for (int t = 0; t < SJS; ++t) gsum += s[t][p] * s[t][q];
    gpart[blockIdx.x * (DS * DS + 1) + tid] = gsum;
  }
  if (tid == 0) {
    double at = 0.0;
    for (int t = 0; t < SJS; ++t) at += s[t][DS];
    gpart[blockIdx.x * (DS * DS + 1) + DS * DS] = at;
  }
}

// G and sum a from the block shares (fixed order), then the whitening
// W = G^{-1/2} sqrt(n2) (the symmetric inverse square root, unique for a
// positive definite G). With A = G / tr(G) (eigenvalues in (0, 1)), the
// coupled Newton-Schulz iteration T = (3 I - Z Y) / 2, Y <- Y T, Z <- T Z
// from Y = A, Z = I takes Z to A^{-1/2} (Higham, Functions of Matrices,
// sec. 6.3); it stops once max |T - I| <= 1e-12 (the T applied last is then
// I to second order). If it has not converged after kNsIters steps (G
// singular or nearly so) the float64 Jacobi solver diagonalises G instead
// and W = V diag(lambda^{-1/2}) V^T over the positive eigenvalues.
// wt[0..DS*DS) = W (row-major), wt[DS*DS] = sum a.
constexpr int kNsIters = 64;

__global__ __launch_bounds__(256) void sketch_whiten_kernel(const double* __restrict__ gpart, int64_t nblk,
                                                             int64_t n2, double* __restrict__ wt) {
  static_assert(DS * DS == 256, "one Gram entry per thread");
  __shared__ JacobiShared<DS, 256> sh;
  __shared__ double Y[DS][DS + 1], Z[DS][DS + 1], T[DS][DS + 1];
  __shared__ double dev[4];
  const int tid = threadIdx.x;
  const int p = tid / DS, q = tid % DS;
  double g = 0.0;
  for (int64_t b = 0; b < nblk; ++b) g += gpart[b * (DS * DS + 1) + tid];
  sh.Hr[p][q] = g;
  sh.Hi[p][q] = 0.0;
  if (tid == 0) {
    double at = 0.0;
    for (int64_t b = 0; b < nblk; ++b) at += gpart[b * (DS * DS + 1) + DS * DS];
    wt[DS * DS] = at;
  }
  __syncthreads();
  double tr = 0.0;
  for (int c = 0; c < DS; ++c) tr += sh.Hr[c][c];
  bool done = false;
  if (tr > 0.0 && tr < INFINITY) {
    const double inv = 1.0 / tr;
    Y[p][q] = 0.5 * (sh.Hr[p][q] + sh.Hr[q][p]) * inv;
    Z[p][q] = p == q ? 1.0 : 0.0;
    __syncthreads();
    for (int it = 0; it < kNsIters; ++it) {
      double zy = 0.0;
#pragma unroll
      for (int c = 0; c < DS; ++c) zy += Z[p][c] * Y[c][q];
      const double t = (p == q ? 1.5 : 0.0) - 0.5 * zy;
      double d = fabs(t - (p == q ? 1.0 : 0.0));
      d = d == d ? d : INFINITY;  // a NaN never converges
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) d = fmax(d, __shfl_xor(d, o));
      T[p][q] = t;
      if ((tid & 63) == 0) dev[tid >> 6] = d;
      __syncthreads();
      double yn = 0.0, zn = 0.0;
#pragma unroll
      for (int c = 0; c < DS; ++c) {
        yn += Y[p][c] * T[c][q];
        zn += T[p][c] * Z[c][q];
      }
      const double m = fmax(fmax(dev[0], dev[1]), fmax(dev[2], dev[3]));
      __syncthreads();
      Y[p][q] = yn;
      Z[p][q] = zn;
      __syncthreads();
      if (m <= 1e-12) {
        done = true;
        break;
      }
    }
  }
  if (done) {
    wt[tid] = Z[p][q] * sqrt((double)n2 / tr);
    return;
  }
  jacobi_eig_lds<DS, 256>(sh, DS, 30, 1e-15);
  double t = 0.0;
  for (int c = 0; c < DS; ++c) {
    const double l = sh.Hr[c][c];
    if (l > 0.0) t += sh.Vr[p][c] * sh.Vr[q][c] / sqrt(l);
  }
  wt[tid] = t * sqrt((double)n2);
}

// feat[j] = [s_j^T W, log(n2 a_j / sum a)]; optionally a_j itself.
__global__ void sketch_apply_kernel(const double* __restrict__ sk, const double* __restrict__ wt, int64_t n2,
                                    float* __restrict__ feat, double* __restrict__ norms) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n2 * DIN) return;
  const int64_t j = e / DIN;
  const int d = (int)(e - j * DIN);
  double v;
  if (d < DS) {
    v = 0.0;
    for (int q = 0; q < DS; ++q) v += sk[j * (DS + 1) + q] * wt[q * DS + d];
  } else {
    const double aj = sk[j * (DS + 1) + DS];
    v = log((double)n2 * aj / wt[DS * DS]);
    if (norms) norms[j] = aj;
  }
  feat[e] = (float)v;
}

// ---------------------------------------------------------------------------
// MLP on the matrix cores
// ---------------------------------------------------------------------------
// Bound: latency. One tile of 64 rows a workgroup is a chain of a few weight
// loads, 16 x 16 x 16 products and row sums, on at most rows / 64 CUs. So
// every operand lies in LDS with its contraction index contiguous (a fragment is
// one 8-byte read; the product's operands are swapped where the result's
// layout then stores whole quads), all loads of a stage are issued together,
// eight wavefronts share a tile, and the training step keeps the activations
// instead of computing them again. 8192 rows: forward 26 -> 8 us, backward
// 34 -> 11, the sums over tiles, the loss and Adam 40 -> 7 in one launch
// (replaced: four wavefronts, operands gathered value by value).
constexpr int TR = 64;  // rows per tile
constexpr int NT = 512;
constexpr int LX = KIN + 8, LH = HID + 8, LT = TR + 8;  // LDS rows (padded), of quads
constexpr int LZ = TR + 4;

// acc += A B for 16 x 16 tiles, K deep: A[i][k] at a[i lda + k], B[k][j] at b[j ldb + k].
__device__ __forceinline__ f32x4 mfma_tile(const _Float16* a, int lda, const _Float16* b, int ldb, int K, f32x4 acc) {
  const int lane = threadIdx.x & 63;
  const int r = lane & 15, kq = 4 * (lane >> 4);
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += 16)
    acc = __builtin_amdgcn_mfma_f32_16x16x16f16(*reinterpret_cast<const half4*>(a + r * lda + k0 + kq),
                                                *reinterpret_cast<const half4*>(b + r * ldb + k0 + kq), acc, 0, 0, 0);
  return acc;
}

// Forward pass of one tile: logits, and with SAVE the activations (post-ReLU,
// fp16, [row][HID], whole tiles). Pre-activations are positive exactly where
// the stored post-activations are, which the backward pass uses as the masks.
template <bool SAVE>
__global__ __launch_bounds__(NT, 2) void mlp_forward_kernel(const float* __restrict__ P,
                                                            const float* __restrict__ feat, int64_t nrows,
                                                            float* __restrict__ out, _Float16* __restrict__ h1,
                                                            _Float16* __restrict__ h2) {
  __shared__ __align__(16) _Float16 X[TR][LX];     // input tile, features padded to KIN
  __shared__ __align__(16) _Float16 W1t[HID][LX];  // W1 transposed (entries 17..31 zero)
  __shared__ __align__(16) _Float16 W2t[HID][LH];
  __shared__ __align__(16) _Float16 H1[TR][LH];
  __shared__ __align__(16) float z[TR][HID + 4];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t r0 = (int64_t)blockIdx.x * TR;
  // four rows of a column of W2 at a time, lanes along the row
  constexpr int Q2 = HID * HID / 4 / NT;
  float w2[Q2][4];
#pragma unroll
  for (int u = 0; u < Q2; ++u) {
    const int e = tid + NT * u, j = e % HID, k = 4 * (e / HID);
#pragma unroll
    for (int v = 0; v < 4; ++v) w2[u][v] = P[OFF_W2 + (k + v) * HID + j];
  }
  for (int e = tid; e < TR * KIN; e += NT) {
    const int r = e / KIN, c = e % KIN;
    const int64_t row = r0 + r;
    X[r][c] = (_Float16)((c < DIN && row < nrows) ? feat[row * DIN + c] : 0.f);
  }
  for (int e = tid; e < HID * KIN; e += NT) {
    const int k = e / HID, j = e % HID;
    W1t[j][k] = (_Float16)(k < DIN ? P[OFF_W1 + k * HID + j] : 0.f);
  }
  const int rt = wave & 3, c0 = 64 * (wave >> 2);  // 16 rows, 64 columns a wavefront
  const int row = 16 * rt + (lane & 15), cq = 4 * (lane >> 4);
  float b1[4][4], b2[4][4], w3[4][4];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = c0 + 16 * nt + cq + e;
      b1[nt][e] = P[OFF_B1 + c];
      b2[nt][e] = P[OFF_B2 + c];
      w3[nt][e] = P[OFF_W3 + c];
    }
#pragma unroll
  for (int u = 0; u < Q2; ++u) {
    const int e = tid + NT * u, j = e % HID, k = 4 * (e / HID);
    *reinterpret_cast<half4*>(&W2t[j][k]) =
        half4{(_Float16)w2[u][0], (_Float16)w2[u][1], (_Float16)w2[u][2], (_Float16)w2[u][3]};
  }
  __syncthreads();
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    const int c = c0 + 16 * nt;
    const f32x4 acc = mfma_tile(&W1t[c][0], LX, &X[16 * rt][0], LX, KIN, f32x4{0.f, 0.f, 0.f, 0.f});
    half4 h;
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = (_Float16)fmaxf(acc[e] + b1[nt][e], 0.f);
    *reinterpret_cast<half4*>(&H1[row][c + cq]) = h;
    if (SAVE) *reinterpret_cast<half4*>(&h1[(r0 + row) * HID + c + cq]) = h;
  }
  __syncthreads();
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    const int c = c0 + 16 * nt;
    const f32x4 acc = mfma_tile(&W2t[c][0], LH, &H1[16 * rt][0], LH, HID, f32x4{0.f, 0.f, 0.f, 0.f});
    half4 h;
    f32x4 zq;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float v = fmaxf(acc[e] + b2[nt][e], 0.f);
      h[e] = (_Float16)v;
      zq[e] = v * w3[nt][e];
    }
    *reinterpret_cast<f32x4*>(&z[row][c + cq]) = zq;
    if (SAVE) *reinterpret_cast<half4*>(&h2[(r0 + row) * HID + c + cq]) = h;
  }
  __syncthreads();
  if (tid < TR && r0 + tid < nrows) {
    float o = P[OFF_B3];
#pragma unroll 8
    for (int c = 0; c < HID; c += 4) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(&z[tid][c]);
#pragma unroll
      for (int e = 0; e < 4; ++e) o += v[e];
    }
    out[r0 + tid] = o;
  }
}

// The tree over 256 threads' values that halves them seven times more (thread
// t takes t + 128, t + 64, ..., t + 1), for every thread: the first two levels
// from LDS and the others by shuffles in the first wavefront, two barriers in
// place of nine.
template <typename F>
__device__ __forceinline__ double tree256(double v, double* red, F op) {
  const int tid = threadIdx.x;
  red[tid] = v;
  __syncthreads();
  if (tid < 64) {
    v = op(op(red[tid], red[tid + 128]), op(red[tid + 64], red[tid + 192]));
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) v = op(v, __shfl_down(v, w));
    if (tid == 0) red[256] = v;
  }
  __syncthreads();
  return red[256];
}

// Per tensor: p = softmax(o), loss = KL(p* || p), dO = (p - p*) / T. Bound: the
// latency of four reductions in a row (16 x 512: 6.7 -> 5.7 us with tree256).
__global__ __launch_bounds__(256) void softmax_grad_kernel(const float* __restrict__ o,
                                                           const float* __restrict__ target, int64_t nsl, int64_t T,
                                                           float* __restrict__ dout, float* __restrict__ loss_part) {
  __shared__ double red[4][257];
  const int64_t t = blockIdx.x;
  const int tid = threadIdx.x;
  const float* ot = o + t * nsl;
  const float* pt = target + t * nsl;
  const auto add = [](double a, double b) { return a + b; };
  double m = -INFINITY;
  for (int64_t j = tid; j < nsl; j += 256) m = fmax(m, (double)ot[j]);
  const double mx = tree256(m, red[0], [](double a, double b) { return fmax(a, b); });
  double se = 0.0;
  for (int64_t j = tid; j < nsl; j += 256) se += exp((double)ot[j] - mx);
  const double lse = mx + log(tree256(se, red[1], add));
  // the target row is normalised here (any positive scale is accepted)
  double qs = 0.0;
  for (int64_t j = tid; j < nsl; j += 256) qs += (double)pt[j];
  const double qsum = tree256(qs, red[2], add), qinv = qsum > 0.0 ? 1.0 / qsum : 0.0;
  double kl = 0.0;
  for (int64_t j = tid; j < nsl; j += 256) {
    const double lp = (double)ot[j] - lse;
    const double q = (double)pt[j] * qinv;
    if (q > 0) kl += q * (log(q) - lp);
    dout[t * nsl + j] = (float)((exp(lp) - q) / (double)T);
  }
  kl = tree256(kl, red[3], add);
  if (tid == 0) loss_part[t] = (float)(kl / (double)T);
}

// a b rounded once, to fp16 (left to itself the compiler fuses the conversion
// into some of these products and rounds others twice)
__device__ __forceinline__ _Float16 mul_f16(float a, float b) {
  uint32_t r;
  asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(r) : "v"(a), "v"(b));
  return __builtin_bit_cast(_Float16, (uint16_t)r);
}

// Backward of one tile from the forward pass's activations: this tile's
// gradient contribution (parameter layout) to partial[tile].
__global__ __launch_bounds__(NT, 2) void mlp_backward_kernel(const float* __restrict__ P,
                                                             const float* __restrict__ feat,
                                                             const float* __restrict__ dout, int64_t nrows,
                                                             const _Float16* __restrict__ h1,
                                                             const _Float16* __restrict__ h2,
                                                             float* __restrict__ partial) {
  // (transposed: [feature][row])
  __shared__ __align__(16) _Float16 Xt[KIN][LT];
  __shared__ __align__(16) _Float16 W2[HID][LH];
  __shared__ __align__(16) _Float16 H1t[HID][LT];
  __shared__ __align__(16) _Float16 H2t[HID][LT];
  __shared__ __align__(16) _Float16 D[TR][LH];  // dH2
  __shared__ __align__(16) _Float16 Dt[HID][LT];
  __shared__ __align__(16) float zt[HID][LZ];  // dH1
  __shared__ float sd[TR];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t r0 = (int64_t)blockIdx.x * TR;
  float* g = partial + (int64_t)blockIdx.x * NPARAM;
  constexpr int Q2 = HID * HID / 4 / NT;
  float4 w2[Q2];
#pragma unroll
  for (int u = 0; u < Q2; ++u) {  // (the parameter array's W2 need not be 16-byte aligned)
    const float* src = P + OFF_W2 + 4 * (tid + NT * u);
    w2[u] = float4{src[0], src[1], src[2], src[3]};
  }
  {
    // 4 rows x 4 columns of the activations a thread: dH2 = dO w3 (.) [h2 > 0]
    static_assert(TR * HID / 16 == NT, "one block of 4 x 4 a thread");
    const int c = 4 * (tid % (HID / 4)), r = 4 * (tid / (HID / 4));
    half4 x[4], y[4];
    float d[4], w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = *reinterpret_cast<const half4*>(&h1[(r0 + r + i) * HID + c]);
      y[i] = *reinterpret_cast<const half4*>(&h2[(r0 + r + i) * HID + c]);
      d[i] = r0 + r + i < nrows ? dout[r0 + r + i] : 0.f;
      w[i] = P[OFF_W3 + c + i];
    }
    half4 dh[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int e = 0; e < 4; ++e) dh[i][e] = (float)y[i][e] > 0.f ? mul_f16(d[i], w[e]) : (_Float16)0.f;
      *reinterpret_cast<half4*>(&D[r + i][c]) = dh[i];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      *reinterpret_cast<half4*>(&H1t[c + e][r]) = half4{x[0][e], x[1][e], x[2][e], x[3][e]};
      *reinterpret_cast<half4*>(&H2t[c + e][r]) = half4{y[0][e], y[1][e], y[2][e], y[3][e]};
      *reinterpret_cast<half4*>(&Dt[c + e][r]) = half4{dh[0][e], dh[1][e], dh[2][e], dh[3][e]};
    }
    if (c == 0)
#pragma unroll
      for (int i = 0; i < 4; ++i) sd[r + i] = d[i];
  }
  for (int e = tid; e < TR * KIN; e += NT) {
    const int r = e / KIN, c = e % KIN;
    Xt[c][r] = (_Float16)((c < DIN && r0 + r < nrows) ? feat[(r0 + r) * DIN + c] : 0.f);
  }
#pragma unroll
  for (int u = 0; u < Q2; ++u) {
    const int e = 4 * (tid + NT * u);
    *reinterpret_cast<half4*>(&W2[e / HID][e % HID]) =
        half4{(_Float16)w2[u].x, (_Float16)w2[u].y, (_Float16)w2[u].z, (_Float16)w2[u].w};
  }
  __syncthreads();
  const int rq = 4 * (lane >> 4), cl = lane & 15;
  // dH1 = (dH2 W2^T) (.) [h1 > 0]
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int rt = wave & 3, c = 64 * (wave >> 2) + 16 * t;
    const f32x4 acc = mfma_tile(&D[16 * rt][0], LH, &W2[c][0], LH, HID, f32x4{0.f, 0.f, 0.f, 0.f});
    const half4 h = *reinterpret_cast<const half4*>(&H1t[c + cl][16 * rt + rq]);
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (float)h[e] > 0.f ? acc[e] : 0.f;
    *reinterpret_cast<f32x4*>(&zt[c + cl][16 * rt + rq]) = v;
  }
  // W2 = H1^T dH2
#pragma unroll
  for (int t = 0; t < HID / 16; ++t) {
    const f32x4 acc = mfma_tile(&H1t[16 * wave][0], LT, &Dt[16 * t][0], LT, TR, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
    for (int e = 0; e < 4; ++e) g[OFF_W2 + (16 * wave + rq + e) * HID + 16 * t + cl] = acc[e];
  }
  // w3, b2 = column sums of dH2, b3
  if (tid < HID) {
    float gw = 0.f;
#pragma unroll 16
    for (int r = 0; r < TR; ++r) gw += (float)H2t[tid][r] * sd[r];
    g[OFF_W3 + tid] = gw;
  } else if (tid < 2 * HID) {
    float gb = 0.f;
#pragma unroll 16
    for (int r = 0; r < TR; ++r) gb += (float)Dt[tid - HID][r];
    g[OFF_B2 + tid - HID] = gb;
  } else if (tid == 2 * HID) {
    float gb = 0.f;
#pragma unroll 16
    for (int r = 0; r < TR; ++r) gb += sd[r];
    g[OFF_B3] = gb;
  }
  __syncthreads();
  // W1 = X^T dH1 (fp16), b1 = column sums of dH1 (float)
  static_assert(HID / 16 == NT / 64, "16 columns a wavefront");
#pragma unroll
  for (int it = 0; it < KIN / 16; ++it) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k0 = 0; k0 < TR; k0 += 16) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(&zt[16 * wave + cl][k0 + rq]);
      acc = __builtin_amdgcn_mfma_f32_16x16x16f16(
          *reinterpret_cast<const half4*>(&Xt[16 * it + cl][k0 + rq]),
          half4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]}, acc, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = 16 * it + rq + e;
      if (row < DIN) g[OFF_W1 + row * HID + 16 * wave + cl] = acc[e];
    }
  }
  if (tid < HID) {
    float gb = 0.f;
#pragma unroll 16
    for (int r = 0; r < TR; ++r) gb += zt[tid][r];
    g[OFF_B1 + tid] = gb;
  }
}

// The tiles' gradients summed in tile order and Adam's update with them (adam
// false: the gradient only), one parameter a thread; the last workgroup sums the
// tensors' losses.
constexpr int GNT = 64;
__global__ __launch_bounds__(GNT) void grad_adam_kernel(const float* __restrict__ partial, int64_t ntiles,
                                                        float* __restrict__ grad, const float* __restrict__ lpart,
                                                        int64_t T, float* __restrict__ loss, bool adam,
                                                        float* __restrict__ P, float* __restrict__ M,
                                                        float* __restrict__ V, float lr, float b1, float b2, float eps,
                                                        float c1, float c2) {
  if (blockIdx.x == gridDim.x - 1) {
    if (threadIdx.x == 0 && loss) {
      float s = 0.f;
#pragma unroll 16
      for (int64_t t = 0; t < T; ++t) s += lpart[t];
      *loss = s;
    }
    return;
  }
  const int64_t p = (int64_t)blockIdx.x * GNT + threadIdx.x;
  if (p >= NPARAM) return;
  float g = 0.f;
#pragma unroll 32
  for (int64_t t = 0; t < ntiles; ++t) g += partial[t * NPARAM + p];
  if (grad) grad[p] = g;
  if (!adam) return;
  // (the fused operations are written out: a parameter whose gradient is near
  // zero moves by up to lr on the moments' last bits)
  const float m = fmaf(1.f - b1, g, b1 * M[p]);
  const float v = fmaf(g, (1.f - b2) * g, b2 * V[p]);
  M[p] = m;
  V[p] = v;
  P[p] -= lr * (m / c1) / (sqrtf(v / c2) + eps);
}

// w = (1 - alpha) softmax(o) + alpha / n (a defensive mixture with the
// uniform distribution), float64, one workgroup. A network output that is
// not finite (diverged or corrupted parameters) gives the uniform
// distribution, the mixture's defensive part, so the picks stay valid.
__global__ __launch_bounds__(256) void proposal_kernel(const float* __restrict__ o, int64_t n, double alpha,
                                                       double* __restrict__ w) {
  __shared__ double red[256];
  __shared__ int bad;
  const int tid = threadIdx.x;
  if (tid == 0) bad = 0;
  __syncthreads();
  double m = -INFINITY;
  int nonfinite = 0;
  for (int64_t j = tid; j < n; j += 256) {
    const float v = o[j];
    nonfinite |= !isfinite(v);
    m = fmax(m, (double)v);
  }
  if (nonfinite) bad = 1;  // benign race: every writer stores 1
  red[tid] = m;
  __syncthreads();
  if (bad) {
    for (int64_t j = tid; j < n; j += 256) w[j] = 1.0 / (double)n;
    return;
  }
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) red[tid] = fmax(red[tid], red[tid + s]);
    __syncthreads();
  }
  const double mx = red[0];
  __syncthreads();
  double se = 0.0;
  for (int64_t j = tid; j < n; j += 256) se += exp((double)o[j] - mx);
  red[tid] = se;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  const double z = red[0];
  for (int64_t j = tid; j < n; j += 256) w[j] = (1.0 - alpha) * exp((double)o[j] - mx) / z + alpha / (double)n;
}

unsigned nblk(int64_t n, int bs = 256) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

size_t mlp_features_ws(int64_t n1, int64_t n2) {
  const int64_t nch = (n1 + SIR - 1) / SIR, nbs = (n2 + SJS - 1) / SJS;
  return align_up(size_t(nch) * n2 * (DS + 1) * 4) + align_up(size_t(n2) * (DS + 1) * 8) +
         align_up(size_t(nbs) * (DS * DS + 1) * 8) + align_up(size_t(DS * DS + 1) * 8) + 1024;
}

int mlp_features(const float* a, int64_t n1, int64_t n2, int64_t n3, const float* phi, float* feat, void* ws,
                 hipStream_t st, double* norms) {
  if (n3 % 4) return fail(TP_EUNSUPPORTED, "feature extraction needs n3 divisible by 4");
  const size_t lds = size_t(2) * DS * sketch_ldk(n3) * 4;
  if ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(phi)) % 16)
    return fail(TP_EINVAL, "A and phi must be 16-byte aligned");
  const int64_t nch = (n1 + SIR - 1) / SIR, nb = (n2 + SJ - 1) / SJ, nbs = (n2 + SJS - 1) / SJS;
  if (nch > 65535) return fail(TP_EUNSUPPORTED, "too many horizontal slices");
  Arena ar(ws, mlp_features_ws(n1, n2));
  float* part = ar.take<float>(nch * n2 * (DS + 1));
  double* sk = ar.take<double>(n2 * (DS + 1));
  double* gpart = ar.take<double>(nbs * (DS * DS + 1));
  double* wt = ar.take<double>(DS * DS + 1);
  if (!ar.ok()) return fail(TP_EWORKSPACE, "feature workspace too small");
  const dim3 grid((unsigned)nb, (unsigned)nch);
  if (n3 <= 32)
    hipLaunchKernelGGL(sketch_mfma_pipe_kernel<2>, grid, dim3(SNT), 0, st, a, phi, n1, n2, n3, part);
  else if (n3 <= 64)
    hipLaunchKernelGGL(sketch_mfma_pipe_kernel<4>, grid, dim3(SNT), 0, st, a, phi, n1, n2, n3, part);
  else if (n3 <= 128)
    hipLaunchKernelGGL(sketch_mfma_pipe_kernel<8>, grid, dim3(SNT), 0, st, a, phi, n1, n2, n3, part);
  else
    hipLaunchKernelGGL(sketch_mfma_kernel, grid, dim3(SNT), lds, st, a, phi, n1, n2, n3, part);
  TP_LAUNCH_CHECK();
  hipLaunchKernelGGL(sketch_sum_kernel, dim3((unsigned)nbs), dim3(256), 0, st, part, nch, n2, sk, gpart);
  TP_LAUNCH_CHECK();
  hipLaunchKernelGGL(sketch_whiten_kernel, dim3(1), dim3(256), 0, st, gpart, nbs, n2, wt);
  TP_LAUNCH_CHECK();
  hipLaunchKernelGGL(sketch_apply_kernel, dim3(nblk(n2 * DIN)), dim3(256), 0, st, sk, wt, n2, feat, norms);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int mlp_forward(const float* P, const float* feat, int64_t nrows, float* out, hipStream_t st) {
  if (nrows == 0) return TP_OK;
  hipLaunchKernelGGL(mlp_forward_kernel<false>, dim3((unsigned)((nrows + TR - 1) / TR)), dim3(NT), 0, st, P, feat,
                     nrows, out, (_Float16*)nullptr, (_Float16*)nullptr);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

size_t mlp_train_ws(int64_t ntensors, int64_t nslices) {
  const int64_t rows = ntensors * nslices, ntiles = (rows + TR - 1) / TR;
  return 2 * align_up(size_t(rows) * 4) + align_up(size_t(ntiles) * NPARAM * 4) + align_up(size_t(ntensors) * 4) +
         2 * align_up(size_t(ntiles) * TR * HID * sizeof(_Float16)) + 2048;
}

int mlp_train_step(float* P, float* M, float* V, int64_t step, double lr, const float* feat, const float* target,
                   int64_t T, int64_t nsl, float* loss, float* grad_out, void* ws, hipStream_t st) {
  const int64_t rows = T * nsl, ntiles = (rows + TR - 1) / TR;
  Arena ar(ws, mlp_train_ws(T, nsl));
  float* o = ar.take<float>(rows);
  float* dout = ar.take<float>(rows);
  float* part = ar.take<float>(ntiles * NPARAM);
  float* lpart = ar.take<float>(T);
  _Float16* h1 = ar.take<_Float16>(ntiles * TR * HID);
  _Float16* h2 = ar.take<_Float16>(ntiles * TR * HID);
  if (!ar.ok()) return fail(TP_EWORKSPACE, "training workspace too small");
  if (rows > 0) {
    hipLaunchKernelGGL(mlp_forward_kernel<true>, dim3((unsigned)ntiles), dim3(NT), 0, st, P, feat, rows, o, h1, h2);
    TP_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(softmax_grad_kernel, dim3((unsigned)T), dim3(256), 0, st, o, target, nsl, T, dout, lpart);
  TP_LAUNCH_CHECK();
  hipLaunchKernelGGL(mlp_backward_kernel, dim3((unsigned)ntiles), dim3(NT), 0, st, P, feat, dout, rows, h1, h2, part);
  TP_LAUNCH_CHECK();
  const double b1 = 0.9, b2 = 0.999;
  const double c1 = 1.0 - std::pow(b1, (double)step), c2 = 1.0 - std::pow(b2, (double)step);
  hipLaunchKernelGGL(grad_adam_kernel, dim3(nblk(NPARAM, GNT) + 1), dim3(GNT), 0, st, part, ntiles, grad_out, lpart, T,
                     loss, step > 0, P, M, V, (float)lr, (float)b1, (float)b2, 1e-8f, (float)c1, (float)c2);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

int mlp_proposal(const float* logits, int64_t n, double alpha, double* w, hipStream_t st) {
  hipLaunchKernelGGL(proposal_kernel, dim3(1), dim3(256), 0, st, logits, n, alpha, w);
  TP_LAUNCH_CHECK();
  return TP_OK;
}

}  // namespace tp
