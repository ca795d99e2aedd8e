// What the tube-transform kernels share: which input tube feeds an output
// slot, and the transforms of the other files.
#pragma once

#include "common.hpp"

namespace tp {

struct FwdArgs {
  int64_t rows, cols, in_cols;
  int64_t ntubes;  // output slots: major x ld
  const int32_t* row_idx;
  const int32_t* col_idx;
  const double* row_scale;
  const double* col_scale;
  const int64_t* count;
  int64_t ld;    // slots per major index (>= cols, or >= rows when colmajor)
  int colmajor;  // slot t = col * ld + row instead of row * ld + col
  // > 0 (column-major spectra with ld a multiple of the tile): workgroup b
  // takes the tile (b / nmaj) of major index b mod nmaj, so workgroups that
  // run together read neighbouring tubes of the tube-major input instead of
  // tubes a whole input row apart
  int64_t nmaj;
};

// Input tube offset and scale of output slot t; returns false for a slot
// that is to be written as zeros (padding, or beyond the live sample count).
__device__ __forceinline__ bool tube_source(const FwdArgs& a, int64_t t, int64_t& src, double& s) {
  const int64_t maj = t / a.ld, mn = t - maj * a.ld;
  const int64_t ra = a.colmajor ? mn : maj, cb = a.colmajor ? maj : mn;
  if (ra >= a.rows || cb >= a.cols) return false;
  int64_t lim = a.count ? *a.count : INT64_MAX;
  if (a.row_idx && ra >= lim) return false;
  if (a.col_idx && cb >= lim) return false;
  const int64_t ir = a.row_idx ? a.row_idx[ra] : ra;
  const int64_t ic = a.col_idx ? a.col_idx[cb] : cb;
  src = ir * a.in_cols + ic;
  s = (a.row_scale ? a.row_scale[ra] : 1.0) * (a.col_scale ? a.col_scale[cb] : 1.0);
  return true;
}

// Launch order. Workgroup L runs on XCD L mod 8, each XCD with its own L2:
// every XCD takes a contiguous range of ceil(total / 8) logical tiles, so the
// workgroups that share cache lines (neighbouring slots) run together on one
// XCD, and the XCD's workgroups (of a grid that is a multiple of 8) walk its
// range side by side.
struct XcdWalk {
  int64_t total, q, i, step;
  __device__ XcdWalk(int64_t total_) : total(total_), q((total_ + 7) / 8), i(blockIdx.x / 8), step(gridDim.x / 8) {}
  __device__ bool next(int64_t& G) {
    G = (blockIdx.x % 8) * q + i;
    const bool ok = i < q && G < total;
    i += step;
    return ok;
  }
};
inline int64_t xcd_grid(int64_t total) { return (total + 7) / 8 * 8; }

// Transforms of many tubes per workgroup in LDS (fft_lds.hip) of lengths
// without prime factors above 13 (in n3 / 2 of an even n3), as far as LDS
// reaches. *handled is false for other lengths.
int lds_forward(const void* x, int dtype, int64_t n3, const FwdArgs& a, void* re, void* im, hipStream_t st,
                bool* handled);
int lds_inverse(const void* re, const void* im, int dtype, int64_t n3, int64_t ntubes, void* y, hipStream_t st,
                bool* handled);

// Dense products with the roots on the matrix cores (fft_dense.hip), for the
// other lengths (3 to 8192).
int dense_forward(const void* x, int dtype, int64_t n3, const FwdArgs& a, void* re, void* im, hipStream_t st);
int dense_inverse(const void* re, const void* im, int dtype, int64_t n3, int64_t ntubes, void* y, hipStream_t st);

// Four-step transforms through HBM (fft_four.hip): even lengths up to 2^19 whose
// half has no prime factor above 13. *handled is false for other lengths.
int four_forward(const void* x, int dtype, int64_t n3, const FwdArgs& a, void* re, void* im, hipStream_t st,
                 bool* handled);
int four_inverse(const void* re, const void* im, int dtype, int64_t n3, int64_t ntubes, void* y, hipStream_t st,
                 bool* handled);

}  // namespace tp
