// fp64 Cholesky factor and inverse of one block of at most 64 x 64 in LDS, by
// one 256-thread work-group on the fp64 matrix cores: the serial part of the
// per-group factors (chol.hip) and of the blocked factorization (linalg.hip).
//
// A right-looking column loop over the whole block meets at barriers several
// times per column (84 us for 64 columns with its inverse).  Here only panels
// of 16 columns are serial: one wavefront holds a row per lane and 16 columns
// in registers and passes pivots and column entries by readlane, no LDS and
// no barrier inside a panel; the rest of the block is updated by
// v_mfma_f64_16x16x4_f64.  The inverse comes from the 16 x 16 diagonal blocks
// (one per wavefront), doubled twice by matrix-core products.
//
// v_mfma_f64_16x16x4_f64, lane l: A(l % 16, l / 16), B(l / 16, l % 16), and
// element v of the result is (4 v + l / 16, l % 16), so a result is the B
// operand of a following product as it stands (element v = k-slice v).
//
// LDS blocks are row-major with stride kCholLd doubles: 16 rows at one k and
// the next, as a fragment read takes them, cover the 64 banks once.
#pragma once

#include "jarq_internal.h"

namespace jarq {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kCholLd = 66;
constexpr int kCholBlock = 64 * kCholLd;   // doubles of one LDS block

__device__ __forceinline__ f64x4 mfma_f64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ double readlane_f64(double x, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// 1 / sqrt(x): the hardware estimate and two Newton steps
// y <- y + y (1 - x y^2) / 2, each of which doubles the correct bits.
__device__ __forceinline__ double chol_rsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const double e = fma(-x * y, y, 1.0);
    y = fma(0.5 * y, e, y);
  }
  return y;
}
// 1 / x: the hardware estimate and two Newton steps y <- y + y (1 - x y).
__device__ __forceinline__ double chol_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
#pragma unroll
  for (int it = 0; it < 2; ++it) y = fma(y, fma(-x, y, 1.0), y);
  return y;
}

// A and B fragments of k-slice ks (4 wide) of a row-major LDS block:
// A(i, k) = m[r0 + i][c0 + k];  B(k, j) = m[r0 + k][c0 + j];
// B from the transpose, B(k, j) = m[r0 + j][c0 + k], is frag_a again.
__device__ __forceinline__ double frag_a(const double* m, int r0, int c0, int ks) {
  const int l = threadIdx.x & 63;
  return m[(r0 + (l & 15)) * kCholLd + c0 + 4 * ks + (l >> 4)];
}
__device__ __forceinline__ double frag_b(const double* m, int r0, int c0, int ks) {
  const int l = threadIdx.x & 63;
  return m[(r0 + 4 * ks + (l >> 4)) * kCholLd + c0 + (l & 15)];
}
__device__ __forceinline__ f64x4 load_c(const double* m, int r0, int c0) {
  const int l = threadIdx.x & 63;
  f64x4 c;
#pragma unroll
  for (int v = 0; v < 4; ++v) c[v] = m[(r0 + 4 * v + (l >> 4)) * kCholLd + c0 + (l & 15)];
  return c;
}
__device__ __forceinline__ void store_c(double* m, int r0, int c0, f64x4 c) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int v = 0; v < 4; ++v) m[(r0 + 4 * v + (l >> 4)) * kCholLd + c0 + (l & 15)] = c[v];
}

// A = L L^T in place for the n x n block (n = 32 or 64; the lower triangle is
// read; the diagonal blocks' upper parts are written as 0), dinv[k] = 1 / L(k, k).
// A pivot that is not positive and finite is replaced by 1 and sets *fail.  col:
// 128 doubles of LDS scratch.  All 256 threads call it; A is complete on return.
//
// Panel (one wavefront, lane = row): column k stays unscaled while it updates
// the later ones, a_j -= (a_k / pivot) a_k[row j].  The chain from a pivot to
// the next is reciprocal, product, readlane of one entry, multiply-add; the
// other entries go through LDS (one write, uniform 16-byte reads) and are
// applied a step later, beside the next pivot's reciprocal.  The square roots
// come at the end, a pivot per lane.
__device__ __forceinline__ void chol64_factor(double* A, int n, double* dinv, double* col,
                                              int* fail) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int c0 = 0; c0 < n; c0 += 16) {
    if (wave == 0) {
      double a[16], t[16];
      double* row = A + lane * kCholLd + c0;
#pragma unroll
      for (int k = 0; k < 16; ++k) a[k] = row[k];
      bool bad = false;
      double own = 1.0, lp = 0.0;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const double pk = readlane_f64(a[k], c0 + k);
        const bool b = !(pk > 0.0 && pk < INFINITY);
        bad |= b;
        const double piv = b ? 1.0 : pk;
        own = lane == c0 + k ? piv : own;
        // (one wavefront: its LDS accesses complete in order)
        double* ck = col + 64 * (k & 1);
        if (k < 14) ck[lane] = a[k];
        const double ip = chol_rcp(piv);
        // step k - 1 on the columns past k
#pragma unroll
        for (int j = k + 1; j < 16; ++j)
          if (k > 0) a[j] = fma(-lp, t[j], a[j]);
        lp = a[k] * ip;
        if (k < 15) a[k < 15 ? k + 1 : 15] =
            fma(-lp, readlane_f64(a[k], c0 + (k < 15 ? k + 1 : 15)), a[k < 15 ? k + 1 : 15]);
        // the reads see the other lanes' writes: not to be moved above them
        asm volatile("" ::: "memory");
#pragma unroll
        for (int j = k + 2; j < 16; ++j) t[j] = ck[c0 + j];
      }
      const double rs = chol_rsqrt(own);
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const double rk = readlane_f64(rs, c0 + k);
        a[k] = lane == c0 + k ? own * rs : (lane > c0 + k ? a[k] * rk : 0.0);
      }
      if (lane >= c0 && lane < n) {
#pragma unroll
        for (int k = 0; k < 16; ++k) row[k] = a[k];
        if (lane < c0 + 16) dinv[lane] = rs;
      }
      if (bad && lane == 0) *fail = 1;
    }
    __syncthreads();
    // trailing blocks (bi, bj), bj <= bi, dealt to the four waves
    const int b0 = c0 / 16 + 1, nb = n / 16;
    int id = 0;
    for (int bi = b0; bi < nb; ++bi)
      for (int bj = b0; bj <= bi; ++bj, ++id) {
        if ((id & 3) != wave) continue;
        f64x4 c = load_c(A, 16 * bi, 16 * bj);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          c = mfma_f64(-frag_a(A, 16 * bi, c0, ks), frag_a(A, 16 * bj, c0, ks), c);
        store_c(A, 16 * bi, 16 * bj, c);
      }
    __syncthreads();
  }
}

// X = L^{-1} (n = 32 or 64; lower triangle; the blocks above the diagonal blocks
// are not written) from the factor chol64_factor left in L and dinv.  All 256
// threads call it; X is complete on return.
__device__ __forceinline__ void chol64_invert(const double* L, int n, const double* dinv,
                                              double* X) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nb = n / 16;
  if (wave < nb) {
    // diagonal block: lane c (mod 16) solves L x = e_c
    const int r0 = 16 * wave, c = lane & 15;
    const double* Lb = L + r0 * kCholLd + r0;
    double x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      double s = i == c ? 1.0 : 0.0;
#pragma unroll
      for (int t = 0; t < i; ++t) s = fma(-Lb[i * kCholLd + t], x[t], s);
      x[i] = s * dinv[r0 + i];
    }
    if (lane < 16) {
#pragma unroll
      for (int i = 0; i < 16; ++i) X[(r0 + i) * kCholLd + r0 + c] = x[i];
    }
  }
  __syncthreads();
  // 16 -> 32: X10 = -X11 (L10 X00) for block pairs (0, 1) and (2, 3)
  if (2 * wave + 1 < nb) {
    const int r = 32 * wave + 16, c = 32 * wave;
    f64x4 t = {0.0, 0.0, 0.0, 0.0}, x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) t = mfma_f64(frag_a(L, r, c, ks), frag_b(X, c, c, ks), t);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) x = mfma_f64(-frag_a(X, r, r, ks), t[ks], x);
    store_c(X, r, c, x);
  }
  __syncthreads();
  // 32 -> 64: wave = block (bi, bj) of the lower left 32 x 32 (a zero block is
  // multiplied where bi or bj leaves one out: no branches, loads up front)
  if (nb == 4) {
    const int bj = wave & 1, bi = 2 + (wave >> 1);
    f64x4 x = {0.0, 0.0, 0.0, 0.0};
    f64x4 t[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const double b = q >= bj ? frag_b(X, 16 * q, 16 * bj, ks) : 0.0;
#pragma unroll
        for (int u = 0; u < 2; ++u) t[u] = mfma_f64(frag_a(L, 32 + 16 * u, 16 * q, ks), b, t[u]);
      }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        x = mfma_f64(2 + u <= bi ? -frag_a(X, 16 * bi, 32 + 16 * u, ks) : 0.0, t[u][ks], x);
    store_c(X, 16 * bi, 16 * bj, x);
  }
  __syncthreads();
}

}  // namespace jarq
