// Per-layer factors of the diagonal Hessian blocks (paper eq. (9)).
//
// The paper factors each group block of the design, A_i = U_i R_i (thin QR,
// no column permutation).  Only R_i enters the code update, and
// R_i^T R_i = A_i^T A_i = H_ii, so R_i is the upper Cholesky factor of H_ii
// (the Babai proposal does not depend on the row signs of R_i).  One work-group
// factors one g x g block in LDS in fp64, inverts the lower factor L_i = R_i^T,
// and writes the forms the later kernels read:
//   lfac  L_i^{-1} in fp64 (zero above the diagonal), for M = blockdiag(L^{-1}) H
//   rcol  column l, chunk c, lane j, w: R_i(m, l) / R_i(m, m) for m < l, 0
//         for m >= l, with m = j + 16 (W c + w), W = min(4, g / 16) (column l
//         of R_i above the diagonal with each row scaled by its inverse
//         diagonal, cut into chunks of W positions per lane and laid out
//         lane-contiguous, as the 16 lanes of a row own positions j + 16 t
//         and read one chunk each with one W-float access); only the chunks
//         a back-substitution step reads are kept (RcolLayout)
//   rdinv 1 / R_i(l, l),  rdsq R_i(l, l)^2,  rmat R_i (row-major).
//
// The block is one 64 x 64 (or 32 x 32) factorization of chol64.h, or for
// g = 128 two of them joined by matrix-core products:
//   L21 = A21 L11^{-T},  A22 -= L21 L21^T,  X21 = -X22 (L21 X11).
// What bounds it is the serial chain of one work-group (there are only G of
// them): 57 us at g = 128 and 21 us at g = 64, against 1062 and 229 us for a
// column loop over the whole block with barriers and fp64 divisions.
#include "chol64.h"

namespace jarq {

template <int G_SIZE>
__global__ __launch_bounds__(256) void chol_groups_kernel(const float* __restrict__ H, int cols,
                                                          double* __restrict__ lfac,
                                                          float* __restrict__ rcol,
                                                          float* __restrict__ rdinv,
                                                          float* __restrict__ rdsq,
                                                          float* __restrict__ rmat,
                                                          Flags* __restrict__ flags) {
  constexpr int g = G_SIZE;
  constexpr int n = g < 64 ? g : 64;   // edge of an LDS block
  extern __shared__ double sm[];
  double* B0 = sm;                     // A11, L11, then X22
  double* B1 = sm + kCholBlock;        // X11
  double* B2 = sm + 2 * kCholBlock;    // A21, L21 (g = 128)
  double* B3 = sm + 3 * kCholBlock;    // A22, L22 (g = 128)
  __shared__ double dinv[128];
  __shared__ __attribute__((aligned(16))) double col_s[128];
  __shared__ int fail;
  const int blk = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* Hb = H + (size_t)blk * g * cols + (size_t)blk * g;
  double* lfac_b = lfac + (size_t)blk * g * g;
  float* rcol_b = rcol + (size_t)blk * g * g;
  float* rmat_b = rmat + (size_t)blk * g * g;

  auto load = [&](double* B, int r0, int c0) {
    for (int e = tid; e < n * n / 4; e += 256) {
      const int i = e / (n / 4), j = 4 * (e % (n / 4));
      const f32x4 v = *(const f32x4*)(Hb + (size_t)(r0 + i) * cols + c0 + j);
#pragma unroll
      for (int u = 0; u < 4; ++u) B[i * kCholLd + j + u] = (double)v[u];
    }
  };
  // rcol and rmat entries of the block of L at (r0, c0)
  auto out_l = [&](const double* B, int r0, int c0) {
    using RL = RcolLayout<g>;
    constexpr int W = RL::W;
    for (int e = tid; e < n * n; e += 256) {
      // W consecutive lanes' positions of one column: m = j + 16 (W c + w)
      const int i = e / n, rem = e % n;
      const int jj = rem / W, m = c0 + (jj & 15) + 16 * (W * (jj >> 4) + rem % W);
      const int l = r0 + i;
      const int cc = (m >> 4) / W;
      rcol_b[RL::offset(l) + (cc * 16 + (m & 15)) * W + (m >> 4) % W] =
          (float)(m < l ? B[i * kCholLd + m - c0] * dinv[m] : 0.0);
    }
    for (int e = tid; e < n * n; e += 256) {
      const int j = e / n, i = e % n;
      rmat_b[(size_t)(c0 + j) * g + r0 + i] =
          (float)(r0 + i >= c0 + j ? B[i * kCholLd + j] : 0.0);
    }
  };
  // the diagonal block of L^{-1} at (r0, r0)
  auto out_x = [&](const double* X, int r0) {
    for (int e = tid; e < n * n; e += 256) {
      const int i = e / n, j = e % n;
      lfac_b[(size_t)(r0 + i) * g + r0 + j] =
          j <= i ? X[i * kCholLd + j] : 0.0;
    }
  };

  if (tid == 0) fail = 0;
  load(B0, 0, 0);
  if constexpr (g == 128) {
    load(B2, 64, 0);
    load(B3, 64, 64);
  }
  __syncthreads();
  chol64_factor(B0, n, dinv, col_s, &fail);
  out_l(B0, 0, 0);
  chol64_invert(B0, n, dinv, B1);
  out_x(B1, 0);
  if constexpr (g == 128) {
    // L21 = A21 X11^T: wave = 16 rows, all read before any is written
    {
      double a[16];
#pragma unroll
      for (int ks = 0; ks < 16; ++ks) a[ks] = frag_a(B2, 16 * wave, 0, ks);
#pragma unroll
      for (int bj = 0; bj < 4; ++bj) {
        f64x4 c = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < 4 * (bj + 1); ++ks) c = mfma_f64(a[ks], frag_a(B1, 16 * bj, 0, ks), c);
        store_c(B2, 16 * wave, 16 * bj, c);
      }
    }
    __syncthreads();
    // A22 -= L21 L21^T, lower blocks
    int id = 0;
    for (int bi = 0; bi < 4; ++bi)
      for (int bj = 0; bj <= bi; ++bj, ++id) {
        if ((id & 3) != wave) continue;
        f64x4 c = load_c(B3, 16 * bi, 16 * bj);
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
          c = mfma_f64(-frag_a(B2, 16 * bi, 0, ks), frag_a(B2, 16 * bj, 0, ks), c);
        store_c(B3, 16 * bi, 16 * bj, c);
      }
    out_l(B2, 64, 0);
    __syncthreads();
    chol64_factor(B3, 64, dinv + 64, col_s, &fail);
    out_l(B3, 64, 64);
    chol64_invert(B3, 64, dinv + 64, B0);
    out_x(B0, 64);
    // X21 = -X22 (L21 X11): wave = 16 columns; T = L21 X11 stays in registers
    {
      f64x4 t[4];
#pragma unroll
      for (int bi = 0; bi < 4; ++bi) t[bi] = f64x4{0.0, 0.0, 0.0, 0.0};
      for (int q = wave; q < 4; ++q)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const double b = frag_b(B1, 16 * q, 16 * wave, ks);
#pragma unroll
          for (int bi = 0; bi < 4; ++bi)
            t[bi] = mfma_f64(frag_a(B2, 16 * bi, 16 * q, ks), b, t[bi]);
        }
#pragma unroll
      for (int bi = 0; bi < 4; ++bi) {
        f64x4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u <= bi; ++u)
#pragma unroll
          for (int ks = 0; ks < 4; ++ks)
            x = mfma_f64(-frag_a(B0, 16 * bi, 16 * u, ks), t[u][ks], x);
#pragma unroll
        for (int v = 0; v < 4; ++v)
          lfac_b[(size_t)(64 + 16 * bi + 4 * v + (lane >> 4)) * g + 16 * wave + (lane & 15)] = x[v];
      }
    }
    // the zero blocks above the diagonal of L^{-1} and below that of R
    for (int e = tid; e < 64 * 64; e += 256) {
      const int i = e / 64, j = e % 64;
      lfac_b[(size_t)i * g + 64 + j] = 0.0;
      rmat_b[(size_t)(64 + i) * g + j] = 0.f;
    }
  }
  for (int l = tid; l < g; l += 256) {
    rdinv[(size_t)blk * g + l] = (float)dinv[l];
    rdsq[(size_t)blk * g + l] = (float)(1.0 / (dinv[l] * dinv[l]));
  }
  if (tid == 0 && fail) atomicAdd(&flags->not_spd, 1);
}

template <int G_SIZE>
static hipError_t launch_chol_t(hipStream_t st, int cols, const float* H, char* ws,
                                const Layout& lay) {
  const int G = cols / G_SIZE;
  const size_t lds = (size_t)(G_SIZE == 128 ? 4 : 2) * kCholBlock * sizeof(double);
  static std::atomic<unsigned long long> lds_set{0};
  hipError_t e = allow_dynamic_lds((const void*)chol_groups_kernel<G_SIZE>, lds, lds_set);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(chol_groups_kernel<G_SIZE>, dim3(G), dim3(256), lds, st, H, cols,
                     (double*)(ws + lay.lfac), (float*)(ws + lay.rcol),
                     (float*)(ws + lay.rdinv), (float*)(ws + lay.rdsq), (float*)(ws + lay.rmat),
                     (Flags*)(ws + lay.flags));
  return hipGetLastError();
}

// R_i rows as two fp16 terms for the objective's products: row c scaled by
// 2^t_c (its largest entry in [2^13, 2^14)), hi = fp16(x), lo = fp16(x - hi).
// One wavefront per row (g <= 128: two entries per lane).
__global__ __launch_bounds__(256) void split_r_kernel(const float* __restrict__ rmat, int nrows,
                                                      int g, _Float16* __restrict__ hi,
                                                      _Float16* __restrict__ lo,
                                                      float* __restrict__ row_inv) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (r >= nrows) return;
  const float* x = rmat + (size_t)r * g;
  const float a = lane < g ? x[lane] : 0.f;
  const float b = lane + 64 < g ? x[lane + 64] : 0.f;
  float m = fmaxf(fabsf(a), fabsf(b));
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  const int t = (m > 0.f && isfinite(m)) ? 13 - ilogbf(m) : 0;
  if (lane == 0) row_inv[r] = ldexpf(1.f, -t);
  if (lane < g) {
    const float v = ldexpf(a, t);
    const _Float16 h = (_Float16)v;
    hi[(size_t)r * g + lane] = h;
    lo[(size_t)r * g + lane] = (_Float16)(v - (float)h);
  }
  if (lane + 64 < g) {
    const float v = ldexpf(b, t);
    const _Float16 h = (_Float16)v;
    hi[(size_t)r * g + lane + 64] = h;
    lo[(size_t)r * g + lane + 64] = (_Float16)(v - (float)h);
  }
}

hipError_t launch_split_r(hipStream_t st, int cols, int g, char* ws, const Layout& lay) {
  if (g > 128) return hipErrorInvalidValue;
  const int nrows = cols;  // G groups of g rows
  hipLaunchKernelGGL(split_r_kernel, dim3((nrows + 3) / 4), dim3(256), 0, st,
                     (const float*)(ws + lay.rmat), nrows, g, (_Float16*)(ws + lay.rph),
                     (_Float16*)(ws + lay.rpl), (float*)(ws + lay.rrow));
  return hipGetLastError();
}

hipError_t launch_chol_groups(hipStream_t st, int cols, int g, const float* H, char* ws,
                              const Layout& lay) {
  switch (g) {
    case 32: return launch_chol_t<32>(st, cols, H, ws, lay);
    case 64: return launch_chol_t<64>(st, cols, H, ws, lay);
    case 128: return launch_chol_t<128>(st, cols, H, ws, lay);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace jarq
