// Products on fp32 matrix cores.
//
// wh_kernel: W H of the scale right-hand sides (prepare; paper App. G.8), from
// the layer's T = W M^T.  M = blockdiag(L_i^{-1}) H, so group i's columns of W H
// are T_i L_i^T: g multiplies a value instead of the cols of the product with H.
//
// gemm_ah_kernel: the row objectives e_j^T H e_j of the stand-alone
// jarq_objective (paper Sec. 3.3.2 and eq. (7)), from E H of every row; the
// sweep's own residual product runs on fp16 matrix cores (sgemm.hip).
// E = W - What with What = s_i (q - z_i) is formed on the fly from the codes,
// scales and zero points (eq. (1)); the epilogue writes, per row and 64-column
// slice, sum_c E(row, c) (E H)(row, c) in fp64.
//
// Tiling: 128 x 128 output tile per 256-thread work-group, 2 x 2 waves of
// 64 x 64, each a 2 x 2 grid of v_mfma_f32_32x32x2f32 accumulators.  H is
// symmetric, so the B operand B(k, n) = H(k, n) is read as H(n, k): every lane
// loads four consecutive k of one A row and one H row (16-byte loads); MFMA
// step t of a chunk of 8 takes k = k0 + 4 * (lane / 32) + t, the same
// permutation for A and B.
#include "jarq_internal.h"

namespace jarq {

namespace {

__device__ __forceinline__ f32x4 load_e4(const float* __restrict__ W,
                                         const uint8_t* __restrict__ codes,
                                         const float* __restrict__ scales,
                                         const int32_t* __restrict__ zeros, int row, int rows,
                                         int k, int cols, int g, int G) {
  if (row >= rows) return f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 w = *(const f32x4*)(W + (size_t)row * cols + k);
  const uint32_t q4 = *(const uint32_t*)(codes + (size_t)row * cols + k);
  const int grp = k / g;
  const float s = scales[(size_t)row * G + grp];
  const int z = zeros[(size_t)row * G + grp];
  w.x -= s * (float)((int)(q4 & 0xffu) - z);
  w.y -= s * (float)((int)((q4 >> 8) & 0xffu) - z);
  w.z -= s * (float)((int)((q4 >> 16) & 0xffu) - z);
  w.w -= s * (float)((int)(q4 >> 24) - z);
  return w;
}

__device__ __forceinline__ f32x4 load_h4(const float* __restrict__ H, int n, int cols, int k) {
  if (n >= cols) return f32x4{0.f, 0.f, 0.f, 0.f};
  return *(const f32x4*)(H + (size_t)n * cols + k);
}

__device__ __forceinline__ float elem_e(const float* __restrict__ W,
                                        const uint8_t* __restrict__ codes,
                                        const float* __restrict__ scales,
                                        const int32_t* __restrict__ zeros, int row, int col,
                                        int cols, int g, int G) {
  const float w = W[(size_t)row * cols + col];
  const int grp = col / g;
  const float s = scales[(size_t)row * G + grp];
  const int z = zeros[(size_t)row * G + grp];
  return w - s * (float)((int)codes[(size_t)row * cols + col] - z);
}

}  // namespace

__global__ __launch_bounds__(256, 2) void gemm_ah_kernel(int rows, int cols, int g,
                                                         const float* __restrict__ W,
                                                         const uint8_t* __restrict__ codes,
                                                         const float* __restrict__ scales,
                                                         const int32_t* __restrict__ zeros,
                                                         const float* __restrict__ H,
                                                         double* __restrict__ objpart) {
  const int G = cols / g;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int lm = lane & 31, kh = lane >> 5;
  const int m0 = blockIdx.y * 128 + wm * 64;
  const int n0 = blockIdx.x * 128 + wn * 64;
  const int ra0 = m0 + lm, ra1 = m0 + 32 + lm;
  const int cb0 = n0 + lm, cb1 = n0 + 32 + lm;

  f32x16 acc00 = {}, acc01 = {}, acc10 = {}, acc11 = {};

  f32x4 a0 = load_e4(W, codes, scales, zeros, ra0, rows, 4 * kh, cols, g, G);
  f32x4 a1 = load_e4(W, codes, scales, zeros, ra1, rows, 4 * kh, cols, g, G);
  f32x4 b0 = load_h4(H, cb0, cols, 4 * kh);
  f32x4 b1 = load_h4(H, cb1, cols, 4 * kh);
  for (int k0 = 0; k0 < cols; k0 += 8) {
    const int kn = k0 + 8 + 4 * kh;
    f32x4 na0, na1, nb0, nb1;
    const bool more = (k0 + 8) < cols;
    if (more) {
      na0 = load_e4(W, codes, scales, zeros, ra0, rows, kn, cols, g, G);
      na1 = load_e4(W, codes, scales, zeros, ra1, rows, kn, cols, g, G);
      nb0 = load_h4(H, cb0, cols, kn);
      nb1 = load_h4(H, cb1, cols, kn);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      acc00 = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[t], b0[t], acc00, 0, 0, 0);
      acc01 = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[t], b1[t], acc01, 0, 0, 0);
      acc10 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[t], b0[t], acc10, 0, 0, 0);
      acc11 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[t], b1[t], acc11, 0, 0, 0);
    }
    if (more) {
      a0 = na0;
      a1 = na1;
      b0 = nb0;
      b1 = nb1;
    }
  }

  // Accumulator layout of a 32x32 block: element v of lane l is
  // (row 8 * (v / 4) + 4 * (l / 32) + v % 4, column l % 32).
  const f32x16* accs[2][2] = {{&acc00, &acc01}, {&acc10, &acc11}};
  const int nt = (cols + kObjTile - 1) / kObjTile;
#pragma unroll
  for (int mb = 0; mb < 2; ++mb) {
    double part[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) part[v] = 0.0;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const int col = n0 + nb * 32 + lm;
      const f32x16 a = *accs[mb][nb];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = m0 + mb * 32 + 8 * (v / 4) + 4 * kh + (v % 4);
        if (row < rows && col < cols) {
          const float e = elem_e(W, codes, scales, zeros, row, col, cols, g, G);
          part[v] += (double)e * (double)a[v];
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      double x = part[v];
#pragma unroll
      for (int off = 16; off >= 1; off >>= 1) x += __shfl_xor(x, off);
      part[v] = x;
    }
    if (lm == 0) {
      const int slice = n0 / kObjTile;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = m0 + mb * 32 + 8 * (v / 4) + 4 * kh + (v % 4);
        if (row < rows && slice < nt) objpart[(size_t)row * nt + slice] = part[v];
      }
    }
  }
}

hipError_t launch_row_products(hipStream_t st, int rows, int cols, int g, const float* W,
                               const uint8_t* codes, const float* scales, const int32_t* zeros,
                               const float* H, double* objpart) {
  dim3 grid((cols + 127) / 128, (rows + 127) / 128);
  hipLaunchKernelGGL(gemm_ah_kernel, grid, dim3(256), 0, st, rows, cols, g, W, codes, scales,
                     zeros, H, objpart);
  return hipGetLastError();
}

// WH(r, n) = sum_{m <= n} T(r, m) L_i(n, m) over the columns of group i, with
// L_i(n, m) = R_i(m, n) (rmat).  Work-group: 128 rows x one group, R_i staged
// in LDS; a wavefront takes 32 rows, with the rows' T values of the group in
// registers, four consecutive k a lane: step t of a chunk of 8 takes k =
// 4 (lane / 32) + t, in both operands.  Blocks of 32 columns skip the k past
// their own (R_i is upper triangular).  Bound by reading T and writing W H
// (8 bytes a value): 176 us for 4096 x 11008 at g = 128 (2.1 TB/s), where the
// fp32 product with H took 17.8 ms, and nearer to the 64-bit value (scales of
// that layer 5.3e-7 off instead of 1.1e-6): T's sums have fewer fp32 roundings.
template <int G_SIZE>
__global__ __launch_bounds__(256) void wh_kernel(int rows, int cols, const float* __restrict__ T,
                                                 const float* __restrict__ rmat,
                                                 float* __restrict__ WH) {
  constexpr int g = G_SIZE;
  constexpr int NB = g / 32, KC = g / 8;
  __shared__ float r_s[g * g];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lm = lane & 31, kh = lane >> 5;
  const int i = blockIdx.x;
  const float* Ri = rmat + (size_t)i * g * g;
  const int r0 = blockIdx.y * 128 + 32 * wave;
  const int row = r0 + lm < rows ? r0 + lm : rows - 1;   // past the end: never stored
  const float* t_row = T + (size_t)row * cols + (size_t)i * g + 4 * kh;
  f32x4 a[KC];
#pragma unroll
  for (int kc = 0; kc < KC; ++kc) a[kc] = *(const f32x4*)(t_row + 8 * kc);
  for (int e = tid; e < g * g / 4; e += 256) *(f32x4*)(r_s + 4 * e) = *(const f32x4*)(Ri + 4 * e);
  __syncthreads();
  f32x16 acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = f32x16{};
#pragma unroll
  for (int kc = 0; kc < KC; ++kc)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
      for (int b = kc / 4; b < NB; ++b)
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(
            a[kc][t], r_s[(8 * kc + 4 * kh + t) * g + 32 * b + lm], acc[b], 0, 0, 0);
    }
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = r0 + 8 * (v / 4) + 4 * kh + (v % 4);
      if (r < rows) WH[(size_t)r * cols + (size_t)i * g + 32 * b + lm] = acc[b][v];
    }
}

hipError_t launch_wh(hipStream_t st, int rows, int cols, int g, char* ws, const Layout& lay) {
  const float* T = (const float*)(ws + lay.tm);
  const float* rmat = (const float*)(ws + lay.rmat);
  float* WH = (float*)(ws + lay.wh);
  const dim3 grid(cols / g, (rows + 127) / 128);
  switch (g) {
    case 32: hipLaunchKernelGGL(wh_kernel<32>, grid, dim3(256), 0, st, rows, cols, T, rmat, WH); break;
    case 64: hipLaunchKernelGGL(wh_kernel<64>, grid, dim3(256), 0, st, rows, cols, T, rmat, WH); break;
    case 128: hipLaunchKernelGGL(wh_kernel<128>, grid, dim3(256), 0, st, rows, cols, T, rmat, WH); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace jarq
