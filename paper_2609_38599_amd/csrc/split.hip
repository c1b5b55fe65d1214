// Two-term fp16 representations for the matrix-core contractions.
//
// gfx950 has no xf32 matrix instruction; its fp16 matrix rate is 16x the fp32
// one.  A fp32 value x scaled by a power of two 2^t is written as
// hi = fp16(x 2^t), lo = fp16(x 2^t - hi), which carries 22 significant bits.
// Products of such planes accumulate in fp32 on the matrix cores.
//   H:  one scale for the whole matrix, chosen so max |H| 2^t lies in [2^13, 2^14).
//   M = blockdiag(L_i^{-1}) H, the code update's coordinates (eq. (10)): one
//       power of two per row, same rule.
//   W: one scale per row, same rule (for the layer's fixed W M^T and W_i L_i).
// Small-integer operands (codes minus zero points, code changes) are exact in fp16.
#include "jarq_internal.h"

namespace jarq {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void atomic_max_abs(float* dst, float v) {
  // |v| >= 0: IEEE ordering of non-negative floats equals their bit ordering.
  atomicMax((unsigned int*)dst, __float_as_uint(fabsf(v)));
}

__device__ __forceinline__ int pow2_exponent(float amax) {
  // t with amax * 2^t in [2^13, 2^14); 0 for an all-zero or nonfinite input.
  if (!(amax > 0.f) || !isfinite(amax)) return 0;
  return 13 - ilogbf(amax);
}

typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

// x 2^t as two fp16 terms, four values
__device__ __forceinline__ void split4(f32x4 x, int t, f16x4& hv, f16x4& lv) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float v = ldexpf(x[i], t);
    const _Float16 h = (_Float16)v;
    hv[i] = h;
    lv[i] = (_Float16)(v - (float)h);
  }
}

// A row of n x n fp32 values per work-group as two fp16 planes, scaled by 2^t
// with t from amax[row] (per_row) or amax[0]; inv[row] or inv[0] = 2^-t.
// Bound by memory traffic (4 bytes in, 4 out per value): 16-byte reads, 173 us
// at 11008 x 11008 (5.6 TB/s); one value per thread and step took 355.
template <bool kPerRow>
__global__ __launch_bounds__(256) void split_rows_kernel(const float* __restrict__ x, int n,
                                                         const float* __restrict__ amax,
                                                         _Float16* __restrict__ hi,
                                                         _Float16* __restrict__ lo,
                                                         float* __restrict__ inv) {
  const int r = blockIdx.x;
  const int t = pow2_exponent(amax[kPerRow ? r : 0]);
  if (threadIdx.x == 0 && (kPerRow || r == 0)) inv[r] = ldexpf(1.f, -t);
  const size_t row = (size_t)r * n;
  for (int c = threadIdx.x * 4; c < n; c += 1024) {
    f16x4 hv, lv;
    split4(*(const f32x4*)(x + row + c), t, hv, lv);
    *(f16x4*)(hi + row + c) = hv;
    *(f16x4*)(lo + row + c) = lv;
  }
}

// H as two planes (after launch_split_m, which leaves max |H| and uses the
// planes' memory).
hipError_t launch_split_h(hipStream_t st, int cols, const float* H, char* ws, const Layout& lay) {
  float* hs = (float*)(ws + lay.hscale);
  hipLaunchKernelGGL(split_rows_kernel<false>, dim3(cols), dim3(256), 0, st, H, cols, hs + 1,
                     (_Float16*)(ws + lay.hhi), (_Float16*)(ws + lay.hlo), hs);
  return hipGetLastError();
}

// M = blockdiag(L_i^{-1}) H.  Row n of M (group i = n / g, local index nl) is
// sum_{m <= nl} L_i^{-1}(nl, m) H(i g + m, :): the residual product with M in place
// of H gives u = L_i^{-1} (H e)_i for every group at once, and its blocks
// M(i-block, h-block) = L_i^{-1} H_ih carry a code change of group h into u_i.
// Formed in fp64 from the fp64 inverse, rounded to fp32 into a temporary, with
// each row's maximum (then split with one scale per row) and the largest |H|.
//
// On the fp64 matrix cores (v_mfma_f64_16x16x4_f64, 64 cycles each): a
// work-group stages L_i^{-1} in LDS once and takes `span` columns, a
// wavefront 16 columns at a time with all g rows of M in registers; the
// 16 x 16 blocks above the diagonal of L_i^{-1} are skipped.  One LDS read per
// matrix instruction (row stride g + 2 doubles: the 16 rows and the k-pairs
// of a read cover the 64 banks once) leaves the matrix rate as the bound:
// 59 us at 4096 columns and 498 us at 11008 (g = 128; 35 TFLOP/s of the 70 the
// fp64 matrix cores sustain, counting the blocks computed), against 875 and
// 6584 us for one column per thread with fp64 vector FMAs.
//
// span: 512, less (a multiple of 128) where that leaves compute units without
// a work-group (2048 columns, g = 128: 35 us; always 512: 55).
static int form_span(int cols, int g) {
  int span = 512;
  while (span > 128 && (long long)((cols + span - 1) / span) * (cols / g) < 256) span /= 2;
  return span;
}

// (g = 128 keeps five registers a lane in scratch around the column loop.)
template <int G_SIZE>
__global__ __launch_bounds__(512) void form_m_kernel(const float* __restrict__ H, int cols,
                                                     const double* __restrict__ linv,
                                                     float* __restrict__ mtmp,
                                                     float* __restrict__ rowmax,
                                                     float* __restrict__ hmax,
                                                     int span) {
  constexpr int g = G_SIZE;
  constexpr int LD = g + 2;
  constexpr int NB = g / 16;
  extern __shared__ double li[];
  __shared__ float hmax_s[8];
  const int i = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lc = lane & 15, lk = lane >> 4;
  const double* Li = linv + (size_t)i * g * g;
  typedef double f64x2 __attribute__((ext_vector_type(2)));
  for (int e = tid; e < g * g / 2; e += 512) {
    const int r = e / (g / 2), c = 2 * (e % (g / 2));
    *(f64x2*)(li + r * LD + c) = *(const f64x2*)(Li + r * g + c);
  }
  __syncthreads();
  const int cend = min(cols, (int)(blockIdx.x + 1) * span);
  // B(k, j) of k-slice ks: H(i g + 4 ks + lane / 16, c + lane % 16)
  // (wave-uniform bases, 32-bit offsets: g rows of at most 16384 columns)
  const float* Hi = H + (size_t)i * g * cols;
  float* Mi = mtmp + (size_t)i * g * cols;
  const uint32_t ucols = (uint32_t)cols, lane_at = (uint32_t)lk * ucols + (uint32_t)lc;
  float h[4 * NB];
  auto fetch = [&](int c, int ks) {
    return Hi[lane_at + (uint32_t)c + (uint32_t)(4 * ks) * ucols];
  };
  float mx[NB][4], ha = 0.f;
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) mx[b][v] = 0.f;
  int c = blockIdx.x * span + 16 * wave;   // cols is a multiple of 16
  if (c < cend) {
#pragma unroll
    for (int ks = 0; ks < 4 * NB; ++ks) h[ks] = fetch(c, ks);
  }
  for (; c < cend; c += 128) {
    // L^{-1} stays in LDS (the compiler would keep it in registers across the
    // columns, and spill)
    asm volatile("" ::: "memory");
    // the next columns, each value loaded as its predecessor is used (the
    // last pass loads its own again)
    const int cn = c + 128 < cend ? c + 128 : c;
    f64x4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < 4 * NB; ++ks) {
      ha = fmaxf(ha, fabsf(h[ks]));
      const double hb = (double)h[ks];
      h[ks] = fetch(cn, ks);
#pragma unroll
      for (int b = ks / 4; b < NB; ++b)
        acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(li[(16 * b + lc) * LD + 4 * ks + lk], hb,
                                                      acc[b], 0, 0, 0);
      if (ks % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    // element v: row 16 b + 4 v + lane / 16, column c + lane % 16
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float m = (float)acc[b][v];
        mx[b][v] = fmaxf(mx[b][v], fabsf(m));
        Mi[lane_at + (uint32_t)c + (uint32_t)(16 * b + 4 * v) * ucols] = m;
      }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float m = mx[b][v];
#pragma unroll
      for (int off = 8; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
      if (lc == 0) atomic_max_abs(rowmax + i * g + 16 * b + 4 * v + lk, m);
    }
  // one atomic per work-group (they all meet at one address)
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) ha = fmaxf(ha, __shfl_xor(ha, off));
  if (lane == 0) hmax_s[wave] = ha;
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int w = 1; w < 8; ++w) ha = fmaxf(ha, hmax_s[w]);
    atomic_max_abs(hmax, ha);
  }
}

template <int G_SIZE>
static hipError_t launch_split_m_t(hipStream_t st, int cols, const float* H, char* ws,
                                   const Layout& lay) {
  // The H planes (written afterwards by launch_split_h) serve as the fp32
  // temporary: together they span cols * cols * 4 bytes.
  float* mtmp = (float*)(ws + lay.hhi);
  float* rowmax = (float*)(ws + lay.mmax);
  float* hmax = (float*)(ws + lay.hscale) + 1;
  const size_t lds = (size_t)G_SIZE * (G_SIZE + 2) * sizeof(double);
  static std::atomic<unsigned long long> lds_set{0};
  const hipError_t e = allow_dynamic_lds((const void*)form_m_kernel<G_SIZE>, lds, lds_set);
  if (e != hipSuccess) return e;
  const int span = form_span(cols, G_SIZE);
  const dim3 grid((cols + span - 1) / span, cols / G_SIZE);
  hipLaunchKernelGGL(form_m_kernel<G_SIZE>, grid, dim3(512), lds, st, H, cols,
                     (const double*)(ws + lay.lfac), mtmp, rowmax, hmax, span);
  hipLaunchKernelGGL(split_rows_kernel<true>, dim3(cols), dim3(256), 0, st, mtmp, cols, rowmax,
                     (_Float16*)(ws + lay.mhi), (_Float16*)(ws + lay.mlo),
                     (float*)(ws + lay.mrow));
  return hipGetLastError();
}

hipError_t launch_split_m(hipStream_t st, int cols, int g, const float* H, char* ws,
                          const Layout& lay) {
  switch (g) {
    case 32: return launch_split_m_t<32>(st, cols, H, ws, lay);
    case 64: return launch_split_m_t<64>(st, cols, H, ws, lay);
    case 128: return launch_split_m_t<128>(st, cols, H, ws, lay);
    default: return hipErrorInvalidValue;
  }
}

// W as two fp16 planes for the layer's constant products (T = W M^T and
// RW = W_i L_i, formed once by jarq_prepare): one work-group per row, the
// row maximum, then the planes and the row's inverse scale 2^-t.  Each thread
// keeps its NCH chunks of four weights in registers between the two passes
// (rows of at most 1024 NCH columns), so W is read once.
template <int NCH>
__global__ __launch_bounds__(256) void split_w_kernel(int cols, const float* __restrict__ W,
                                                      _Float16* __restrict__ whi,
                                                      _Float16* __restrict__ wlo,
                                                      float* __restrict__ wrow_inv) {
  const int row = blockIdx.x;
  __shared__ float red[4];
  const float* wr = W + (size_t)row * cols;
  f32x4 wv[NCH];
  float m = 0.f;
#pragma unroll
  for (int k = 0; k < NCH; ++k) {
    const int c = (threadIdx.x + 256 * k) * 4;
    if (c < cols) {
      wv[k] = *(const f32x4*)(wr + c);
#pragma unroll
      for (int i = 0; i < 4; ++i) m = fmaxf(m, fabsf(wv[k][i]));
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  const int t = pow2_exponent(m);
  if (threadIdx.x == 0) wrow_inv[row] = ldexpf(1.f, -t);
  _Float16* hr = whi + (size_t)row * cols;
  _Float16* lr = wlo + (size_t)row * cols;
  typedef _Float16 h4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int k = 0; k < NCH; ++k) {
    const int c = (threadIdx.x + 256 * k) * 4;
    if (c < cols) {
      h4 hv, lv;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = ldexpf(wv[k][i], t);
        const _Float16 h = (_Float16)e;
        hv[i] = h;
        lv[i] = (_Float16)(e - (float)h);
      }
      *(h4*)(hr + c) = hv;
      *(h4*)(lr + c) = lv;
    }
  }
}

hipError_t launch_split_w(hipStream_t st, int rows, int cols, const float* W, _Float16* whi,
                          _Float16* wlo, float* wrow_inv) {
  if (rows <= 0) return hipSuccess;
  if (cols <= 4096)
    hipLaunchKernelGGL(split_w_kernel<4>, dim3(rows), dim3(256), 0, st, cols, W, whi, wlo, wrow_inv);
  else if (cols <= 12288)
    hipLaunchKernelGGL(split_w_kernel<12>, dim3(rows), dim3(256), 0, st, cols, W, whi, wlo, wrow_inv);
  else if (cols <= 16384)   // the most a layer can have: 128 groups of at most 128
    hipLaunchKernelGGL(split_w_kernel<16>, dim3(rows), dim3(256), 0, st, cols, W, whi, wlo, wrow_inv);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// cz = q - z as fp16 (exact: codes and zero points are small integers), by
// layer row; 16 codes per thread and step.  With flags, also the checks of a
// run's inputs: codes at most qmax, |z| at most 1024 (q - z and 1024 + z stay
// exact in fp16).
__global__ void codes_cz_kernel(int rows, int cols, int g, int qmax,
                                const uint8_t* __restrict__ codes,
                                const int32_t* __restrict__ zeros, _Float16* __restrict__ cz,
                                Flags* __restrict__ flags) {
  const int sh = __ffs(g) - 5;   // g / 16 pieces a group, a power of two
  const size_t chunks = (size_t)rows * cols / 16;
  int bad_q = 0, bad_z = 0;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < chunks;
       e += (size_t)gridDim.x * blockDim.x) {
    const size_t off = e * 16;
    const uint4 q = *(const uint4*)(codes + off);
    const int zi = zeros[e >> sh];
    const float z = (float)zi;
    bad_z += zi > 1024 || zi < -1024;
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
    f16x8 h0, h1;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const int q0 = (int)((w[b >> 2] >> (8 * (b & 3))) & 0xffu);
      const int q1 = (int)((w[2 + (b >> 2)] >> (8 * (b & 3))) & 0xffu);
      bad_q += (q0 > qmax) + (q1 > qmax);
      h0[b] = (_Float16)((float)q0 - z);
      h1[b] = (_Float16)((float)q1 - z);
    }
    *(f16x8*)(cz + off) = h0;
    *(f16x8*)(cz + off + 8) = h1;
  }
  if (flags != nullptr) {
    if (bad_q) atomicAdd(&flags->bad_codes, bad_q);
    if (bad_z) atomicAdd(&flags->bad_zeros, bad_z);
  }
}

hipError_t launch_codes_cz(hipStream_t st, int rows, int cols, int g, int bits,
                           const uint8_t* codes, const int32_t* zeros, _Float16* cz,
                           Flags* flags) {
  if (rows <= 0 || cols % 16 != 0) return rows <= 0 ? hipSuccess : hipErrorInvalidValue;
  const size_t blocks = ((size_t)rows * cols / 16 + 255) / 256;
  hipLaunchKernelGGL(codes_cz_kernel, dim3((unsigned)(blocks < 2048 ? blocks : 2048)), dim3(256), 0,
                     st, rows, cols, g, (1 << bits) - 1, codes, zeros, cz, flags);
  return hipGetLastError();
}

}  // namespace jarq
