// Per-layer setup before the refinement path: the damped Hessian from its
// accumulator (hessian.hip) and the round-to-nearest host.
//
// hessian_finalize_* writes the fp32 H the refinement path reads:
// Hacc + (damp mean(diag Hacc) + nu^2) I.
//
// RTN host (App. A.1 names asymmetric group-wise round-to-nearest without a
// formula; the min/max reading with 0 forced into the range):
//   lo = min(min_group, 0), hi = max(max_group, 0), s = (hi - lo) / (2^b - 1)
//   (s = 1 when hi == lo), z = clip(rint(-lo / s), 0, 2^b - 1),
//   q = clip(rint(w / s) + z, 0, 2^b - 1),
// with s rounded to fp32 first and z, q computed on the stored grid in fp64
// (correctly rounded division and rint), so every code is exact.
#include "jarq_internal.h"

namespace jarq {

// Off-diagonal entries: H = (float) Hacc.
__global__ __launch_bounds__(256) void hessian_finalize_offdiag_kernel(const double* __restrict__ Hacc,
                                                                       int d,
                                                                       float* __restrict__ H) {
  const size_t n = (size_t)d * d;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    if (e % (size_t)(d + 1) != 0) H[e] = (float)Hacc[e];
  }
}

// Diagonal: H_ii = (float)(Hacc_ii + damp mean(diag Hacc) + nu2), one work-group.
__global__ __launch_bounds__(1024) void hessian_finalize_diag_kernel(const double* __restrict__ Hacc,
                                                                     int d, double damp, double nu2,
                                                                     float* __restrict__ H) {
  __shared__ double red[16];
  double s = 0.0;
  for (int i = threadIdx.x; i < d; i += 1024) s += Hacc[(size_t)i * (d + 1)];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  double tot = 0.0;
  for (int w = 0; w < 16; ++w) tot += red[w];
  const double add = damp * (tot / (double)d) + nu2;
  for (int i = threadIdx.x; i < d; i += 1024)
    H[(size_t)i * (d + 1)] = (float)(Hacc[(size_t)i * (d + 1)] + add);
}

hipError_t launch_hessian_finalize(hipStream_t st, const double* Hacc, int d, double damp,
                                   double nu2, float* H) {
  const size_t n = (size_t)d * d;
  const size_t blocks = (n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192;
  hipLaunchKernelGGL(hessian_finalize_offdiag_kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                     Hacc, d, H);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(hessian_finalize_diag_kernel, dim3(1), dim3(1024), 0, st, Hacc, d, damp, nu2,
                     H);
  return hipGetLastError();
}

// g / 4 lanes per group, four weights a lane: 16-byte reads along the row, the
// group's range by a reduction over its lanes.  w / s is the correctly rounded
// quotient as a division gives it: q0 = w (1 / s), then q0 + (w - q0 s) (1 / s)
// with fused multiply-adds, q0 held to the codes' range first so that an
// infinity keeps its sign (a NaN takes code 0 either way).  Bound by memory
// traffic and by two fp64 divisions a lane: 6.1 us at 1000 x 2752, g = 32 (a
// lane per group with a division per weight: 11).
template <int g>
__global__ __launch_bounds__(256) void rtn_kernel(const float* __restrict__ W, long long groups,
                                                  int bits, uint8_t* __restrict__ codes,
                                                  float* __restrict__ scales,
                                                  int32_t* __restrict__ zeros) {
  constexpr int LPG = g / 4;   // 8, 16 or 32 lanes
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long e = t / LPG;
  if (e >= groups) return;     // whole groups of lanes
  const int l = (int)(t % LPG);
  const double qmax = (double)((1 << bits) - 1);
  const f32x4 w = *(const f32x4*)(W + e * g + 4 * l);
  // min and max are exact in fp32
  float lo = fminf(0.f, fminf(fminf(w.x, w.y), fminf(w.z, w.w)));
  float hi = fmaxf(0.f, fmaxf(fmaxf(w.x, w.y), fmaxf(w.z, w.w)));
#pragma unroll
  for (int off = LPG / 2; off >= 1; off >>= 1) {
    lo = fminf(lo, __shfl_xor(lo, off));
    hi = fmaxf(hi, __shfl_xor(hi, off));
  }
  const double s = hi > lo ? ((double)hi - (double)lo) / qmax : 1.0;
  const float s32 = (float)s;
  const double s64 = (double)s32;
  const double z = fmin(fmax(rint(-(double)lo / s64), 0.0), qmax);
  const double sinv = 1.0 / s64, dlo = -z, dhi = qmax - z;
  uint32_t packed = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double x = (double)w[i];
    const double q0 = fmin(fmax(x * sinv, dlo), dhi);
    const double q1 = fma(fma(-q0, s64, x), sinv, q0);
    packed |= (uint32_t)(fmin(fmax(rint(q1), dlo), dhi) + z) << (8 * i);
  }
  *(uint32_t*)(codes + e * g + 4 * l) = packed;
  if (l == 0) {
    scales[e] = s32;
    zeros[e] = (int32_t)z;
  }
}

hipError_t launch_rtn(hipStream_t st, const float* W, int rows, int cols, int g, int bits,
                      uint8_t* codes, float* scales, int32_t* zeros) {
  const long long groups = (long long)rows * (cols / g);
  const dim3 grid((unsigned)((groups * (g / 4) + 255) / 256));
  switch (g) {
    case 32: hipLaunchKernelGGL(rtn_kernel<32>, grid, dim3(256), 0, st, W, groups, bits, codes, scales, zeros); break;
    case 64: hipLaunchKernelGGL(rtn_kernel<64>, grid, dim3(256), 0, st, W, groups, bits, codes, scales, zeros); break;
    case 128: hipLaunchKernelGGL(rtn_kernel<128>, grid, dim3(256), 0, st, W, groups, bits, codes, scales, zeros); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace jarq
