// GPTQ-style host on the GPU: the starting state (S0, Q0, Z) from sequential
// error compensation (App. A.1 names GPTQ as a host; its recursion is the
// nearest-plane relation of App. G.7), columns in their natural order, the
// grid of each group fixed at its first column from the compensated weights by
// the min/max rule of the RTN host.
//
// Formulation without any inverse.  Let M be the lower-triangular matrix with
// M^T M = H; with J the order-reversing permutation, J H J = C C^T (C lower,
// the ordinary Cholesky factor) and M = J C^T J.  With e = w - what (original
// weights minus quantized ones), GPTQ's update rule is equivalent to
//   column k is rounded from  w_k + (sum_{i<k} M_ki e_i) / M_kk,
// and the compensated weights of a whole group G at its first column are
//   w_G + M_GG^{-1} (M_GP e_P),   P = the columns before G
// (the group's block of the triangular system restricted to the prefix).
//
// comp [rows][cols] holds sum_i M_ki e_i over the columns i handled so far.
// Columns go in panels of kPanel: before a group the contributions of the
// panel's earlier groups are added (one product of at most kPanel columns),
// after a panel those of the whole panel to every later column, so most of the
// rows cols^2 work is in a few large products (linalg.hip).  A group's errors
// take the place of its sums.  The triangular parts run per row, sixteen lanes
// per row.
#include "jarq_internal.h"

namespace jarq {

namespace {
constexpr int kPanel = 512;   // columns per panel, a multiple of every group size

template <int V>
struct Step {
  static constexpr int value = V;
};
template <int K, int N>
struct Steps {
  template <typename F>
  static __device__ __forceinline__ void run(F&& f) {
    if constexpr (K < N) {
      f(Step<K>{});
      Steps<K + 1, N>::run(f);
    }
  }
};

// Value of lane JL of each row of 16 lanes, in every lane of that row.
template <int JL>
__device__ __forceinline__ double row_share(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x150 + JL, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x150 + JL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
}  // namespace

size_t gptq_workspace_bytes(int rows, int cols, int g) {
  const size_t R = rows, C = cols;
  auto a = [](size_t x) { return (x + 255) & ~size_t(255); };
  return a(C * C * 8) + a(C * C * 8) + a(R * C * 8) + a(2 * 64 * 64 * 8) + a(4);
}

// Sixteen lanes per row (blockDim / 16 rows per work-group): lane j owns the
// group positions n = j + 16 t (t = 0 .. g/16 - 1) and keeps their sums in
// registers.  The g sequential steps are column-oriented: at step n every lane
// forms the candidate value of its own position, that of the owner reaches the
// row by a DPP broadcast, and each lane subtracts or adds M(m, n) times it to
// the sums of its positions m > n.  (A dot product over the row's lanes at
// every step, with an fp64 division on it, made a chain about six times as
// long: 86 us for 4096 rows at g = 128, now 25.)  Nothing is recorded at a
// step: a position's sum is final once its step has come, so its value is
// formed again from it afterwards.
// Pass 1: y = M_GG^{-1} c and the group's grid from w + y (0 forced into the
// range); pass 2: the columns in order, each rounded from
// w_m + (c_m + sum_{n<m} M_mn e_n) / M_mm.
// M_GG sits in LDS column by column with its rows divided by their diagonal
// (element (m, n) / M_mm at n (g + 1) + m, zero on and above the diagonal), so
// the lanes of a row read consecutive values and the sums are kept divided
// too: no multiplication by 1 / M_mm is left on the chain.
//
// x / s of the rounding is the correctly rounded quotient, as a division
// gives it: q0 = x (1 / s), then q0 + (x - q0 s) (1 / s) with fused
// multiply-adds; q0 is held to the codes' range first, so that an infinite x
// keeps its sign (a NaN rounds to code 0 either way).
template <int G_SIZE>
__global__ __launch_bounds__(512) void gptq_group_kernel(int rows, int cols, int bits, int grp,
                                                         const float* __restrict__ W,
                                                         const double* __restrict__ M,
                                                         double* __restrict__ comp, int has_comp,
                                                         uint8_t* __restrict__ codes,
                                                         float* __restrict__ scales,
                                                         int32_t* __restrict__ zeros) {
  constexpr int g = G_SIZE;
  constexpr int NT = g / 16;
  constexpr int LD = g + 1;
  extern __shared__ double mc[];     // g x LD, then 1 / M_mm of the g rows
  double* minv = mc + g * LD;
  const int tid = threadIdx.x;
  const int j = tid & 15;
  const int r = blockIdx.x * (blockDim.x >> 4) + (tid >> 4);
  const bool live = r < rows;
  const int rr = live ? r : rows - 1;
  const int b0 = grp * g;
  const int G = cols / g;
  const double qmax = (double)((1 << bits) - 1);
  double cl[NT], wl[NT], acc[NT];
  {
    const float* w = W + (long long)rr * cols + b0 + j;
    const double* c = comp + (long long)rr * cols + b0 + j;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      wl[t] = (double)w[16 * t];
      cl[t] = has_comp ? c[16 * t] : 0.0;
    }
  }
  if (tid < g) minv[tid] = 1.0 / M[(long long)(b0 + tid) * (cols + 1)];
  __syncthreads();
  {
    // M_GG by rows, two values a load, eight loads in flight a thread (the
    // part above the diagonal is read and dropped)
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    constexpr int NE = g * g / 2, BATCH = NE < 2048 ? NE / 256 : 8;
    const double* Mg = M + (long long)b0 * cols + b0;
    for (int e0 = tid; e0 < NE; e0 += BATCH * blockDim.x) {
      f64x2 v[BATCH];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int e = min(e0 + u * (int)blockDim.x, NE - 1);
        v[u] = *(const f64x2*)(Mg + (long long)(e / (g / 2)) * cols + 2 * (e % (g / 2)));
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int e = e0 + u * (int)blockDim.x;
        if (e < NE) {
          const int m = e / (g / 2), n = 2 * (e % (g / 2));
          const double im = minv[m];
#pragma unroll
          for (int q = 0; q < 2; ++q) mc[(n + q) * LD + m] = n + q < m ? v[u][q] * im : 0.0;
        }
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < NT; ++t) cl[t] *= minv[j + 16 * t];

  // pass 1: y = M_GG^{-1} c
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = cl[t];
  Steps<0, g>::run([&](auto nc) __attribute__((always_inline)) {
    constexpr int n = decltype(nc)::value;
    const double y = row_share<n % 16>(acc[n / 16]);
#pragma unroll
    for (int t = n / 16; t < NT; ++t) acc[t] = fma(-mc[n * LD + j + 16 * t], y, acc[t]);
  });
  double lo = 0.0, hi = 0.0;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const double v = wl[t] + acc[t];
    lo = fmin(lo, v);
    hi = fmax(hi, v);
  }
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off));
    hi = fmax(hi, __shfl_xor(hi, off));
  }
  const double s = hi > lo ? (hi - lo) / qmax : 1.0;
  const float s32 = (float)s;
  const double s64 = (double)s32;
  const double zp = fmin(fmax(rint(-lo / s64), 0.0), qmax);
  const double sinv = 1.0 / s64;
  const double dlo = -zp, dhi = qmax - zp;   // the range of q - z

  // pass 2: the columns in order
  // q - z of this lane's position t, from its sum
  auto step_of = [&](int t) __attribute__((always_inline)) {
    const double x = wl[t] + acc[t];
    const double q0 = fmin(fmax(x * sinv, dlo), dhi);
    const double q1 = fma(fma(-q0, s64, x), sinv, q0);
    return fmin(fmax(rint(q1), dlo), dhi);
  };
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = cl[t];
  Steps<0, g>::run([&](auto nc) __attribute__((always_inline)) {
    constexpr int n = decltype(nc)::value;
    const double e = row_share<n % 16>(fma(-s64, step_of(n / 16), wl[n / 16]));
#pragma unroll
    for (int t = n / 16; t < NT; ++t) acc[t] = fma(mc[n * LD + j + 16 * t], e, acc[t]);
  });
  if (live) {
    uint8_t* q_out = codes + (long long)r * cols + b0 + j;
    double* e_out = comp + (long long)r * cols + b0 + j;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const double dz = step_of(t);
      q_out[16 * t] = (uint8_t)(dz + zp);
      e_out[16 * t] = fma(-s64, dz, wl[t]);
    }
    if (j == 0) {
      scales[(long long)r * G + grp] = s32;
      zeros[(long long)r * G + grp] = (int32_t)zp;
    }
  }
}

template <int G_SIZE>
static hipError_t launch_gptq_group_t(hipStream_t st, int rows, int cols, int bits, int grp,
                                      const float* W, const double* M, double* comp, int has_comp,
                                      uint8_t* codes, float* scales, int32_t* zeros) {
  const size_t lds = ((size_t)G_SIZE * (G_SIZE + 1) + G_SIZE) * sizeof(double);
  static std::atomic<unsigned long long> lds_set{0};
  hipError_t e = allow_dynamic_lds((const void*)gptq_group_kernel<G_SIZE>, lds, lds_set);
  if (e != hipSuccess) return e;
  // One work-group's copy of M_GG fills most of a compute unit's LDS at
  // g = 128: up to 16 rows for each of 256 units the rows are spread over all of
  // them; with more, 32 rows share a copy and two wavefronts a SIMD hide each
  // other's latency.
  const int threads = rows <= 4096 ? 256 : 512;
  hipLaunchKernelGGL(gptq_group_kernel<G_SIZE>, dim3((rows + threads / 16 - 1) / (threads / 16)),
                     dim3(threads), lds, st, rows, cols, bits, grp, W, M, comp, has_comp, codes,
                     scales, zeros);
  return hipGetLastError();
}

// The whole host: factor the reversed Hessian, form M, then the groups in
// order.  Returns the HIP error of the first failed launch; *flag (device) is
// set when H is not positive definite.
hipError_t launch_gptq(hipStream_t st, int rows, int cols, int g, int bits, const float* W,
                       const float* H, char* ws, uint8_t* codes, float* scales, int32_t* zeros,
                       int** flag_out) {
  auto a = [](size_t x) { return (x + 255) & ~size_t(255); };
  const size_t CC = (size_t)cols * cols * 8;
  double* Cf = (double*)ws;
  double* M = (double*)(ws + a(CC));
  double* comp = (double*)(ws + 2 * a(CC));
  double* Linv = (double*)((char*)comp + a((size_t)rows * cols * 8));
  int* flag = (int*)((char*)Linv + a(2 * 64 * 64 * 8));
  *flag_out = flag;
  hipError_t e = launch_zero_bytes(st, flag, sizeof(int));
  if (e != hipSuccess) return e;
  e = launch_copy_lower(st, H, cols, true, Cf);
  if (e != hipSuccess) return e;
  e = launch_potrf_f64(st, Cf, cols, cols, Linv, flag, false);
  if (e != hipSuccess) return e;
  e = launch_antitranspose_lower(st, Cf, cols, M);
  if (e != hipSuccess) return e;
  const long long d = cols;
  for (int p0 = 0; p0 < cols; p0 += kPanel) {
    const int p1 = p0 + kPanel < cols ? p0 + kPanel : cols;
    for (int b0 = p0; b0 < p1; b0 += g) {
      const int grp = b0 / g;
      if (b0 > p0) {
        // comp_G (+)= E(panel so far) M(G, panel so far)^T
        e = launch_gemm_nt_f64(st, rows, g, b0 - p0, 1.0, comp + p0, d, M + b0 * d + p0, d,
                               comp + b0, d, p0 > 0);
        if (e != hipSuccess) return e;
      }
      switch (g) {
        case 32: e = launch_gptq_group_t<32>(st, rows, cols, bits, grp, W, M, comp, b0 > 0, codes, scales, zeros); break;
        case 64: e = launch_gptq_group_t<64>(st, rows, cols, bits, grp, W, M, comp, b0 > 0, codes, scales, zeros); break;
        case 128: e = launch_gptq_group_t<128>(st, rows, cols, bits, grp, W, M, comp, b0 > 0, codes, scales, zeros); break;
        default: return hipErrorInvalidValue;
      }
      if (e != hipSuccess) return e;
    }
    if (p1 < cols) {
      e = launch_gemm_nt_f64(st, rows, cols - p1, p1 - p0, 1.0, comp + p0, d, M + p1 * d + p0, d,
                             comp + p1, d, p0 > 0);
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

}  // namespace jarq
