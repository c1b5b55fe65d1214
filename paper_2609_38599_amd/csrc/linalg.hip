// Dense fp64 kernels of the per-layer set-up: a blocked Cholesky factorization
// and the matrix products it, the GPTQ-style host and the corrected target are
// built from.  Products run on the fp64 matrix cores
// (v_mfma_f64_16x16x4_f64, 64 cycles each: 70 TFLOP/s sustained); a vector
// version of the same tiles reached about a third of that, bound by its LDS
// reads (eight operands for sixteen FMAs, where a matrix instruction takes two
// per lane for its 1024).
#include "chol64.h"

namespace jarq {

namespace {
constexpr int LT = 64;   // Cholesky block size
constexpr int KB = 16;   // k-step of the products
// two doubles from an address that is only 8-byte aligned
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x2_u __attribute__((ext_vector_type(2), aligned(8)));
}  // namespace

// C[i][j] (+)= alpha sum_k A[i][k] B(j, k) for i < M, j < N, with B(j, k) =
// B[j][k], or B[k][j] when BK.  K is a multiple of 16.  blockIdx.z picks one of
// a batch of products (strides az, bz, cz).  C must not overlap A or B.  lower:
// tiles wholly above the diagonal are left out.
//
// TM x TN output tile per 256-thread work-group, 2 x 2 wavefronts, k in steps
// of 16 through two LDS stages; the next step's values are loaded into
// registers during the current one's products.  Row-major operand tiles have
// rows of 18 doubles and k-major ones rows of TN + 16: a fragment read (16 rows
// or columns at four k) covers the 64 banks once per half wave.
template <int TM, int TN, bool BK>
__global__ __launch_bounds__(256, 2) void gemm_f64_kernel(int M, int N, int K, double alpha,
                                                          const double* __restrict__ A,
                                                          long long lda, long long az,
                                                          const double* __restrict__ B,
                                                          long long ldb, long long bz, double* C,
                                                          long long ldc, long long cz,
                                                          int accumulate, int lower) {
  constexpr int LDR = KB + 2;                  // row stride of a row-major tile
  constexpr int LDK = TN + 16;                 // row stride of a k-major tile
  constexpr int ASZ = TM * LDR, BSZ = BK ? KB * LDK : TN * LDR;
  constexpr int MB = TM / 32, NB = TN / 32;    // 16 x 16 blocks per wavefront
  constexpr int APT = TM * KB / 512, BPT = TN * KB / 512;  // 16-byte loads per thread
  __shared__ __attribute__((aligned(16))) double as[2][ASZ];
  __shared__ __attribute__((aligned(16))) double bs[2][BSZ];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int lc = lane & 15, lk = lane >> 4;
  const int i0 = blockIdx.y * TM, j0 = blockIdx.x * TN;
  if (lower && j0 >= i0 + TM) return;   // wholly above the diagonal
  A += (long long)blockIdx.z * az;
  B += (long long)blockIdx.z * bz;
  C += (long long)blockIdx.z * cz;
  // rows and columns past the edge repeat the last one; their results are not
  // stored
  const double* ap[APT];
  const double* bp[BPT];
#pragma unroll
  for (int u = 0; u < APT; ++u) {
    const int e = tid + 256 * u;
    ap[u] = A + (long long)min(i0 + (e >> 3), M - 1) * lda + 2 * (e & 7);
  }
#pragma unroll
  for (int u = 0; u < BPT; ++u) {
    const int e = tid + 256 * u;
    if (BK)
      bp[u] = B + (long long)(e / (TN / 2)) * ldb + min(j0 + 2 * (e % (TN / 2)), N - 2);
    else
      bp[u] = B + (long long)min(j0 + (e >> 3), N - 1) * ldb + 2 * (e & 7);
  }
  f64x2 ra[APT], rb[BPT];
  auto load = [&](int k0) {
#pragma unroll
    for (int u = 0; u < APT; ++u) ra[u] = *(const f64x2_u*)(ap[u] + k0);
#pragma unroll
    for (int u = 0; u < BPT; ++u)
      rb[u] = *(const f64x2_u*)(bp[u] + (BK ? (long long)k0 * ldb : (long long)k0));
  };
  auto stage = [&](int s) {
#pragma unroll
    for (int u = 0; u < APT; ++u) {
      const int e = tid + 256 * u;
      *(f64x2*)&as[s][(e >> 3) * LDR + 2 * (e & 7)] = ra[u];
    }
#pragma unroll
    for (int u = 0; u < BPT; ++u) {
      const int e = tid + 256 * u;
      if (BK)
        *(f64x2*)&bs[s][(e / (TN / 2)) * LDK + 2 * (e % (TN / 2))] = rb[u];
      else
        *(f64x2*)&bs[s][(e >> 3) * LDR + 2 * (e & 7)] = rb[u];
    }
  };
  f64x4 acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  load(0);
  stage(0);
  __syncthreads();
  const int nk = K / KB;
  for (int t = 0; t < nk; ++t) {
    const int s = t & 1;
    if (t + 1 < nk) load((t + 1) * KB);
#pragma unroll
    for (int ks = 0; ks < KB / 4; ++ks) {
      double fa[MB], fb[NB];
#pragma unroll
      for (int a = 0; a < MB; ++a)
        fa[a] = as[s][(wm * (TM / 2) + 16 * a + lc) * LDR + 4 * ks + lk];
#pragma unroll
      for (int b = 0; b < NB; ++b)
        fb[b] = BK ? bs[s][(4 * ks + lk) * LDK + wn * (TN / 2) + 16 * b + lc]
                   : bs[s][(wn * (TN / 2) + 16 * b + lc) * LDR + 4 * ks + lk];
#pragma unroll
      for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = mfma_f64(fa[a], fb[b], acc[a][b]);
    }
    // the other stage was last read before the barrier that ended step t - 1
    if (t + 1 < nk) stage(s ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int j = j0 + wn * (TN / 2) + 16 * b + lc;
      const int ib = i0 + wm * (TM / 2) + 16 * a + lk;
      double* c = C + (long long)ib * ldc + j;
      double old[4];
      if (accumulate) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          old[v] = (ib + 4 * v < M && j < N) ? c[(long long)(4 * v) * ldc] : 0.0;
      }
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (ib + 4 * v < M && j < N)
          c[(long long)(4 * v) * ldc] =
              accumulate ? fma(alpha, acc[a][b][v], old[v]) : alpha * acc[a][b][v];
    }
}

template <bool BK>
static hipError_t launch_gemm_t(hipStream_t st, int M, int N, int K, double alpha, const double* A,
                                long long lda, const double* B, long long ldb, double* C,
                                long long ldc, bool accumulate, int batch, long long az,
                                long long bz, long long cz, bool lower = false) {
  if (M <= 0 || N <= 0 || batch <= 0) return hipSuccess;
  if (K <= 0 || K % KB != 0 || N % 2 != 0) return hipErrorInvalidValue;
  // 128 x 128 tiles read half of what 64 x 64 ones do for a product and run at
  // 64 TFLOP/s (4096^3; 64 x 64: 48); with fewer of them than about one and a
  // half per compute unit the smaller tiles spread the work better (4096 x 512 x
  // 512: 45 us in 64 x 64 tiles, where 128 x 128 ones would use half the units).
  const long long big = (long long)((M + 127) / 128) * ((N + 127) / 128) * batch / (lower ? 2 : 1);
  if (big >= 384) {
    hipLaunchKernelGGL((gemm_f64_kernel<128, 128, BK>), dim3((N + 127) / 128, (M + 127) / 128, batch),
                       dim3(256), 0, st, M, N, K, alpha, A, lda, az, B, ldb, bz, C, ldc, cz,
                       (int)accumulate, (int)lower);
  } else {
    const long long mid = (long long)((M + 63) / 64) * ((N + 63) / 64) * batch / (lower ? 2 : 1);
    if (mid >= 384 || M < 64)
      hipLaunchKernelGGL((gemm_f64_kernel<64, 64, BK>), dim3((N + 63) / 64, (M + 63) / 64, batch),
                         dim3(256), 0, st, M, N, K, alpha, A, lda, az, B, ldb, bz, C, ldc, cz,
                         (int)accumulate, (int)lower);
    else
      hipLaunchKernelGGL((gemm_f64_kernel<32, 64, BK>), dim3((N + 63) / 64, (M + 31) / 32, batch),
                         dim3(256), 0, st, M, N, K, alpha, A, lda, az, B, ldb, bz, C, ldc, cz,
                         (int)accumulate, (int)lower);
  }
  return hipGetLastError();
}

hipError_t launch_gemm_nt_f64(hipStream_t st, int M, int N, int K, double alpha, const double* A,
                              long long lda, const double* B, long long ldb, double* C,
                              long long ldc, bool accumulate, int batch, long long az,
                              long long bz, long long cz) {
  return launch_gemm_t<false>(st, M, N, K, alpha, A, lda, B, ldb, C, ldc, accumulate, batch, az,
                              bz, cz);
}

hipError_t launch_gemm_nn_f64(hipStream_t st, int M, int N, int K, double alpha, const double* A,
                              long long lda, const double* B, long long ldb, double* C,
                              long long ldc, bool accumulate, int batch, long long az,
                              long long bz, long long cz) {
  return launch_gemm_t<true>(st, M, N, K, alpha, A, lda, B, ldb, C, ldc, accumulate, batch, az,
                             bz, cz);
}

// ---- Cholesky factorization, right-looking in blocks of 64 columns ----
//
// Per block two launches: the panel below the factored diagonal block is
// multiplied by the block's inverse transpose, then the columns up to the end
// of the block's 512-wide outer panel are updated.  The update's first
// work-group takes the next diagonal block alone and goes on to factor and
// invert it (chol64.h) while the others work on their tiles, so the update
// hides behind that serial part.  At the end of an outer panel one product
// with 512 columns updates the rest of the lower triangle: with every update
// carried through the whole triangle, 64 columns at a time, the first half of
// the steps were bound by reading and writing it (52 us for the first, 5 TB/s).
// 4096 channels: 64 diagonal steps of 16 to 25 us (mean 20) and 63 panels of 6 us;
// 84 us for the diagonal block alone before.  The serial part bounds it: of a
// step's 20 us, 11 factor the block and 3 invert it.

// 64 x 64 part of a row-major matrix into an LDS block (rows past `rows` repeat
// the last one; `cols` is 32 or 64).
__device__ __forceinline__ void load_block(double* dst, const double* src, long long ld, int rows,
                                           int cols) {
  const int i = threadIdx.x >> 5, j = 2 * (threadIdx.x & 31);
  if (j >= cols) return;
  f64x2 v[8];   // every load before the first store
#pragma unroll
  for (int u = 0; u < 8; ++u) v[u] = *(const f64x2_u*)(src + (long long)min(i + 8 * u, rows - 1) * ld + j);
#pragma unroll
  for (int u = 0; u < 8; ++u) *(f64x2*)&dst[(i + 8 * u) * kCholLd + j] = v[u];
}

// panel[i][c] = sum_{k <= c} panel[i][k] Linv[c][k] in place: 32 rows per
// work-group, all read before any is written; wave = 16 columns.
__global__ __launch_bounds__(256) void potrf_panel_kernel(double* __restrict__ panel, long long ld,
                                                          int rows,
                                                          const double* __restrict__ Linv) {
  __shared__ __attribute__((aligned(16))) double x_s[kCholBlock];
  __shared__ __attribute__((aligned(16))) double p_s[32 * kCholLd];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lc = lane & 15, lk = lane >> 4;
  const int i0 = blockIdx.x * 32;
  double* P = panel + (long long)i0 * ld;
  const int live = min(32, rows - i0);
  for (int e = tid; e < 32 * 32; e += 256) {
    const int i = e >> 5, j = 2 * (e & 31);
    *(f64x2*)&p_s[i * kCholLd + j] = *(const f64x2_u*)(P + (long long)min(i, live - 1) * ld + j);
  }
  load_block(x_s, Linv, LT, LT, LT);
  __syncthreads();
  f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
  for (int ks = 0; ks < 4 * (wave + 1); ++ks) {
    const double b = frag_a(x_s, 16 * wave, 0, ks);
#pragma unroll
    for (int a = 0; a < 2; ++a) acc[a] = mfma_f64(frag_a(p_s, 16 * a, 0, ks), b, acc[a]);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * a + 4 * v + lk;
      if (i < live) P[(long long)i * ld + 16 * wave + lc] = acc[a][v];
    }
}

// Update of the columns right of a panel: A22 -= P P^T on 64 x 64 tiles (P = the
// panel's 64 columns, A22 the n x n trailing matrix; tile column blockIdx.y,
// tile row blockIdx.x, those above the diagonal skipped), and the next
// diagonal block's factor (in place) and inverse (Linv, 64 x 64, zero above the
// diagonal) by work-group (0, 0).  P null: no update (a first diagonal block).
__global__ __launch_bounds__(256, 2) void potrf_trail_kernel(double* __restrict__ A22,
                                                             const double* __restrict__ P,
                                                             long long ld, int n,
                                                             double* __restrict__ Linv,
                                                             int* __restrict__ flag) {
  __shared__ __attribute__((aligned(16))) double p_s[kCholBlock];
  __shared__ __attribute__((aligned(16))) double q_s[kCholBlock];
  __shared__ double dinv[64];
  __shared__ __attribute__((aligned(16))) double col_s[128];
  __shared__ int fail;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lc = lane & 15, lk = lane >> 4;
  const int bi = blockIdx.x, bj = blockIdx.y;
  if (bi < bj) return;
  if (bi == 0) {
    const int nb = min(LT, n);
    if (tid == 0) fail = 0;
    load_block(q_s, A22, ld, nb, nb);
    if (P != nullptr) load_block(p_s, P, ld, nb, LT);
    __syncthreads();
    if (P != nullptr) {
      int id = 0;
      for (int ti = 0; ti < nb / 16; ++ti)
        for (int tj = 0; tj <= ti; ++tj, ++id) {
          if ((id & 3) != wave) continue;
          f64x4 c = load_c(q_s, 16 * ti, 16 * tj);
#pragma unroll
          for (int ks = 0; ks < 16; ++ks)
            c = mfma_f64(-frag_a(p_s, 16 * ti, 0, ks), frag_a(p_s, 16 * tj, 0, ks), c);
          store_c(q_s, 16 * ti, 16 * tj, c);
        }
      __syncthreads();
    }
    chol64_factor(q_s, nb, dinv, col_s, &fail);
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int i = (tid >> 6) + 4 * u, j = tid & 63;
      if (i < nb && j <= i) A22[(long long)i * ld + j] = q_s[i * kCholLd + j];
    }
    chol64_invert(q_s, nb, dinv, p_s);
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int i = (tid >> 6) + 4 * u, j = tid & 63;
      Linv[i * LT + j] = (i < nb && j <= i) ? p_s[i * kCholLd + j] : 0.0;
    }
    if (tid == 0 && fail) *flag = 1;
    return;
  }
  const int i0 = bi * LT, j0 = bj * LT;
  const int wm = wave >> 1, wn = wave & 1;
  double* Ct = A22 + (long long)i0 * ld + j0;
  const int mi = min(LT, n - i0), mj = min(LT, n - j0);
  f64x4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = min(32 * wm + 16 * a + 4 * v + lk, mi - 1);
        const int j = min(32 * wn + 16 * b + lc, mj - 1);
        acc[a][b][v] = Ct[(long long)i * ld + j];
      }
  load_block(p_s, P + (long long)i0 * ld, ld, mi, LT);
  load_block(q_s, P + (long long)j0 * ld, ld, mj, LT);
  __syncthreads();
#pragma unroll
  for (int ks = 0; ks < 16; ++ks) {
    double fa[2], fb[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) fa[a] = -frag_a(p_s, 32 * wm + 16 * a, 0, ks);
#pragma unroll
    for (int b = 0; b < 2; ++b) fb[b] = frag_a(q_s, 32 * wn + 16 * b, 0, ks);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[a][b] = mfma_f64(fa[a], fb[b], acc[a][b]);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 32 * wm + 16 * a + 4 * v + lk;
        const int j = 32 * wn + 16 * b + lc;
        if (i < mi && j < mj && j0 + j <= i0 + i) Ct[(long long)i * ld + j] = acc[a][b][v];
      }
}

// In-place lower Cholesky factor of A [d][d] (d a multiple of 32, leading
// dimension lda; what lies above the diagonal is scratch).  Linv: scratch of two
// 64 x 64 blocks, or, with keep_inverses, one 64 x 64 block per diagonal block
// (block b at Linv + 4096 b holds the inverse of the factor's diagonal block
// b).  *flag is set when a pivot is not positive (the caller clears it first).
hipError_t launch_potrf_f64(hipStream_t st, double* A, int d, long long lda, double* Linv_base,
                            int* flag, bool keep_inverses) {
  if (d % 32 != 0) return hipErrorInvalidValue;
  auto linv = [&](int k) { return Linv_base + (long long)(keep_inverses ? k : k & 1) * LT * LT; };
  constexpr int kOuter = 512;   // columns per outer panel
  hipError_t e = hipSuccess;
  for (int o0 = 0; o0 < d && e == hipSuccess; o0 += kOuter) {
    const int o1 = min(o0 + kOuter, d);
    hipLaunchKernelGGL(potrf_trail_kernel, dim3(1), dim3(256), 0, st, A + (long long)o0 * (lda + 1),
                       (const double*)nullptr, lda, d - o0, linv(o0 / LT), flag);
    for (int k0 = o0; k0 < o1 && k0 + LT < d; k0 += LT) {
      const int n0 = k0 + LT, rest = d - n0, k = k0 / LT;
      double* panel = A + (long long)n0 * lda + k0;
      hipLaunchKernelGGL(potrf_panel_kernel, dim3((rest + 31) / 32), dim3(256), 0, st, panel, lda,
                         rest, linv(k));
      if (n0 < o1)
        hipLaunchKernelGGL(potrf_trail_kernel, dim3((rest + LT - 1) / LT, (o1 - n0 + LT - 1) / LT),
                           dim3(256), 0, st, A + (long long)n0 * (lda + 1), panel, lda, rest,
                           linv(k + 1), flag);
    }
    e = hipGetLastError();
    const int rest = d - o1;
    if (rest > 0 && e == hipSuccess) {
      const double* p = A + (long long)o1 * lda + o0;
      e = launch_gemm_t<false>(st, rest, rest, o1 - o0, -1.0, p, lda, p, lda,
                               A + (long long)o1 * (lda + 1), lda, true, 1, 0, 0, 0, true);
    }
  }
  return e;
}

// Lower part of H in fp64: C[i][j] = H[i][j], or with reverse the Hessian
// with its channel order reversed, C[i][j] = H[d-1-i][d-1-j].  One work-group
// per row.
__global__ __launch_bounds__(256) void copy_lower_kernel(const float* __restrict__ H, int d,
                                                         int reverse, double* __restrict__ C) {
  const int i = blockIdx.x;
  const float* h = H + (long long)(reverse ? d - 1 - i : i) * d;
  double* c = C + (long long)i * d;
  for (int j = threadIdx.x; j <= i; j += 256) c[j] = (double)h[reverse ? d - 1 - j : j];
}

// M[k][t] = C[d-1-t][d-1-k] for t <= k (reflection about the anti-diagonal,
// which maps a lower triangle onto a lower triangle), 32 x 32 tiles through LDS.
__global__ __launch_bounds__(256) void antitranspose_lower_kernel(const double* __restrict__ C,
                                                                  int d, double* __restrict__ M) {
  __shared__ double tile[32][33];
  const int k0 = blockIdx.y * 32, t0 = blockIdx.x * 32;
  if (t0 > k0 + 31) return;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // ty < 8
  // The source block holds rows d-1-t and columns d-1-k: read row r = d-1-(t0+31-a)
  // for a = 0..31 with consecutive columns.
  for (int a = ty; a < 32; a += 8) {
    const int t = t0 + 31 - a, k = k0 + 31 - tx;
    if (t < d && k < d && t <= k) tile[a][tx] = C[(long long)(d - 1 - t) * d + (d - 1 - k)];
  }
  __syncthreads();
  for (int a = ty; a < 32; a += 8) {
    const int k = k0 + a, t = t0 + tx;
    if (k < d && t < d && t <= k) M[(long long)k * d + t] = tile[31 - tx][31 - a];
  }
}

hipError_t launch_copy_lower(hipStream_t st, const float* H, int d, bool reverse, double* C) {
  hipLaunchKernelGGL(copy_lower_kernel, dim3(d), dim3(256), 0, st, H, d, (int)reverse, C);
  return hipGetLastError();
}

hipError_t launch_antitranspose_lower(hipStream_t st, const double* C, int d, double* M) {
  const int nt = (d + 31) / 32;
  hipLaunchKernelGGL(antitranspose_lower_kernel, dim3(nt, nt), dim3(256), 0, st, C, d, M);
  return hipGetLastError();
}

}  // namespace jarq
