// Propagation-corrected target (App. E.5, eqs. (mu-target) and (w-corr)).
// Mixing the full-precision response into the target, Y(mu) = (1 - mu) X W +
// mu X~ W, makes the refinement problem the main one with W replaced by
//   W_corr = W + (1 - mu) H^{-1} X~^T (X - X~) W        (columns = output channels),
// H = X~^T X~ + nu^2 I.  With rows as output channels (this library's layout)
// and D = X~^T (X - X~):   W_corr = W + (1 - mu) (W D^T) H^{-1}.
//
// On the GPU, in fp64: T = W D^T (one product), H = L L^T (blocked Cholesky,
// keeping the inverse of every 64 x 64 diagonal block), then T H^{-1} by two
// blocked triangular solves over blocks of kSolve columns:
//   forward   Y L^T = T:  Y_k = T_k L_kk^{-T},  T_j -= Y_k L_jk^T  (j > k),
//   backward  Z L   = Y:  Z_k = Y_k L_kk^{-1},  Y_j -= Z_k L_kj    (j < k),
// and W_corr = W + (1 - mu) Z rounded once to fp32.  The inverses of the
// kSolve-wide diagonal blocks grow from the 64-wide ones, doubling:
// X21 = -X22 (L21 X11).  With 64-wide blocks the solves were chains of
// 3 cols / 64 small products a direction; kSolve = 512 leaves cols / 256 large
// ones for an eighth more arithmetic at 4096 columns.
#include "jarq_internal.h"

namespace jarq {

namespace {
constexpr int QB = 64;
constexpr int kSolve = 512;   // columns per block of the solves
size_t al(size_t x) { return (x + 255) & ~size_t(255); }
}  // namespace

// L, the two [rows][cols] work arrays, the kSolve-wide inverses, the 64-wide
// ones (whose memory then holds the doubling's intermediate products), flag.
size_t qep_workspace_bytes(int rows, int cols) {
  const size_t R = rows, C = cols, nb = (C + QB - 1) / QB, ns = (C + kSolve - 1) / kSolve;
  return al(C * C * 8) + 2 * al(R * C * 8) + al(ns * kSolve * kSolve * 8) +
         al((nb * QB * QB > ns * (kSolve / 2) * (kSolve / 2) ? nb * QB * QB
                                                             : ns * (kSolve / 2) * (kSolve / 2)) * 8) +
         al(4);
}

// The 64-wide inverses onto the diagonals of the kSolve-wide blocks (zero
// elsewhere); one work-group per row of a block.
__global__ __launch_bounds__(256) void spread_inverses_kernel(const double* __restrict__ Linv,
                                                              int cols, double* __restrict__ X) {
  const int row = blockIdx.x;                  // row of the stacked blocks
  const int i = row % kSolve;                  // row within its block
  const int blk = row / QB;                    // 64-wide block of the row
  double* x = X + (long long)row * kSolve;
  for (int j = threadIdx.x; j < kSolve; j += 256) {
    const bool in = j / QB == i / QB && row < cols;
    x[j] = in ? Linv[(long long)blk * QB * QB + (i % QB) * QB + j % QB] : 0.0;
  }
}

__global__ __launch_bounds__(256) void to_f64_kernel(const float* __restrict__ x, long long n,
                                                     double* __restrict__ y) {
  for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < n;
       e += (long long)gridDim.x * 256)
    y[e] = (double)x[e];
}

__global__ __launch_bounds__(256) void qep_finish_kernel(const float* __restrict__ W,
                                                         const double* __restrict__ Z,
                                                         long long n, double c,
                                                         float* __restrict__ out) {
  for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < n;
       e += (long long)gridDim.x * 256)
    out[e] = (float)((double)W[e] + c * Z[e]);
}

static unsigned grid_for(long long n) {
  const long long b = (n + 255) / 256;
  return (unsigned)(b < 16384 ? b : 16384);
}

// The diagonal inverses of width w doubled to 2 w in every kSolve-wide block:
// X21 = -X22 (L21 X11).  P: scratch for the products L21 X11.
static hipError_t double_inverses(hipStream_t st, const double* L, int cols, int w, double* X,
                                  double* P) {
  const long long d = cols;
  const int pairs = cols / (2 * w);   // whole pairs; what remains is handled below
  // pairs of one kSolve-wide block are 2 w apart in both directions, the
  // blocks themselves kSolve rows apart: batched over the pairs of each
  // position within a block
  const int per = kSolve / (2 * w);
  for (int q = 0; q < per; ++q) {
    const int full = pairs > q ? (pairs - q + per - 1) / per : 0;
    const long long o = (long long)q * 2 * w;
    double* Xq = X + o * kSolve + o;
    const double* Lq = L + (o + w) * d + o;
    const long long lz = (long long)kSolve * (d + 1), xz = (long long)kSolve * kSolve;
    double* Pq = P + (long long)q * w * w;
    const long long pz = (long long)per * w * w;
    hipError_t e = launch_gemm_nn_f64(st, w, w, w, 1.0, Lq, d, Xq, kSolve, Pq, w, false, full, lz,
                                      xz, pz);
    if (e == hipSuccess)
      e = launch_gemm_nn_f64(st, w, w, w, -1.0, Xq + (long long)w * kSolve + w, kSolve, Pq, w,
                             Xq + (long long)w * kSolve, kSolve, false, full, xz, pz, xz);
    if (e != hipSuccess) return e;
  }
  // a last pair whose second half is shorter than w
  const int at = pairs * 2 * w, h = cols - at - w;
  if (h > 0) {
    const long long o = at % kSolve;
    double* Xq = X + (long long)(at / kSolve) * kSolve * kSolve + o * kSolve + o;
    hipError_t e = launch_gemm_nn_f64(st, h, w, w, 1.0, L + (long long)(at + w) * d + at, d, Xq,
                                      kSolve, P, w, false);
    if (e == hipSuccess)
      e = launch_gemm_nn_f64(st, h, w, h, -1.0, Xq + (long long)w * kSolve + w, kSolve, P, w,
                             Xq + (long long)w * kSolve, kSolve, false);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_qep_correct(hipStream_t st, int rows, int cols, const float* W, const float* H,
                              const double* D, double mu, float* Wcorr, char* ws,
                              int** flag_out) {
  const size_t R = rows, C = cols, nblk = (C + QB - 1) / QB, ns = (C + kSolve - 1) / kSolve;
  double* L = (double*)ws;
  double* Y = (double*)(ws + al(C * C * 8));
  double* T = (double*)((char*)Y + al(R * C * 8));
  double* X = (double*)((char*)T + al(R * C * 8));
  double* Linv = (double*)((char*)X + al(ns * kSolve * kSolve * 8));
  const size_t half = ns * (kSolve / 2) * (kSolve / 2), small = nblk * QB * QB;
  int* flag = (int*)((char*)Linv + al((small > half ? small : half) * 8));
  *flag_out = flag;
  const long long n = (long long)rows * cols;
  const long long d = cols;
  hipError_t e = launch_zero_bytes(st, flag, sizeof(int));
  if (e != hipSuccess) return e;
  e = launch_copy_lower(st, H, cols, false, L);
  if (e != hipSuccess) return e;
  e = launch_potrf_f64(st, L, cols, d, Linv, flag, true);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(spread_inverses_kernel, dim3((unsigned)(ns * kSolve)), dim3(256), 0, st, Linv,
                     cols, X);
  for (int w = QB; w < kSolve; w *= 2)
    if ((e = double_inverses(st, L, cols, w, X, Linv)) != hipSuccess) return e;
  hipLaunchKernelGGL(to_f64_kernel, dim3(grid_for(n)), dim3(256), 0, st, W, n, Y);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // T[r][a] = sum_b W[r][b] D[a][b]
  e = launch_gemm_nt_f64(st, rows, cols, cols, 1.0, Y, d, D, d, T, d, false);
  if (e != hipSuccess) return e;
  // forward: Y L^T = T
  for (int k0 = 0; k0 < cols; k0 += kSolve) {
    const int nb = min(kSolve, cols - k0), rest = cols - k0 - nb;
    e = launch_gemm_nt_f64(st, rows, nb, nb, 1.0, T + k0, d, X + (long long)k0 * kSolve, kSolve,
                           Y + k0, d, false);
    if (e == hipSuccess && rest > 0)
      e = launch_gemm_nt_f64(st, rows, rest, nb, -1.0, Y + k0, d, L + (k0 + nb) * d + k0, d,
                             T + k0 + nb, d, true);
    if (e != hipSuccess) return e;
  }
  // backward: Z L = Y (Z into T)
  for (int k0 = (int)(ns - 1) * kSolve; k0 >= 0; k0 -= kSolve) {
    const int nb = min(kSolve, cols - k0);
    e = launch_gemm_nn_f64(st, rows, nb, nb, 1.0, Y + k0, d, X + (long long)k0 * kSolve, kSolve,
                           T + k0, d, false);
    if (e == hipSuccess && k0 > 0)
      e = launch_gemm_nn_f64(st, rows, k0, nb, -1.0, T + k0, d, L + k0 * d, d, Y, d, true);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(qep_finish_kernel, dim3(grid_for(n)), dim3(256), 0, st, W, T, n, 1.0 - mu,
                     Wcorr);
  return hipGetLastError();
}

}  // namespace jarq
