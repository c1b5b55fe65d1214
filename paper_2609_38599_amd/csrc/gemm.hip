// The product E H of the stand-alone row objectives.
//
// row_products_kernel (three bf16 planes, bf16x3.h): the row objectives
// e_j^T H e_j of the stand-alone jarq_objective (paper Sec. 3.3.2 and eq. (7)),
// from E H of every row; the sweep's own residual product runs on fp16 matrix
// cores (sgemm.hip).  E = W - What with What = s_i (q - z_i) is formed on the fly
// from the codes, scales and zero points (eq. (1)); the epilogue writes, per
// row and 64-column slice, sum_c E(row, c) (E H)(row, c) in fp64.
//
// Tiling: 512 threads; 128 x 128 tile, 2 x 4 wavefronts of 64 x 32, k in steps
// of 32; where that gives fewer tiles than compute units, 64 x 64 tiles, 2 x 2
// wavefronts of 32 x 32 twice, k in steps of 64, the second four taking the odd
// k-slices.  H is symmetric, so B(k, n) = H(k, n) is read along row n.  Both
// operands go through registers (split there) into LDS, rows padded by 16
// bytes: two stages for the large tile, one for the small (two work-groups a CU
// cover each other's loads).  1000 x 2752:
// 172 us (the fp32 instruction: 517), and a quarter of its error.
#include "bf16x3.h"

namespace jarq {

namespace {

// E(row, k): the weight minus its quantized value
struct ErrorOf {
  const float* W;
  const uint8_t* codes;
  const float* scales;
  const int32_t* zeros;
  int cols, gs, G;   // gs = log2 of the group size
  __device__ __forceinline__ float at(int row, int col) const {
    const float w = W[(size_t)row * cols + col];
    const float s = scales[(size_t)row * G + (col >> gs)];
    const int z = zeros[(size_t)row * G + (col >> gs)];
    return w - s * (float)((int)codes[(size_t)row * cols + col] - z);
  }
};

// The 32 x 32 block of E H at (r0, c0) with the fp32 instruction straight from
// memory (one wave): for blocks the three planes cannot do.
__device__ __forceinline__ f32x16 slow_block(const ErrorOf& E, const float* __restrict__ H,
                                             int rows, int r0, int c0) {
  const int lane = threadIdx.x & 63, lm = lane & 31, kh = lane >> 5;
  const int row = min(r0 + lm, rows - 1), col = min(c0 + lm, E.cols - 1);
  f32x16 acc = f32x16{};
  for (int k = 0; k < E.cols; k += 2)   // cols is even
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(E.at(row, k + kh), H[(size_t)col * E.cols + k + kh],
                                               acc, 0, 0, 0);
  return acc;
}

}  // namespace

template <bool BIG>
__global__ __launch_bounds__(512, BIG ? 2 : 4) void row_products_kernel(int rows, ErrorOf E,
                                                              const float* __restrict__ H,
                                                              double* __restrict__ objpart) {
  constexpr int TE = BIG ? 128 : 64;
  constexpr int CH = BIG ? 32 : 64;           // k per step
  constexpr int LD = 2 * CH + 16;             // row stride in bytes
  constexpr int PLANE = 2 * TE * LD;          // E rows, then H rows
  constexpr int STAGE = 3 * PLANE;
  constexpr int AB = BIG ? 2 : 1;             // 32-row blocks per wavefront
  constexpr int PR = CH / 8;                  // pieces of 8 values per row
  constexpr int WN = BIG ? 4 : 2;             // wavefronts along the columns
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int cols = E.cols;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = BIG ? wave >> 2 : (wave >> 1) & 1, wn = BIG ? wave & 3 : wave & 1;
  const int wk = BIG ? 0 : wave >> 2;
  const int lm = lane & 31, kh = lane >> 5;
  const int m0 = blockIdx.y * TE, n0 = blockIdx.x * TE;
  // staging: piece tid of the E rows and piece tid of the H rows (both have
  // TE PR = 512 pieces); rows past the edge repeat the last one (their results
  // are not stored); k past cols stages 0
  static_assert(TE * PR == 512, "one piece of each operand per thread");
  const int pr = tid / PR, pk = 8 * (tid % PR);
  const int er = min(m0 + pr, rows - 1), hr = min(n0 + pr, cols - 1);
  const float* w_row = E.W + (size_t)er * cols;
  const uint8_t* q_row = E.codes + (size_t)er * cols;
  const float* h_row = H + (size_t)hr * cols;
  f32x4 we[2], wh[2];
  uint2 qe;
  float se;
  int ze;
  auto load = [&](int k0) {
    const int k = min(k0 + pk, cols - 8);
    we[0] = *(const f32x4*)(w_row + k);
    we[1] = *(const f32x4*)(w_row + k + 4);
    qe = *(const uint2*)(q_row + k);
    se = E.scales[(size_t)er * E.G + (k >> E.gs)];
    ze = E.zeros[(size_t)er * E.G + (k >> E.gs)];
    wh[0] = *(const f32x4*)(h_row + k);
    wh[1] = *(const f32x4*)(h_row + k + 4);
  };
  auto store = [&](int k0, char* stage) {
    const bool in = k0 + pk < cols;
    float e[8], h[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t q = ((i < 4 ? qe.x : qe.y) >> (8 * (i & 3))) & 0xffu;
      e[i] = in ? we[i >> 2][i & 3] - se * (float)((int)q - ze) : 0.f;
      h[i] = in ? wh[i >> 2][i & 3] : 0.f;
    }
    u32x4 p[2][3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t a, b, c;
      split_pair(e[2 * i], e[2 * i + 1], a, b, c);
      p[0][0][i] = a, p[0][1][i] = b, p[0][2][i] = c;
      split_pair(h[2 * i], h[2 * i + 1], a, b, c);
      p[1][0][i] = a, p[1][1][i] = b, p[1][2][i] = c;
    }
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int pl = 0; pl < 3; ++pl)
        *(u32x4*)(stage + pl * PLANE + (o * TE + pr) * LD + 2 * pk) = p[o][pl];
  };
  f32x16 acc[AB], low[AB];
#pragma unroll
  for (int a = 0; a < AB; ++a) acc[a] = low[a] = f32x16{};
  const int nk = (cols + CH - 1) / CH;
  load(0);
  store(0, smem);
  __syncthreads();
  for (int q = 0; q < nk; ++q) {
    const char* cur = smem + (BIG ? (q & 1) * STAGE : 0);
    if (q + 1 < nk) load((q + 1) * CH);   // in flight during this step
    const char* ra = cur + (wm * 32 * AB + lm) * LD + 16 * kh;
    const char* rb = cur + (TE + wn * 32 + lm) * LD + 16 * kh;
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      const int ks = BIG ? k2 : 2 * k2 + wk;
      bf16x8 fb[3], fa[AB][3];
#pragma unroll
      for (int p = 0; p < 3; ++p) fb[p] = *(const bf16x8*)(rb + p * PLANE + 32 * ks);
#pragma unroll
      for (int a = 0; a < AB; ++a)
#pragma unroll
        for (int p = 0; p < 3; ++p)
          fa[a][p] = *(const bf16x8*)(ra + p * PLANE + 32 * a * LD + 32 * ks);
      mfma_bf16x3<AB>(fa, fb, acc, low);
    }
    // the other stage was last read before the barrier that ended step q - 1;
    // a single stage is free once every wave is here
    if (!BIG) __syncthreads();
    if (q + 1 < nk) store((q + 1) * CH, smem + (BIG ? ((q + 1) & 1) * STAGE : 0));
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < AB; ++a) acc[a] += low[a];
  double* part_s = (double*)smem;             // [TE][WN]
  float* red = (float*)(part_s + TE * WN);    // small tile: sums of the odd k-slices
  if (!BIG) {
    if (wk == 1) {
#pragma unroll
      for (int v = 0; v < 16; ++v) red[(wave & 3) * 1024 + 64 * v + lane] = acc[0][v];
    }
    __syncthreads();
    if (wk == 0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[0][v] += red[wave * 1024 + 64 * v + lane];
    }
  }
  if (wk == 0) {
#pragma unroll
    for (int a = 0; a < AB; ++a) {
      const int rb0 = m0 + 32 * (AB * wm + a), col = n0 + 32 * wn + lm;
      bool fine = true;
#pragma unroll
      for (int v = 0; v < 16; ++v) fine &= isfinite(acc[a][v]);
      if (!__all(fine)) acc[a] = slow_block(E, H, rows, rb0, n0 + 32 * wn);
      // element v of lane l: row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = rb0 + 8 * (v / 4) + 4 * kh + (v % 4);
        double x = 0.0;
        if (row < rows && col < cols) x = (double)E.at(row, col) * (double)acc[a][v];
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) x += __shfl_xor(x, off);
        if (lm == 0) part_s[(row - m0) * WN + wn] = x;
      }
    }
  }
  __syncthreads();
  // 64-column slices: two wavefronts' columns each
  const int nt = (cols + kObjTile - 1) / kObjTile;
  for (int t = tid; t < TE * WN / 2; t += 512) {
    const int r = t / (WN / 2), sl = t % (WN / 2);
    const int slice = n0 / kObjTile + sl;
    if (m0 + r < rows && slice < nt)
      objpart[(size_t)(m0 + r) * nt + slice] = part_s[r * WN + 2 * sl] + part_s[r * WN + 2 * sl + 1];
  }
}

template <bool BIG>
static hipError_t launch_row_products_t(hipStream_t st, int rows, const ErrorOf& E, const float* H,
                                        double* objpart) {
  constexpr int TE = BIG ? 128 : 64;
  constexpr size_t lds = 3 * (BIG ? 2 * 256 * 80 : 128 * 144);
  static_assert(lds >= 64 * 2 * sizeof(double) + 4 * 1024 * sizeof(float), "LDS");
  static std::atomic<unsigned long long> lds_set{0};
  const hipError_t e = allow_dynamic_lds((const void*)row_products_kernel<BIG>, lds, lds_set);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(row_products_kernel<BIG>, dim3((E.cols + TE - 1) / TE, (rows + TE - 1) / TE),
                     dim3(512), lds, st, rows, E, H, objpart);
  return hipGetLastError();
}

hipError_t launch_row_products(hipStream_t st, int rows, int cols, int g, const float* W,
                               const uint8_t* codes, const float* scales, const int32_t* zeros,
                               const float* H, double* objpart) {
  const ErrorOf E{W, codes, scales, zeros, cols, g == 32 ? 5 : g == 64 ? 6 : 7, cols / g};
  // large tiles from one per compute unit on (large and small: 500 x 4096, 128 large
  // tiles, 224 and 167 us; 1000 x 4096, 256 of them, 233 and 289; 1500 x 4096, 384,
  // 431 and 420; 2000 x 4096, 512, 458 and 553).  Somewhat below that the large ones
  // are already the faster (1000 x 2752, 176 of them, 164 and 175), but the small
  // ones sum in two halves of k, nearer to the 64-bit value.
  const long long big = (long long)((cols + 127) / 128) * ((rows + 127) / 128);
  if (big >= 256) return launch_row_products_t<true>(st, rows, E, H, objpart);
  return launch_row_products_t<false>(st, rows, E, H, objpart);
}

}  // namespace jarq
