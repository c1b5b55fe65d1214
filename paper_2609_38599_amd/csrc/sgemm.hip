// Split-precision products on fp16 matrix cores for the residual product of
// the sweep (paper Sec. 3.3.2: the conditional residual of eq. (7) needs
// (H e)_i for every row and group, used in the coordinates of eq. (10)).
// split3_kernel (three products of two-term planes of both operands) forms
// the layer's fixed T = W M^T once per layer; resid_kernel (further below)
// forms every sweep's U = T - What M^T with the exact q - z as one operand;
// wh_kernel (at the end) forms W H of the scale update from three-term planes.
//
// Operands arrive as two-term fp16 planes with power-of-two scales (split.hip):
// A = (Ah + Al) ra_m per row m, B(k, n) = Bt(n, k) with Bt = (Bh + Bl) rb_n per
// row n.  The product keeps the three terms above 2^-22 relative,
// A B = (Ah Bh + Ah Bl + Al Bh) ra_m rb_n, accumulated in fp32 by
// v_mfma_f32_32x32x16_f16 — fp32-class accuracy at 3/16 of the fp32 matrix
// work.  With Bt = M = blockdiag(L_i^{-1}) H the product E M^T has in group
// i's columns of row j L_i^{-1} (H e_j)_i, the u of eq. (10) before division
// by the scale.
//
// The objective that follows the residual product is in objective.hip.
//
// Tiling: 256 x BN output tile per 512-thread work-group, 2 x 4 waves of
// 128 x BN/4 (two waves per SIMD, so one wave's waits are covered by the
// other's matrix work), K in steps of 32.  Both planes of both operands go
// straight from global memory to LDS (global_load_lds_dwordx4, no register
// staging) into one of two stages (128 KB for BN = 256); the eight loads of
// the next stage are spread over the first four fragment blocks of the
// current one.  Fragment reads are software-pipelined one block ahead (see
// compute).  One work-group per CU.  Tiles are ordered so that
// each XCD (work-groups are dealt to the 8 XCDs round-robin) works on a
// compact block of tiles that share A row-tiles and B column-tiles in its L2.
#include <hip/hip_ext.h>

#include "bf16x3.h"

namespace jarq {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

namespace {
constexpr int BM = 256, BK = 32;

// Tile of work-group wid; false when wid has none (the grid may be sized for
// more rows than the sweep has).
__device__ __forceinline__ bool tile_of(int wid, int nbm, int nbn, int& tm, int& tn) {
  const int total = nbm * nbn;
  const int q = total / 8, r = total % 8;
  const int x = wid % 8, loc = wid / 8;
  if (loc >= q + (x < r ? 1 : 0)) return false;  // this XCD's share is taken
  const int id = (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + loc;
  constexpr int GM = 4;  // tile-rows per band
  const int band = id / (GM * nbn);
  const int first = band * GM;
  const int gsz = min(nbm - first, GM);
  const int within = id - band * GM * nbn;
  tm = first + within % gsz;
  tn = within / gsz;
  return true;
}

// LDS holds each plane tile as rows of 32 halves (four 16-byte chunks); chunk
// c of row r sits at position c ^ swz(r).  A fragment read (lane = row, two
// chunks across the wave halves) serves 16 consecutive rows per clock, and
// the 64-byte rows share 256-byte bank lines four at a time: rows r, r + 4,
// r + 8 and r + 12 take distinct positions.
__device__ __forceinline__ int swz(int r) { return (r >> 2) & 3; }

// One 16-byte direct global -> LDS load per lane (lane L writes lds + 16 L bytes).
// A plain device function: the builtin and the LDS address space exist on the
// device side only.
__device__ __forceinline__ void dma16(const _Float16* src, _Float16* lds) {
  __builtin_amdgcn_global_load_lds((const void*)src,
                                   (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}
}  // namespace

template <int BN>
__global__ __launch_bounds__(512, 1) void split3_kernel(
    int M, int N, int K, int lda, int ldb, int ldc, const _Float16* __restrict__ Ah,
    const _Float16* __restrict__ Al, const float* __restrict__ arow_inv,
    const _Float16* __restrict__ Bh, const _Float16* __restrict__ Bl,
    const float* __restrict__ bcol_inv, float* __restrict__ C, const int* __restrict__ m_dev) {
  if (m_dev != nullptr) M = *m_dev;
  constexpr int WN = BN / 4;   // wave tile columns
  constexpr int NB = WN / 32;  // 32-column blocks per wave
  constexpr int A_PLANE = BM * BK, B_PLANE = BN * BK;  // halves
  constexpr int STAGE = 2 * A_PLANE + 2 * B_PLANE;
  // Two stages in two distinct arrays, so that the compiler can tell which
  // one an outstanding direct-to-LDS load writes.
  __shared__ __attribute__((aligned(1024))) _Float16 buf0[STAGE];
  __shared__ __attribute__((aligned(1024))) _Float16 buf1[STAGE];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave >> 2, wn = wave & 3;
  const int lm = lane & 31, kh = lane >> 5;
  const int nbm = (M + BM - 1) / BM, nbn = (N + BN - 1) / BN;
  int tm, tn;
  if (M <= 0 || !tile_of(blockIdx.x, nbm, nbn, tm, tn)) return;  // uniform across the work-group
  const int m0 = tm * BM, n0 = tn * BN;

  // Direct global -> LDS loads, 16 bytes per lane: one instruction fills 1 KB
  // of LDS (16 rows of a plane tile).  Wave w fills the 1 KB pieces w, w + 4,
  // ...; lane L of a piece holds row 16 j + L / 4 at chunk position L % 4, i.e.
  // chunk (L % 4) ^ swz(row).  Rows past the edge read row 0 instead: their
  // products only reach output rows and columns that are never stored.
  // Element offsets are 32-bit (operands stay below 2^31 elements).
  constexpr int APW = A_PLANE / 512 / 8;  // 1 KB pieces per wave per A plane
  constexpr int BPW = B_PLANE / 512 / 8;
  unsigned aoff[APW], boff[BPW];
#pragma unroll
  for (int i = 0; i < APW; ++i) {
    const int r = 16 * (wave + 8 * i) + (lane >> 2);
    const int gm = m0 + r;
    aoff[i] = (unsigned)(gm < M ? gm : 0) * (unsigned)lda + (unsigned)(((lane & 3) ^ swz(r)) * 8);
  }
#pragma unroll
  for (int i = 0; i < BPW; ++i) {
    const int r = 16 * (wave + 8 * i) + (lane >> 2);
    const int gn = n0 + r;
    boff[i] = (unsigned)(gn < N ? gn : 0) * (unsigned)ldb + (unsigned)(((lane & 3) ^ swz(r)) * 8);
  }
  // Load j of the eight direct loads of a stage: j = 0..3 the A planes
  // (hi, lo of piece 0, then of piece 1), j = 4..7 the B planes.
  auto issue_one = [&](int j, int k0, _Float16* stage) {
    static_assert(APW == 2 && BPW == 2, "eight loads per stage");
    const int i = (j >> 1) & 1;
    if (j < 4) {
      _Float16* dst = stage + (wave + 8 * i) * 512;
      if (j & 1) dma16(Al + k0 + aoff[i], dst + A_PLANE); else dma16(Ah + k0 + aoff[i], dst);
    } else {
      _Float16* dst = stage + 2 * A_PLANE + (wave + 8 * i) * 512;
      if (j & 1) dma16(Bl + k0 + boff[i], dst + B_PLANE); else dma16(Bh + k0 + boff[i], dst);
    }
  };
  auto issue = [&](int k0, _Float16* stage) {
#pragma unroll
    for (int i = 0; i < APW; ++i) {
      _Float16* dst = stage + (wave + 8 * i) * 512;
      dma16(Ah + k0 + aoff[i], dst);
      dma16(Al + k0 + aoff[i], dst + A_PLANE);
    }
#pragma unroll
    for (int i = 0; i < BPW; ++i) {
      _Float16* dst = stage + 2 * A_PLANE + (wave + 8 * i) * 512;
      dma16(Bh + k0 + boff[i], dst);
      dma16(Bl + k0 + boff[i], dst + B_PLANE);
    }
  };

  f32x16 acc[4][NB];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = f32x16{};

  // Fragment reads are inline asm, paired with explicit waits whose operands
  // are the fragments they guard (the compiler neither sees when the data
  // arrives nor can move a use above its wait).  The reads also carry no
  // dependence on the direct loads, so no drain of those is inserted: every
  // stage is complete before the barrier that precedes its reads.
  auto lds_rd = [&](const _Float16* plane, int r, int ks) {
    const int c = (ks >> 3) + kh;
    const uint32_t ad = (uint32_t)(size_t)(const __attribute__((address_space(3))) void*)(
        plane + r * BK + ((c ^ swz(r)) << 3));
    f16x8 v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(ad));
    return v;
  };
  // One k-step on stage `base` as eight blocks s (k-slice s / 4, A row block
  // s % 4).  Block s first issues the reads for block s + 1 (block 1 also those
  // of the second k-slice's B fragments) and two of the next stage's direct
  // loads (into `stn` at k0n; none if k0n < 0), then waits only for the reads
  // issued before this block (LDS returns in order) and runs its 6 products,
  // so the reads of block s + 1 overlap them.
  auto compute = [&](const _Float16* base, int k0n, _Float16* stn) {
    f16x8 bh[2][NB], bl[2][NB], ah[2], al[2];
    auto loadB = [&](int ks, f16x8 (&h)[NB], f16x8 (&l)[NB]) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int r = wn * WN + b * 32 + lm;
        h[b] = lds_rd(base + 2 * A_PLANE, r, ks);
        l[b] = lds_rd(base + 2 * A_PLANE + B_PLANE, r, ks);
      }
    };
    auto loadA = [&](int ks, int a, f16x8& h, f16x8& l) {
      const int r = wm * 128 + a * 32 + lm;
      h = lds_rd(base, r, ks);
      l = lds_rd(base + A_PLANE, r, ks);
    };
    loadB(0, bh[0], bl[0]);
    loadA(0, 0, ah[0], al[0]);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int ksl = s >> 2, a = s & 3, c = s & 1;
      if (s + 1 < 8) loadA(((s + 1) >> 2) * 16, (s + 1) & 3, ah[c ^ 1], al[c ^ 1]);
      if (s == 1) loadB(16, bh[1], bl[1]);
      if (k0n >= 0 && s < 4) {
        issue_one(2 * s, k0n, stn);
        issue_one(2 * s + 1, k0n, stn);
      }
      static_assert(NB == 2, "wait operands list two B fragments");
#define JARQ_WAIT_OPS \
  "+v"(ah[c]), "+v"(al[c]), "+v"(bh[ksl][0]), "+v"(bh[ksl][1]), "+v"(bl[ksl][0]), "+v"(bl[ksl][1])
      if (s == 7)
        asm volatile("s_waitcnt lgkmcnt(0)" : JARQ_WAIT_OPS);
      else if (s == 1)
        asm volatile("s_waitcnt lgkmcnt(6)" : JARQ_WAIT_OPS);
      else
        asm volatile("s_waitcnt lgkmcnt(2)" : JARQ_WAIT_OPS);
#undef JARQ_WAIT_OPS
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[c], bh[ksl][b], acc[a][b], 0, 0, 0);
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[c], bl[ksl][b], acc[a][b], 0, 0, 0);
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al[c], bh[ksl][b], acc[a][b], 0, 0, 0);
      }
    }
  };

  // Double buffering: the loads of step k + 1 fly while step k computes; the
  // barrier at the end of a step (which waits for this thread's outstanding
  // loads) makes the next stage visible and frees the one just read.
  const int nk = K / BK;
  issue(0, buf0);
  __syncthreads();
  int kt = 0;
  for (; kt + 2 <= nk; kt += 2) {
    compute(buf0, (kt + 1) * BK, buf1);
    __syncthreads();
    compute(buf1, kt + 2 < nk ? (kt + 2) * BK : -1, buf0);
    __syncthreads();
  }
  if (kt < nk) compute(buf0, -1, buf1);  // odd step count: the last step sits in buf0

  // Epilogue.  Accumulator element v of lane l in a 32x32 block:
  // (row 8 * (v / 4) + 4 * (l / 32) + v % 4, column l % 32).
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int rb0 = m0 + wm * 128 + a * 32 + 4 * kh;  // row of element v: rb0 + 8 (v / 4) + v % 4
    // Unconditional loads from clamped addresses (a load under a branch is
    // waited for inside the branch); out-of-range elements are never stored.
    float rsc[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) rsc[v] = arow_inv[min(rb0 + 8 * (v / 4) + (v % 4), M - 1)];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int col = n0 + wn * WN + b * 32 + lm;
      const float cs = bcol_inv[min(col, N - 1)];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = rb0 + 8 * (v / 4) + (v % 4);
        if (row < M && col < N) C[(size_t)row * ldc + col] = acc[a][b][v] * (rsc[v] * cs);
      }
    }
  }
}

template <int BN>
static hipError_t launch_split3_t(hipStream_t st, int M, int N, int K, int lda, int ldb,
                                  int ldc, const _Float16* ah, const _Float16* al,
                                  const float* arow, const _Float16* bh, const _Float16* bl,
                                  const float* bcol, float* C, const int* m_dev) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (K % BK != 0) return hipErrorInvalidValue;
  const int tiles = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  hipLaunchKernelGGL((split3_kernel<BN>), dim3(tiles), dim3(512), 0, st, M, N, K, lda, ldb,
                     ldc, ah, al, arow, bh, bl, bcol, C, m_dev);
  return hipGetLastError();
}

// The same product in 64 x 64 tiles, 2 x 2 wavefronts of 32 x 32, for layers
// with too few 256-wide tiles; every element's products and their order are
// those of split3_kernel, so the results are the same bits.
__global__ __launch_bounds__(256, 1) void split3_small_kernel(
    int M, int N, int K, const _Float16* __restrict__ Ah, const _Float16* __restrict__ Al,
    const float* __restrict__ arow_inv, const _Float16* __restrict__ Bh,
    const _Float16* __restrict__ Bl, const float* __restrict__ bcol_inv, float* __restrict__ C) {
  constexpr int T = 64, PLANE = T * BK, STAGE = 4 * PLANE;   // halves
  __shared__ __attribute__((aligned(1024))) _Float16 buf0[STAGE];
  __shared__ __attribute__((aligned(1024))) _Float16 buf1[STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int lm = lane & 31, kh = lane >> 5;
  int tm, tn;
  if (!tile_of(blockIdx.x, (M + T - 1) / T, (N + T - 1) / T, tm, tn)) return;  // uniform
  const int m0 = tm * T, n0 = tn * T;
  // wave w fills the 1 KB piece w (16 rows) of each of the four planes
  const int r = 16 * wave + (lane >> 2);
  const unsigned chunk = (unsigned)(((lane & 3) ^ swz(r)) * 8);
  const unsigned aoff = (unsigned)(m0 + r < M ? m0 + r : 0) * (unsigned)K + chunk;
  const unsigned boff = (unsigned)(n0 + r < N ? n0 + r : 0) * (unsigned)K + chunk;
  auto issue = [&](int k0, _Float16* stage) {
    _Float16* dst = stage + wave * 512;
    dma16(Ah + k0 + aoff, dst);
    dma16(Al + k0 + aoff, dst + PLANE);
    dma16(Bh + k0 + boff, dst + 2 * PLANE);
    dma16(Bl + k0 + boff, dst + 3 * PLANE);
  };
  f32x16 acc = f32x16{};
  auto compute = [&](const _Float16* st) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      auto frag = [&](int plane, int row) __attribute__((always_inline)) {
        return *(const f16x8*)(st + plane * PLANE + row * BK + (((2 * ks + kh) ^ swz(row)) << 3));
      };
      const f16x8 ah = frag(0, wm * 32 + lm), al = frag(1, wm * 32 + lm);
      const f16x8 bh = frag(2, wn * 32 + lm), bl = frag(3, wn * 32 + lm);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh, acc, 0, 0, 0);
    }
  };
  const int nk = K / BK;
  issue(0, buf0);
  __syncthreads();
  for (int kt = 0; kt < nk; kt += 2) {
    // a stage was last read before the barrier that precedes its loads; the
    // barrier after a step waits for the next one's loads
    if (kt + 1 < nk) issue((kt + 1) * BK, buf1);
    compute(buf0);
    __syncthreads();
    if (kt + 1 < nk) {
      if (kt + 2 < nk) issue((kt + 2) * BK, buf0);
      compute(buf1);
      __syncthreads();
    }
  }
  const int col = n0 + wn * 32 + lm;
  const float cs = bcol_inv[min(col, N - 1)];
  float rsc[16];
#pragma unroll
  for (int v = 0; v < 16; ++v)
    rsc[v] = arow_inv[min(m0 + wm * 32 + 8 * (v / 4) + 4 * kh + (v % 4), M - 1)];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int row = m0 + wm * 32 + 8 * (v / 4) + 4 * kh + (v % 4);
    if (row < M && col < N) C[(size_t)row * N + col] = acc[v] * (rsc[v] * cs);
  }
}

// T = W M^T for the layer, all rows (jarq_prepare): W's two fp16 planes
// against M's, three products.
hipError_t launch_wm_product(hipStream_t st, int rows, int cols, const char* ws,
                             const Layout& lay, const _Float16* whi, const _Float16* wlo,
                             const float* wrow_inv) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  const _Float16* bh = (const _Float16*)(ws + lay.mhi);
  const _Float16* bl = (const _Float16*)(ws + lay.mlo);
  const float* bc = (const float*)(ws + lay.mrow);
  // 64 x 64 tiles where there are few of 256 x 256 (a whole set-up, large tiles
  // and small: 611 x 1312, 18 large tiles, 175 and 123 us; 300 x 11008, 86 of
  // them, 1711 and 1565; 1500 x 4096, 96, 511 and 522)
  const long long big = (long long)((rows + 255) / 256) * ((cols + 255) / 256);
  if (big < 96) {
    if (cols % BK != 0) return hipErrorInvalidValue;
    const int tiles = ((rows + 63) / 64) * ((cols + 63) / 64);
    hipLaunchKernelGGL(split3_small_kernel, dim3(tiles), dim3(256), 0, st, rows, cols, cols, whi,
                       wlo, wrow_inv, bh, bl, bc, (float*)(ws + lay.tm));
    return hipGetLastError();
  }
  return launch_split3_t<256>(st, rows, cols, cols, cols, cols, cols, whi, wlo, wrow_inv, bh,
                                 bl, bc, (float*)(ws + lay.tm), nullptr);
}

// ---- residual product from the exact codes ----
//
// With E = W - What and What(j, k) = s(j, i) (q(j, k) - z(j, i)) for k in group
// i (eq. (1)), U = E M^T = T - What M^T with T = W M^T fixed for the layer
// (formed once by jarq_prepare with split3_kernel).  The codes minus
// zero points are small integers, exact in fp16 (the cz plane), so
//   (What M^T)(j, n) = 2^-t_n sum_i s(j, i) sum_{k in i} cz(j, k) (Mh + Ml)(n, k)
// needs two products per k-slice instead of three; each group's partial sum
// (seg, exact products accumulated in fp32 on the matrix cores) is scaled by
// its row's s and added to the running sum in fp32 when the group ends.
//
// Tiling: 256 x 128 output tile per 512-thread work-group, 4 x 2 waves of
// 64 x 64 (two 32 x 32 blocks each way: the accumulators and the group's
// partial sums both fit next to the fragments at two waves per SIMD), or 64 x 64
// per 256 threads, 2 x 2 waves of 32 x 32 (the same products in the same order),
// by the number of tiles (launch_resid); K in steps of 64 (32 when g = 32) straight from global memory into two LDS
// stages by direct loads.  A stage row holds CPR 16-byte chunks; chunk c of
// tile row r sits at position c ^ rswz(r).  A 16-byte read serves 16 lanes
// (256 bytes, all 64 banks) per clock, and the lanes of a fragment read are
// 16 consecutive rows at one chunk: with 128-byte rows, two rows share each
// 256-byte bank line, so row r's position must differ from every other row
// of the 16 with the same parity (rswz = (r / 2) mod 8); with 64-byte rows,
// four rows share a line and (r / 4) mod 4 separates the rows of each
// residue mod 4.  Fragment reads run one k-slice ahead of the products.  Rows
// of cz, the scales and T are the layer's rows (gathered through the row
// map); U is stored by position.
namespace {
template <int CPR>
__device__ __forceinline__ int rswz(int r) {
  if constexpr (CPR == 8) return (r >> 1) & 7;
  return (r >> 2) & 3;
}
}  // namespace

template <int G_SIZE, bool BIG>
__global__ __launch_bounds__(BIG ? 512 : 256, 1) void resid_kernel(
    int M, int N, int K, const _Float16* __restrict__ Cz, const float* __restrict__ scales,
    const _Float16* __restrict__ Bh, const _Float16* __restrict__ Bl,
    const float* __restrict__ bcol_inv, const float* __restrict__ T, float* __restrict__ U,
    const int32_t* __restrict__ rowmap, const int* __restrict__ m_dev) {
  if (m_dev != nullptr) M = *m_dev;
  constexpr int g = G_SIZE;
  constexpr int RBM = BIG ? 256 : 64, RBN = BIG ? 128 : 64;
  constexpr int NW = BIG ? 8 : 4;                        // wavefronts, two along the columns
  constexpr int AB = BIG ? 2 : 1;                        // 32 x 32 blocks per wavefront each way
  constexpr int WT = 32 * AB;                            // wavefront tile
  constexpr int RBK = g >= 64 ? 64 : 32;                 // k per stage
  constexpr int KQ = RBK / 16;                           // k-slices per stage
  constexpr int CPR = RBK / 8;                           // 16-byte chunks per stage row
  constexpr int RPP = 64 / CPR;                          // rows per 1 KB piece
  constexpr int SPG = g / RBK;                           // stages per group
  constexpr int A_PLANE = RBM * RBK, B_PLANE = RBN * RBK;  // halves
  constexpr int APW = RBM / RPP / NW, BPW = RBN / RPP / NW;  // pieces per wave per plane
  constexpr int STAGE = A_PLANE + 2 * B_PLANE;
  __shared__ __attribute__((aligned(1024))) _Float16 buf0[STAGE];
  __shared__ __attribute__((aligned(1024))) _Float16 buf1[STAGE];
  __shared__ __attribute__((aligned(16))) float sc_s[2][RBM];  // s of the tile's rows, current / next group
  __shared__ int lr_s[RBM];                                     // layer row of each tile row
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int lm = lane & 31, kh = lane >> 5;
  const int G = K / g;
  const int nbm = (M + RBM - 1) / RBM, nbn = (N + RBN - 1) / RBN;
  int tm, tn;
  if (M <= 0 || !tile_of(blockIdx.x, nbm, nbn, tm, tn)) return;  // uniform across the work-group
  const int m0 = tm * RBM, n0 = tn * RBN;
  // Tile rows past the edge take the tile's first row: their products only
  // reach outputs that are never stored.
  if (tid < RBM) lr_s[tid] = map_row(rowmap, m0 + (m0 + tid < M ? tid : 0));
  __syncthreads();

  // Direct loads, 16 bytes per lane, one 1 KB piece (RPP rows) per
  // instruction: wave w fills pieces w, w + NW, ... of each plane; lane L holds
  // row RPP j + L / CPR at position L % CPR, i.e. chunk (L % CPR) ^ rswz(row).
  unsigned aoff[APW], boff[BPW];
#pragma unroll
  for (int i = 0; i < APW; ++i) {
    const int r = RPP * (wave + NW * i) + lane / CPR;
    aoff[i] = (unsigned)lr_s[r] * (unsigned)K + (unsigned)(((lane % CPR) ^ rswz<CPR>(r)) * 8);
  }
#pragma unroll
  for (int i = 0; i < BPW; ++i) {
    const int r = RPP * (wave + NW * i) + lane / CPR;
    const int gn = n0 + r;
    boff[i] = (unsigned)(gn < N ? gn : 0) * (unsigned)K + (unsigned)(((lane % CPR) ^ rswz<CPR>(r)) * 8);
  }
  // load j (0 .. NDMA - 1) of a stage's direct loads: the cz pieces first,
  // then the M pieces, high and low plane in turn
  constexpr int NDMA = APW + 2 * BPW;
  auto issue_one = [&](int j, int k0, _Float16* stage) {
    if (j < APW) {
      dma16(Cz + k0 + aoff[j], stage + (wave + NW * j) * 512);
    } else {
      const int i = (j - APW) >> 1;
      if (((j - APW) & 1) == 0)
        dma16(Bh + k0 + boff[i], stage + A_PLANE + (wave + NW * i) * 512);
      else
        dma16(Bl + k0 + boff[i], stage + A_PLANE + B_PLANE + (wave + NW * i) * 512);
    }
  };
  auto issue = [&](int k0, _Float16* stage) {
#pragma unroll
    for (int j = 0; j < NDMA; ++j) issue_one(j, k0, stage);
  };
  // the tile's scales of group i into sc_s[i & 1] (threads 0..RBM-1)
  auto stage_scales = [&](int i) {
    if (tid < RBM) sc_s[i & 1][tid] = scales[(size_t)lr_s[tid] * G + i];
  };

  f32x16 acc[AB][AB], seg[AB][AB];
#pragma unroll
  for (int a = 0; a < AB; ++a)
#pragma unroll
    for (int b = 0; b < AB; ++b) acc[a][b] = f32x16{};

  auto lds_rd = [&](const _Float16* plane, int r, int q) {
    const int c = 2 * q + kh;  // k-slice q: chunks 2 q (lanes 0-31) and 2 q + 1
    const uint32_t ad = (uint32_t)(size_t)(const __attribute__((address_space(3))) void*)(
        plane + r * RBK + ((c ^ rswz<CPR>(r)) << 3));
    f16x8 v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(ad));
    return v;
  };
  // One stage (KQ k-slices of 16) on `base`; `first`: the stage opens a group
  // (its products start the partial sums from zero).  The 3 AB reads of slice
  // q + 1 are issued before the wait for slice q (LDS returns in order), and
  // the next stage's direct loads (into `stn` at k0n; none if k0n < 0) are
  // spread over the slices.
  auto compute = [&](const _Float16* base, bool first, int k0n, _Float16* stn) {
    f16x8 af[2][AB], bh[2][AB], bl[2][AB];  // [slot][block]
    auto rd = [&](int q, int sl) {
#pragma unroll
      for (int a = 0; a < AB; ++a) af[sl][a] = lds_rd(base, wm * WT + a * 32 + lm, q);
#pragma unroll
      for (int b = 0; b < AB; ++b) {
        bh[sl][b] = lds_rd(base + A_PLANE, wn * WT + b * 32 + lm, q);
        bl[sl][b] = lds_rd(base + A_PLANE + B_PLANE, wn * WT + b * 32 + lm, q);
      }
    };
    rd(0, 0);
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
      const int sl = q & 1;
      if (k0n >= 0) {
#pragma unroll
        for (int j = q * NDMA / KQ; j < (q + 1) * NDMA / KQ; ++j) issue_one(j, k0n, stn);
      }
      const bool more = q + 1 < KQ;
      if (more) rd(q + 1, sl ^ 1);
      // wait for slice q's reads (all but the ones just issued); the operands
      // are the fragments that the wait guards
      if constexpr (AB == 2) {
#define JARQ_WAIT_OPS(x) \
  "+v"(af[x][0]), "+v"(af[x][1]), "+v"(bh[x][0]), "+v"(bh[x][1]), "+v"(bl[x][0]), "+v"(bl[x][1])
        if (more && sl == 0) asm volatile("s_waitcnt lgkmcnt(6)" : JARQ_WAIT_OPS(0));
        if (more && sl == 1) asm volatile("s_waitcnt lgkmcnt(6)" : JARQ_WAIT_OPS(1));
        if (!more && sl == 0) asm volatile("s_waitcnt lgkmcnt(0)" : JARQ_WAIT_OPS(0));
        if (!more && sl == 1) asm volatile("s_waitcnt lgkmcnt(0)" : JARQ_WAIT_OPS(1));
#undef JARQ_WAIT_OPS
      } else {
#define JARQ_WAIT_OPS(x) "+v"(af[x][0]), "+v"(bh[x][0]), "+v"(bl[x][0])
        if (more && sl == 0) asm volatile("s_waitcnt lgkmcnt(3)" : JARQ_WAIT_OPS(0));
        if (more && sl == 1) asm volatile("s_waitcnt lgkmcnt(3)" : JARQ_WAIT_OPS(1));
        if (!more && sl == 0) asm volatile("s_waitcnt lgkmcnt(0)" : JARQ_WAIT_OPS(0));
        if (!more && sl == 1) asm volatile("s_waitcnt lgkmcnt(0)" : JARQ_WAIT_OPS(1));
#undef JARQ_WAIT_OPS
      }
#pragma unroll
      for (int a = 0; a < AB; ++a)
#pragma unroll
        for (int b = 0; b < AB; ++b) {
          const f32x16 c0 = (first && q == 0) ? f32x16{} : seg[a][b];
          seg[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[sl][a], bh[sl][b], c0, 0, 0, 0);
          seg[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[sl][a], bl[sl][b], seg[a][b], 0, 0, 0);
        }
    }
  };
  // acc += s (per row) * seg at the end of group i; element v of a block is
  // row 8 (v / 4) + 4 (lane / 32) + v % 4
  auto fold = [&](int i) {
#pragma unroll
    for (int a = 0; a < AB; ++a) {
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const f32x4 s4 = *(const f32x4*)&sc_s[i & 1][wm * WT + a * 32 + 8 * v4 + 4 * kh];
#pragma unroll
        for (int b = 0; b < AB; ++b)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            acc[a][b][4 * v4 + u] = fmaf(seg[a][b][4 * v4 + u], s4[u], acc[a][b][4 * v4 + u]);
      }
    }
  };

  // Double buffering: the loads of stage k + 1 fly while stage k computes;
  // the barrier at the end of a stage (which waits for this thread's
  // outstanding loads) makes the next stage visible and frees the one just
  // read.  The scales of group i + 1 are staged during group i (their buffer
  // was last read by group i - 1's fold, before a barrier).
  const int nk = K / RBK;
  stage_scales(0);
  issue(0, buf0);
  __syncthreads();
  for (int i = 0; i < G; ++i) {
    if (i + 1 < G) stage_scales(i + 1);
#pragma unroll
    for (int ks = 0; ks < SPG; ++ks) {  // unrolled: whether a stage opens its group is known
      const int kt = i * SPG + ks;
      _Float16* cur = (kt & 1) ? buf1 : buf0;
      _Float16* nxt = (kt & 1) ? buf0 : buf1;
      compute(cur, ks == 0, kt + 1 < nk ? (kt + 1) * RBK : -1, nxt);
      if (ks == SPG - 1) fold(i);
      __syncthreads();
    }
  }

  // Epilogue: U = T - acc 2^-t_n.  Accumulator element v of lane l in a
  // 32 x 32 block: (row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32).
#pragma unroll
  for (int a = 0; a < AB; ++a) {
    const int tb = wm * WT + a * 32 + 4 * kh;  // tile row of element v: tb + 8 (v / 4) + v % 4
#pragma unroll
    for (int b = 0; b < AB; ++b) {
      const int col = n0 + wn * WT + b * 32 + lm;
      const int colc = min(col, N - 1);
      const float cs = bcol_inv[colc];
      float tv[16];
#pragma unroll
      for (int v = 0; v < 16; ++v)
        tv[v] = T[(size_t)lr_s[tb + 8 * (v / 4) + (v % 4)] * N + colc];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = m0 + tb + 8 * (v / 4) + (v % 4);
        if (row < M && col < N) U[(size_t)row * N + col] = tv[v] - acc[a][b][v] * cs;
      }
    }
  }
}

template <int G_SIZE, bool BIG>
static hipError_t launch_resid_t(hipStream_t st, int rows, int cols, const char* ws,
                                 const Layout& lay, const float* scales, float* U,
                                 const int32_t* rowmap, const int* n_dev, hipEvent_t ev_start,
                                 hipEvent_t ev_stop) {
  constexpr int RBM = BIG ? 256 : 64, RBN = BIG ? 128 : 64;
  const dim3 grid(((rows + RBM - 1) / RBM) * ((cols + RBN - 1) / RBN)), block(BIG ? 512 : 256);
  if (ev_start != nullptr || ev_stop != nullptr) {
    // timed: the events take the dispatch's own timestamps
    hipExtLaunchKernelGGL((resid_kernel<G_SIZE, BIG>), grid, block, 0, st, ev_start, ev_stop, 0u,
                          rows, cols, cols, (const _Float16*)(ws + lay.cz), scales,
                          (const _Float16*)(ws + lay.mhi), (const _Float16*)(ws + lay.mlo),
                          (const float*)(ws + lay.mrow), (const float*)(ws + lay.tm), U, rowmap,
                          n_dev);
  } else {
    hipLaunchKernelGGL((resid_kernel<G_SIZE, BIG>), grid, block, 0, st, rows, cols, cols,
                       (const _Float16*)(ws + lay.cz), scales, (const _Float16*)(ws + lay.mhi),
                       (const _Float16*)(ws + lay.mlo), (const float*)(ws + lay.mrow),
                       (const float*)(ws + lay.tm), U, rowmap, n_dev);
  }
  return hipGetLastError();
}

hipError_t launch_resid(hipStream_t st, int rows, int cols, int g, const char* ws,
                        const Layout& lay, const float* scales, float* U, const int32_t* rowmap,
                        const int* n_dev, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (rows <= 0 || cols <= 0) {  // nothing to launch: the events still mark the spot
    hipError_t e = hipSuccess;
    if (ev_start != nullptr) e = hipEventRecord(ev_start, st);
    if (e == hipSuccess && ev_stop != nullptr) e = hipEventRecord(ev_stop, st);
    return e;
  }
  if (cols % BK != 0) return hipErrorInvalidValue;
  // 64 x 64 tiles where 256 x 128 ones would leave half of the compute units
  // without work (a whole code update, large tiles and small: 512 x 4096, 64
  // large tiles, 432 and 383 us; 1024 x 4096, 128 of them, 437 and 441; 2048 x
  // 4096 492 and 556)
  const long long big = (long long)((rows + 255) / 256) * ((cols + 127) / 128);
#define JARQ_RESID(g)                                                                            \
  case g:                                                                                        \
    return (big >= 128 ? launch_resid_t<g, true> : launch_resid_t<g, false>)(                    \
        st, rows, cols, ws, lay, scales, U, rowmap, n_dev, ev_start, ev_stop)
  switch (g) {
    JARQ_RESID(32);
    JARQ_RESID(64);
    JARQ_RESID(128);
    default: return hipErrorInvalidValue;
  }
#undef JARQ_RESID
}

// ---- W H (the right-hand sides of the scale update, App. G.8) ----
//
// An fp32-grade product of fp32 operands: both as three bf16 planes, which hold
// all 24 bits of every value whatever the range of its row, and the six products
// above 2^-25 relative (bf16x3.h), so that what is exact in fp32 (small
// integers) stays exact.  (Taking W H from T = W M^T and L_i is cheaper, 0.18
// instead of 5.3 ms at 4096 x 11008, but M is rounded and the fp16 planes hold 22
// bits below the largest value of a row: integers lost their last bits, and rows
// that span more than 2^17 their small weights.)
//
// H is symmetric, so B(k, n) = H(k, n) is read along row n.  256 x 128 tiles, 4 x 2
// wavefronts of 64 x 64, or 64 x 64 tiles of 2 x 2 wavefronts of 32 x 32 (the same
// products in the same order: the same bits), K in steps of 32 straight from
// memory into two LDS stages.  Bound by the matrix cores: 4096 x 4096 0.7 ms with
// the splits (1.2 PFLOP/s), 4096 x 11008 5.6 ms (the fp32 instruction: 1.5 and
// 17.8 ms).
namespace {
// n8 pieces of eight values of x as three planes.
__global__ __launch_bounds__(256) void split_bf16x3_kernel(const float* __restrict__ x, size_t n8,
                                                           u32x4* __restrict__ h,
                                                           u32x4* __restrict__ m,
                                                           u32x4* __restrict__ l) {
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n8; e += (size_t)gridDim.x * 256) {
    const f32x4 v0 = ((const f32x4*)x)[2 * e], v1 = ((const f32x4*)x)[2 * e + 1];
    u32x4 p[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t a, b, c;
      split_pair(i < 2 ? v0[2 * i] : v1[2 * i - 4], i < 2 ? v0[2 * i + 1] : v1[2 * i - 3], a, b, c);
      p[0][i] = a, p[1][i] = b, p[2][i] = c;
    }
    h[e] = p[0];
    m[e] = p[1];
    l[e] = p[2];
  }
}

hipError_t launch_split_bf16x3(hipStream_t st, const float* x, size_t n, __bf16* const (&pl)[3]) {
  const size_t n8 = n / 8, blocks = (n8 + 255) / 256;   // cols is a multiple of 32
  hipLaunchKernelGGL(split_bf16x3_kernel, dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256),
                     0, st, x, n8, (u32x4*)pl[0], (u32x4*)pl[1], (u32x4*)pl[2]);
  return hipGetLastError();
}

struct Planes {
  const __bf16* p[3];
};

// The 32 x 32 block of W H at (r0, c0) with the fp32 instruction straight from
// memory (one wavefront): for sums the planes cannot do (bf16x3.h).
__device__ __forceinline__ f32x16 wh_slow_block(const float* __restrict__ W,
                                                const float* __restrict__ H, int M, int N, int r0,
                                                int c0) {
  const int lane = threadIdx.x & 63, lm = lane & 31, kh = lane >> 5;
  const float* w = W + (size_t)min(r0 + lm, M - 1) * N + kh;
  const float* h = H + (size_t)min(c0 + lm, N - 1) * N + kh;
  f32x16 acc = f32x16{};
  for (int k = 0; k < N; k += 2)   // N is even
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[k], h[k], acc, 0, 0, 0);
  return acc;
}
}  // namespace

// C [M][N] = A B, A [M][N] and B [N][N] symmetric.
template <bool BIG>
__global__ __launch_bounds__(BIG ? 512 : 256, 1) void wh_kernel(int M, int N, Planes A, Planes B,
                                                                const float* __restrict__ W,
                                                                const float* __restrict__ H,
                                                                float* __restrict__ C) {
  constexpr int TM = BIG ? 256 : 64, TN = BIG ? 128 : 64;
  constexpr int NW = BIG ? 8 : 4, AB = BIG ? 2 : 1, WT = 32 * AB;
  constexpr int A_PLANE = TM * BK, B_PLANE = TN * BK;          // values
  constexpr int STAGE = 3 * (A_PLANE + B_PLANE);
  constexpr int APW = TM / 16 / NW, BPW = TN / 16 / NW;        // 1 KB pieces per wave and plane
  __shared__ __attribute__((aligned(1024))) _Float16 buf0[STAGE];
  __shared__ __attribute__((aligned(1024))) _Float16 buf1[STAGE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int lm = lane & 31, kh = lane >> 5;
  int tm, tn;
  if (!tile_of(blockIdx.x, (M + TM - 1) / TM, (N + TN - 1) / TN, tm, tn)) return;  // uniform
  const int m0 = tm * TM, n0 = tn * TN;
  // rows past the edge read the tile's first row: their results are not stored
  unsigned aoff[APW], boff[BPW];
#pragma unroll
  for (int i = 0; i < APW; ++i) {
    const int r = 16 * (wave + NW * i) + (lane >> 2);
    aoff[i] = (unsigned)(m0 + r < M ? r : 0) * (unsigned)N + (unsigned)(((lane & 3) ^ swz(r)) * 8);
  }
#pragma unroll
  for (int i = 0; i < BPW; ++i) {
    const int r = 16 * (wave + NW * i) + (lane >> 2);
    boff[i] = (unsigned)(n0 + r < N ? r : 0) * (unsigned)N + (unsigned)(((lane & 3) ^ swz(r)) * 8);
  }
  const size_t a0 = (size_t)m0 * N, b0 = (size_t)n0 * N;
  auto issue = [&](int k0, _Float16* stage) {
#pragma unroll
    for (int p = 0; p < 3; ++p) {
#pragma unroll
      for (int i = 0; i < APW; ++i)
        dma16((const _Float16*)(A.p[p] + a0 + k0) + aoff[i],
              stage + p * A_PLANE + (wave + NW * i) * 512);
#pragma unroll
      for (int i = 0; i < BPW; ++i)
        dma16((const _Float16*)(B.p[p] + b0 + k0) + boff[i],
              stage + 3 * A_PLANE + p * B_PLANE + (wave + NW * i) * 512);
    }
  };
  f32x16 big[AB][AB], low[AB][AB];
#pragma unroll
  for (int b = 0; b < AB; ++b)
#pragma unroll
    for (int a = 0; a < AB; ++a) big[b][a] = low[b][a] = f32x16{};
  auto compute = [&](const _Float16* st) __attribute__((always_inline)) {
    auto frag = [&](const _Float16* plane, int r, int ks) __attribute__((always_inline)) {
      return *(const bf16x8*)(plane + r * BK + (((2 * ks + kh) ^ swz(r)) << 3));
    };
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 fa[AB][3], fb[AB][3];
#pragma unroll
      for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int a = 0; a < AB; ++a) {
          fa[a][p] = frag(st + p * A_PLANE, wm * WT + a * 32 + lm, ks);
          fb[a][p] = frag(st + 3 * A_PLANE + p * B_PLANE, wn * WT + a * 32 + lm, ks);
        }
#pragma unroll
      for (int b = 0; b < AB; ++b) mfma_bf16x3<AB>(fa, fb[b], big[b], low[b]);
    }
  };
  const int nk = N / BK;
  issue(0, buf0);
  __syncthreads();
  for (int kt = 0; kt < nk; kt += 2) {
    // a stage was last read before the barrier that precedes its loads; the
    // barrier after a step waits for the next one's loads
    if (kt + 1 < nk) issue((kt + 1) * BK, buf1);
    compute(buf0);
    __syncthreads();
    if (kt + 1 < nk) {
      if (kt + 2 < nk) issue((kt + 2) * BK, buf0);
      compute(buf1);
      __syncthreads();
    }
  }
#pragma unroll
  for (int a = 0; a < AB; ++a)
#pragma unroll
    for (int b = 0; b < AB; ++b) {
      const int rb = m0 + wm * WT + a * 32, cb = n0 + wn * WT + b * 32;
      f32x16 acc = big[b][a] + low[b][a];
      bool fine = true;
#pragma unroll
      for (int v = 0; v < 16; ++v) fine &= isfinite(acc[v]);
      if (!__all(fine)) {
        const f32x16 slow = wh_slow_block(W, H, M, N, rb, cb);
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = isfinite(acc[v]) ? acc[v] : slow[v];
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = rb + 8 * (v / 4) + 4 * kh + (v % 4);
        if (row < M && cb + lm < N) C[(size_t)row * N + cb + lm] = acc[v];
      }
    }
}

hipError_t launch_wh(hipStream_t st, int rows, int cols, const float* W, const float* H, char* ws,
                     const Layout& lay) {
  if (cols % BK != 0) return hipErrorInvalidValue;
  __bf16* const wp[3] = {(__bf16*)(ws + lay.cz), (__bf16*)(ws + lay.dq), (__bf16*)(ws + lay.p)};
  __bf16* const hp[3] = {(__bf16*)(ws + lay.hhi), (__bf16*)(ws + lay.hlo), (__bf16*)(ws + lay.mhi)};
  hipError_t e = launch_split_bf16x3(st, W, (size_t)rows * cols, wp);
  if (e == hipSuccess) e = launch_split_bf16x3(st, H, (size_t)cols * cols, hp);
  if (e != hipSuccess) return e;
  const Planes A{{wp[0], wp[1], wp[2]}}, B{{hp[0], hp[1], hp[2]}};
  float* C = (float*)(ws + lay.wh);
  // large tiles from 160 of them on (a whole set-up, large tiles and small:
  // 1024 x 4096, 128 large tiles, 748 and 723 us; 1280 x 4096, 160 of them, 807 and
  // 819; 1536 x 4096 818 and 886)
  const long long big = (long long)((rows + 255) / 256) * ((cols + 127) / 128);
  if (big >= 160)
    hipLaunchKernelGGL(wh_kernel<true>, dim3((unsigned)big), dim3(512), 0, st, rows, cols, A, B, W,
                       H, C);
  else
    hipLaunchKernelGGL(wh_kernel<false>, dim3(((rows + 63) / 64) * ((cols + 63) / 64)), dim3(256),
                       0, st, rows, cols, A, B, W, H, C);
  return hipGetLastError();
}

}  // namespace jarq
