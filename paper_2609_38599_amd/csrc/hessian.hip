// The calibration Hessian (App. E.1): with A = [X~; nu I], H = A^T A =
// X~^T X~ + nu^2 I.  The calibration inputs arrive in chunks of tokens; the
// kernels add alpha X^T X of one chunk (X: m tokens x d channels, row-major) to
// an fp64 accumulator in full symmetric storage, and alpha Xq^T (X - Xq), the
// propagation term of App. E.5, to one that is not symmetric.  Sums are fp32
// over at most 256 tokens; those are added in fp64.  An entry (a, b) with
// a <= b is computed once and stored at (a, b) and (b, a), so the accumulator
// stays exactly symmetric.
//
// bf16 inputs: products of bf16 values are exact in fp32, so
// v_mfma_f32_32x32x16_bf16 forms them at 16 times the fp32 matrix rate.
//
// fp32 inputs: as three bf16 planes, six exact products (bf16x3.h).  A block
// whose sums come out infinite or NaN is formed again with the fp32
// instruction, which treats such inputs as fp32 arithmetic does.
//
// Work: 128 x 128 tiles, 128 x 64 and 64 x 64 ones (Split below), each with its fp64
// sums of 256-token partial sums in registers.  Bound by the matrix cores and the
// reads that feed them.  8192 tokens x 4096 channels: bf16 0.25 ms (0.55 PFLOP/s;
// 64 x 64 tiles staged through registers: 0.41), fp32 1.0 ms (the fp32
// instruction: 1.45).
#include "bf16x3.h"
#include "token_spans.h"

namespace jarq {

namespace {
// The tiles of one launch: `big` 128 x 128 tiles (of the strict upper triangle,
// or of the full grid for the cross term), then smaller ones: the three 64 x 64 of
// each diagonal tile (symmetric), and each of the last `cut` big ones in `parts`
// parts, two of 128 x 64 or four of 64 x 64.
struct Split {
  int nt;       // 128-wide tiles per side
  int big, cut, parts, small;
};
Split split_of(int d, bool sym) {
  Split s;
  s.nt = (d + 127) / 128;
  s.big = sym ? s.nt * (s.nt - 1) / 2 : s.nt * s.nt;
  s.cut = 0;
  s.parts = 4;
  s.small = sym ? 3 * s.nt : 0;
  return s;
}
void cut_last(Split& s, int cut, int parts) {
  s.big -= cut;
  s.cut = cut;
  s.parts = parts;
  s.small += parts * cut;
}

// Tile `id` of the strict upper triangle, row by row.
__device__ __forceinline__ void upper_tile(int id, int nt, int& ta, int& tb) {
  const float q = 2.f * nt - 1.f;
  ta = (int)((q - sqrtf(fmaxf(q * q - 8.f * (float)id, 0.f))) * 0.5f);
  ta = max(0, min(ta, nt - 2));
  auto start = [&](int r) { return r * (nt - 1) - r * (r - 1) / 2; };
  while (ta > 0 && start(ta) > id) --ta;
  while (ta + 1 < nt - 1 && start(ta + 1) <= id) ++ta;
  tb = ta + 1 + id - start(ta);
}

// Origin of the work-group's tile and its edges.
enum Tile { kWhole, kHalf, kQuarter };   // 128 x 128, 128 x 64, 64 x 64
template <bool CROSS>
__device__ __forceinline__ Tile tile_of(int id, const Split& s, int& a0, int& b0) {
  int ta, tb;
  auto big_tile = [&](int t) {
    if (CROSS) {
      ta = t / s.nt;
      tb = t % s.nt;
    } else {
      upper_tile(t, s.nt, ta, tb);
    }
    a0 = 128 * ta;
    b0 = 128 * tb;
  };
  if (id < s.big) {
    big_tile(id);
    return kWhole;
  }
  id -= s.big;
  if (id < s.parts * s.cut) {
    big_tile(s.big + id / s.parts);
    const int q = id % s.parts;
    b0 += 64 * (q & 1);
    a0 += 64 * (q >> 1);
    return s.parts == 2 ? kHalf : kQuarter;
  }
  id -= s.parts * s.cut;
  const int q = id % 3;   // (0, 0), (0, 1), (1, 1)
  a0 = 128 * (id / 3) + 64 * (q >> 1);
  b0 = 128 * (id / 3) + 64 * (q > 0);
  return kQuarter;
}

// Adds alpha sum to the accumulator at the 32 x 32 block (a0, b0): element v
// of a lane is (a0 + 8 (v / 4) + 4 (lane / 32) + v % 4, b0 + lane % 32).  The
// product alpha * sum is rounded once and the new value stored at both
// places (no contraction into an fma).  buf: 32 x 33 doubles of LDS of this
// wave, through which the mirrored block is stored along rows.
__device__ __forceinline__ void add_block(double* __restrict__ Hacc, int d, double alpha, int a0,
                                          int b0, const double (&sum)[16], double* buf) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63, lc = lane & 31, kh = lane >> 5;
  const int b = b0 + lc;
  double old[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    // (clamped: every load goes out, none under a branch)
    const int a = min(a0 + 8 * (v / 4) + 4 * kh + (v % 4), d - 1);
    old[v] = Hacc[(size_t)a * d + min(b, d - 1)];
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int a = a0 + 8 * (v / 4) + 4 * kh + (v % 4);
    const double t = alpha * sum[v];
    const double now = old[v] + t;
    if (b < d && a <= b) Hacc[(size_t)a * d + b] = now;
    buf[(a - a0) * 33 + lc] = now;
  }
  // (one wavefront: its LDS accesses complete in order)
  asm volatile("" ::: "memory");
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int i = 2 * v + kh;   // mirrored row b0 + i, columns a0 + lane % 32
    if (a0 + lc < b0 + i && b0 + i < d) Hacc[(size_t)(b0 + i) * d + a0 + lc] = buf[lc * 33 + i];
  }
  asm volatile("" ::: "memory");
}

// The same for the AB blocks from row a0 on of an accumulator that is not
// symmetric, every load ahead of the stores (with few tokens a launch lasts as
// long as these: 60 tokens x 4096 channels 63 us, block by block 69).
template <int AB>
__device__ __forceinline__ void add_blocks(double* __restrict__ Dacc, int d, double alpha, int a0,
                                           int b0, const double (&sum)[AB][16]) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63, kh = lane >> 5;
  const int b = b0 + (lane & 31);
  double old[AB][16];
#pragma unroll
  for (int i = 0; i < AB; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int a = min(a0 + 32 * i + 8 * (v / 4) + 4 * kh + (v % 4), d - 1);
      old[i][v] = Dacc[(size_t)a * d + min(b, d - 1)];
    }
#pragma unroll
  for (int i = 0; i < AB; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int a = a0 + 32 * i + 8 * (v / 4) + 4 * kh + (v % 4);
      const double t = alpha * sum[i][v];
      if (a < d && b < d) Dacc[(size_t)a * d + b] = old[i][v] + t;
    }
}

}  // namespace

// ---- bf16 inputs ----
// 256 threads, 2 x 2 wavefronts of 64 x 64 (big tile) or 32 x 32; two
// work-groups per CU, so that one's barriers and fp64 sums are covered by the
// other's products.  Chunks of 64 tokens go straight from memory to LDS
// (global_load_lds_dwordx4, token-major as they are), one chunk ahead, and
// fragments come out through the transposing read (ds_read_b64_tr_b16): in
// each 16-lane group, lane p points at token base + p / 4, channels 4 (p % 4)
// .. +3, and lane i receives channel i of tokens base .. base + 3 - the
// matrix-core operand layout, with the same token order in A and B.  A half
// wave reads 64 bytes of four consecutive tokens, so the 64-byte blocks of a
// token's row are permuted by the token (swz) to put the four in distinct banks.
namespace {
constexpr int BCH = 64;   // tokens per chunk
typedef short v4i16 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4i16 lds_tr16(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) v4i16*)(const __attribute__((address_space(3))) void*)p);
}
}  // namespace

template <bool BIG>
__device__ __forceinline__ void syrk_bf16_tile(const __bf16* __restrict__ X, int m, int d,
                                               double alpha, double* __restrict__ Hacc, int a0,
                                               int b0, char* buf0, char* buf1) {
  constexpr int TE = BIG ? 128 : 64;          // tile edge
  constexpr int RB = 2 * TE;                  // bytes per token
  constexpr int CPR = RB / 16;                // 16-byte pieces per token
  constexpr int RPP = 64 / CPR;               // tokens per load instruction (1 KB)
  constexpr int OP = BCH * RB;                // bytes of an operand's chunk
  constexpr int NP = BCH / RPP / 4;           // load instructions per wave and operand
  constexpr int AB = BIG ? 2 : 1;             // 32-wide blocks per wavefront, each way
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  // token t's 64-byte block x is stored at x ^ swz(t)
  auto swz = [](int t) { return BIG ? t & 3 : (t >> 1) & 1; };
  // staging: instruction i of a wave fills tokens RPP (wave + 4 i) ..; lane L
  // token L / CPR of those, piece L % CPR.  Channels past d (a multiple of 8)
  // read the last ones (their results are not stored).
  const int lt = lane / CPR;
  const int lpiece = (lane % CPR) ^ (swz(lt) << 2);
  const uint32_t row = 2u * (uint32_t)d;      // bytes per token of X
  // 32-bit byte offsets from the chunk's first token (64 tokens of 32768
  // channels are 4 MB)
  const uint32_t srow = (uint32_t)(RPP * wave + lt) * row;
  const uint32_t oa = 2u * (uint32_t)min(a0 + 8 * lpiece, d - 8);
  const uint32_t ob = 2u * (uint32_t)min(b0 + 8 * lpiece, d - 8);
  auto issue = [&](int t0, char* stage) {
    const char* base = (const char*)(X + (size_t)t0 * d);
    if (t0 + BCH <= m) {   // uniform
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const uint32_t at = srow + (uint32_t)(4 * RPP * i) * row;
        __builtin_amdgcn_global_load_lds(
            (const void*)(base + (at + oa)),
            (__attribute__((address_space(3))) void*)(stage + 1024 * (wave + 4 * i)), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(
            (const void*)(base + (at + ob)),
            (__attribute__((address_space(3))) void*)(stage + OP + 1024 * (wave + 4 * i)), 16, 0,
            0);
      }
    } else {               // the last chunk: tokens past m are 0
      const int left = m - t0;
#pragma unroll 1
      for (int i = 0; i < NP; ++i) {
        const int t = RPP * (wave + 4 * i) + lt;
        const uint32_t at = (uint32_t)min(t, left - 1) * row;
        u32x4 va = *(const u32x4*)(base + (at + oa)), vb = *(const u32x4*)(base + (at + ob));
        if (t >= left) va = vb = u32x4{};
        *(u32x4*)(stage + 1024 * (wave + 4 * i) + 16 * lane) = va;
        *(u32x4*)(stage + OP + 1024 * (wave + 4 * i) + 16 * lane) = vb;
      }
    }
  };
  // fragment reads: 16-lane group gi takes channels 16 (gi % 2) .. of the
  // block and tokens 8 (gi / 2) ..
  const int gi = lane >> 4, pi = lane & 15;
  const int ft = 8 * (gi >> 1) + (pi >> 2);
  const int fin = 32 * (gi & 1) + 8 * (pi & 3);   // byte within the 64-byte block
  int fa[AB], fb[AB];
#pragma unroll
  for (int a = 0; a < AB; ++a) {
    fa[a] = ft * RB + (((AB * wm + a) ^ swz(pi >> 2)) << 6) + fin;
    fb[a] = OP + ft * RB + (((AB * wn + a) ^ swz(pi >> 2)) << 6) + fin;
  }
  f32x16 acc[AB][AB];
  double sum[AB][AB][16];
#pragma unroll
  for (int a = 0; a < AB; ++a)
#pragma unroll
    for (int b = 0; b < AB; ++b) {
      acc[a][b] = f32x16{};
#pragma unroll
      for (int v = 0; v < 16; ++v) sum[a][b][v] = 0.0;
    }
  auto compute = [&](const char* cur) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < BCH / 16; ++ks) {
      bf16x8 xa[AB], xb[AB];
      auto frag = [&](const char* p) __attribute__((always_inline)) {
        const v4i16 w[2] = {lds_tr16(p), lds_tr16(p + 4 * RB)};
        return __builtin_bit_cast(bf16x8, w);
      };
#pragma unroll
      for (int a = 0; a < AB; ++a) {
        xa[a] = frag(cur + fa[a] + 16 * ks * RB);
        xb[a] = frag(cur + fb[a] + 16 * ks * RB);
      }
#pragma unroll
      for (int a = 0; a < AB; ++a)
#pragma unroll
        for (int b = 0; b < AB; ++b) acc[a][b] = mfma_bf16(xa[a], xb[b], acc[a][b]);
    }
  };
  auto flush = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < AB; ++a)
#pragma unroll
      for (int b = 0; b < AB; ++b) {
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[a][b][v] += (double)acc[a][b][v];
        acc[a][b] = f32x16{};
      }
  };
  static_assert(kSumTokens % (2 * BCH) == 0, "flushed at an even chunk");
  const int nch = (m + BCH - 1) / BCH;
  issue(0, buf0);
  __syncthreads();
  for (int q = 0; q < nch; q += 2) {
    // a stage was last read before the barrier that precedes its loads; the
    // barrier after a chunk waits for the next one's loads
    if (q + 1 < nch) issue((q + 1) * BCH, buf1);
    compute(buf0);
    __syncthreads();
    if (q + 1 < nch) {
      if (q + 2 < nch) issue((q + 2) * BCH, buf0);
      compute(buf1);
      __syncthreads();
    }
    if ((q + 2) % (kSumTokens / BCH) == 0) flush();
  }
  flush();
  // a part of its own for each wave (the stages are done with)
  double* out = (double*)(wave < 2 ? buf0 : buf1) + (wave & 1) * 32 * 33;
#pragma unroll
  for (int a = 0; a < AB; ++a)
#pragma unroll
    for (int b = 0; b < AB; ++b)
      add_block(Hacc, d, alpha, a0 + 32 * (AB * wm + a), b0 + 32 * (AB * wn + b), sum[a][b],
                       out);
}

// WHOLE: 128-wide tiles among them (their 128 registers of fp64 sums leave 228
// bytes a lane in scratch: in the epilogue, once a tile, but for one pair around
// each 256-token addition); otherwise 64-wide ones alone, whose stages leave room
// for four work-groups on a CU.
template <bool WHOLE>
__global__ __launch_bounds__(256, WHOLE ? 2 : 4) void syrk_bf16_kernel(
    const __bf16* __restrict__ X, int m, int d, double alpha, double* __restrict__ Hacc, Split s) {
  constexpr int STAGE = 2 * BCH * (WHOLE ? 256 : 128);     // bytes
  constexpr int OUT = 2 * 32 * 33 * sizeof(double);        // two wavefronts' blocks
  constexpr int BUF = STAGE > OUT ? STAGE : (OUT + 1023) / 1024 * 1024;
  // two arrays, so that the compiler can tell which one a load in flight writes
  __shared__ __attribute__((aligned(1024))) char buf0[BUF];
  __shared__ __attribute__((aligned(1024))) char buf1[BUF];
  int a0, b0;
  const Tile tile = tile_of<false>(blockIdx.x, s, a0, b0);   // uniform
  if constexpr (WHOLE) {
    if (tile == kWhole) {
      syrk_bf16_tile<true>(X, m, d, alpha, Hacc, a0, b0, buf0, buf1);
      return;
    }
  }
  if (a0 < d && b0 < d) syrk_bf16_tile<false>(X, m, d, alpha, Hacc, a0, b0, buf0, buf1);
}

// 64-wide tiles alone below 256 128-wide ones (each would have a CU to itself;
// 4096 tokens x 2048 channels, 120 of them: 46 us, whole 79, cut but with the
// stages of the whole ones 75; x 2816, 231 of them: 64, 81 and 81); beyond, the last
// round of 128-wide ones (512 at a time, two on a CU) is cut where it would leave
// more than half of the chip idle (x 6144, 104 left over: 320, whole 326; x 3072,
// 276 of them: 91, all cut 115).
hipError_t launch_hessian_update_bf16(hipStream_t st, const void* X, int m, int d, double alpha,
                                      double* Hacc) {
  Split s = split_of(d, true);
  const int last = s.big % 512;
  if (last < 256) cut_last(s, last, 4);
  if (s.big == 0)
    hipLaunchKernelGGL(syrk_bf16_kernel<false>, dim3(s.small), dim3(256), 0, st, (const __bf16*)X,
                       m, d, alpha, Hacc, s);
  else
    hipLaunchKernelGGL(syrk_bf16_kernel<true>, dim3(s.big + s.small), dim3(256), 0, st,
                       (const __bf16*)X, m, d, alpha, Hacc, s);
  return hipGetLastError();
}

// ---- fp32 inputs ----
// 512 threads.  128 x 128: 2 x 4 wavefronts of 64 x 32, chunks of 32 tokens;
// 128 x 64: 4 x 2 wavefronts of 32 x 32, the same chunks; 64 x 64: 2 x 2 wavefronts
// of 32 x 32 twice, chunks of 64 tokens, the second four wavefronts taking the odd
// k-slices (their sums are added to the first four's at the end).  A thread
// stages 8 tokens x 2 channels and converts them to the planes; two LDS stages
// of three planes; one work-group per CU.  The planes lie channel-major (a row per
// channel, tokens along it), so a fragment (32 channels x 16 tokens) is one
// 16-byte read a lane; rows are padded by 16 bytes, which puts the 16 rows of a
// read, and the 16 chunks of a write, in distinct banks.
//
// The tile's sums with the fp32 instruction straight from memory (one wave,
// blocks of 32 x 32): for the tiles the three planes cannot do.
template <bool CROSS>
__device__ __forceinline__ void syrk_f32_slow(const float* __restrict__ Xq,
                                              const float* __restrict__ X, int m, int d, int a0,
                                              int b0, double (&sum)[16]) {
  const int lane = threadIdx.x & 63, lm = lane & 31, kh = lane >> 5;
  const bool ia = a0 + lm < d, ib = b0 + lm < d;
  const size_t ca = ia ? a0 + lm : 0, cb = ib ? b0 + lm : 0;
#pragma unroll
  for (int v = 0; v < 16; ++v) sum[v] = 0.0;
  for (int t0 = 0, t1; t0 < m; t0 = t1) {
    f32x16 acc = f32x16{};
    t1 = span_end(t0, m);
    for (int t = t0; t < t1; t += 2) {
      const bool it = t + kh < m;
      const size_t r = (size_t)(it ? t + kh : m - 1) * d;
      float fa = Xq[r + ca], fb = Xq[r + cb];
      if (CROSS) fb = X[r + cb] - fb;
      fa = it && ia ? fa : 0.f;
      fb = it && ib ? fb : 0.f;
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa, fb, acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[v] += (double)acc[v];
  }
}

template <bool CROSS, int TA, int TB>
__device__ __forceinline__ void syrk_f32_tile(const float* __restrict__ Xq,
                                              const float* __restrict__ X, int m, int d,
                                              double alpha, double* __restrict__ Hacc, int a0,
                                              int b0, char* smem) {
  constexpr bool TWICE = TA == 64;            // eight wavefronts on four blocks
  constexpr int CH = TWICE ? 64 : 32;         // tokens per chunk
  constexpr int LD = 2 * CH + 16;             // row stride in bytes
  constexpr int PLANE = (TA + TB) * LD;       // A rows, then B rows
  constexpr int STAGE = 3 * PLANE;
  constexpr int WN = TB / 32;                 // wavefronts along the columns
  constexpr int AB = TA * TB == 128 * 128 ? 2 : 1;   // 32-row blocks per wavefront
  constexpr int FLUSH = kSumTokens / CH;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN % (TA / (32 * AB)), wn = wave % WN;
  const int wk = TWICE ? wave >> 2 : 0;       // first k-slice (64 x 64: every second one)
  const int lm = lane & 31, kh = lane >> 5;
  // staging: 8 tokens at 8 tg, 2 channels from tile row r2
  constexpr int TGB = TWICE ? 2 : 1;          // token-group bits taken from the wave
  const int tg = (lane & 1) + 2 * (wave & ((1 << TGB) - 1));
  const int r2 = 64 * (wave >> TGB) + 2 * (lane >> 1);
  // (128 x 64: six wavefronts stage; uniform in a wave, as is_b)
  const bool stages = TA == TB || r2 < TA + TB;
  const bool is_b = r2 >= TA;
  const int ch = is_b ? b0 + r2 - TA : a0 + r2;
  const bool in_ch = ch < d;                  // d is even
  // 32-bit byte offsets from the chunk's first token
  const uint32_t row = 4u * (uint32_t)d, c4 = 4u * (uint32_t)(in_ch ? ch : 0);
  // raw values: they are first touched when they are stored, a chunk later
  float2 st[8], sx[CROSS ? 8 : 1];
  auto load = [&](int t0) {
    if (!stages) return;
    const int last = m - 1 - t0;   // tokens past m read the last one
    const char* bq = (const char*)(Xq + (size_t)t0 * d);
    const char* bx = (const char*)(X + (size_t)t0 * d);
    const bool full = t0 + CH <= m;   // uniform
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t at = c4 + (uint32_t)(full ? 8 * tg + i : min(8 * tg + i, last)) * row;
      st[i] = *(const float2*)(bq + at);
      if constexpr (CROSS) {
        if (is_b) sx[i] = *(const float2*)(bx + at);   // uniform in a wave
      }
    }
  };
  auto store = [&](int t0, char* stage) {
    if (!stages) return;
    if constexpr (CROSS) {
      if (is_b) {
#pragma unroll
        for (int i = 0; i < 8; ++i) st[i] = make_float2(sx[i].x - st[i].x, sx[i].y - st[i].y);
      }
    }
    if (t0 + CH > m || !in_ch) {   // tokens past m and channels past d are 0
      const int left = in_ch ? m - t0 - 8 * tg : 0;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (i >= left) st[i] = make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      u32x4 h, mm, l;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        uint32_t wh, wm_, wl;
        split_pair(c ? st[2 * p].y : st[2 * p].x, c ? st[2 * p + 1].y : st[2 * p + 1].x, wh, wm_, wl);
        h[p] = wh;
        mm[p] = wm_;
        l[p] = wl;
      }
      char* at = stage + (r2 + c) * LD + 16 * tg;
      *(u32x4*)at = h;
      *(u32x4*)(at + PLANE) = mm;
      *(u32x4*)(at + 2 * PLANE) = l;
    }
  };
  f32x16 acc[AB], low[AB];
  double sum[AB][16];
#pragma unroll
  for (int a = 0; a < AB; ++a) {
    acc[a] = low[a] = f32x16{};
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[a][v] = 0.0;
  }
  auto flush = [&]() {
#pragma unroll
    for (int a = 0; a < AB; ++a) {
#pragma unroll
      for (int v = 0; v < 16; ++v) sum[a][v] += (double)(acc[a][v] + low[a][v]);
      acc[a] = low[a] = f32x16{};
    }
  };
  const int nch = (m + CH - 1) / CH;
  load(0);
  store(0, smem);
  __syncthreads();
  for (int q = 0; q < nch; ++q) {
    const char* cur = smem + (q & 1) * STAGE;
    if (q + 1 < nch) load((q + 1) * CH);   // in flight during this chunk
    const char* ra = cur + (wm * 32 * AB + lm) * LD + 16 * kh;
    const char* rb = cur + (TA + wn * 32 + lm) * LD + 16 * kh;
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      const int ks = TWICE ? 2 * k2 + wk : k2;
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
    if ((q + 1) % FLUSH == 0) flush();
    // the other stage was last read before the barrier that ended chunk q - 1
    if (q + 1 < nch) store((q + 1) * CH, smem + ((q + 1) & 1) * STAGE);
    __syncthreads();
  }
  flush();
  if (TWICE) {
    // the second four wavefronts hand their sums to the first four
    double* red = (double*)smem + (wave & 3) * 1024;
    if (wk == 1) {
#pragma unroll
      for (int v = 0; v < 16; ++v) red[64 * v + lane] = sum[0][v];
    }
    __syncthreads();
    if (wk == 1) return;
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[0][v] += red[64 * v + lane];
  }
  // a part of its own for each wave, apart from the sums above
  double* buf = (double*)smem + (TWICE ? 4096 + (wave & 3) * 32 * 33 : wave * 32 * 33);
#pragma unroll
  for (int a = 0; a < AB; ++a) {
    const int ba = a0 + 32 * (AB * wm + a), bb = b0 + 32 * wn;
    bool fine = true;
#pragma unroll
    for (int v = 0; v < 16; ++v) fine &= isfinite(sum[a][v]);
    if (!__all(fine)) syrk_f32_slow<CROSS>(Xq, X, m, d, ba, bb, sum[a]);
    if (!CROSS) add_block(Hacc, d, alpha, ba, bb, sum[a], buf);
  }
  if constexpr (CROSS) add_blocks<AB>(Hacc, d, alpha, a0 + 32 * AB * wm, b0 + 32 * wn, sum);
}

// HALVES: 128 x 64 tiles among them (an instance of its own: their code in the
// other one costs its whole tiles 2 % by the registers they get).
template <bool CROSS, bool HALVES>
__global__ __launch_bounds__(512, 1) void syrk_f32_kernel(const float* __restrict__ Xq,
                                                          const float* __restrict__ X, int m,
                                                          int d, double alpha,
                                                          double* __restrict__ Hacc, Split s) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int a0, b0;
  const Tile tile = tile_of<CROSS>(blockIdx.x, s, a0, b0);   // uniform
  if (tile == kWhole) {
    syrk_f32_tile<CROSS, 128, 128>(Xq, X, m, d, alpha, Hacc, a0, b0, smem);
  } else if (a0 < d && b0 < d) {
    if constexpr (HALVES) {
      if (tile == kHalf) {
        syrk_f32_tile<CROSS, 128, 64>(Xq, X, m, d, alpha, Hacc, a0, b0, smem);
        return;
      }
    }
    syrk_f32_tile<CROSS, 64, 64>(Xq, X, m, d, alpha, Hacc, a0, b0, smem);
  }
}

template <bool CROSS, bool HALVES>
static hipError_t launch_syrk_f32_split(hipStream_t st, const float* Xq, const float* X, int m,
                                        int d, double alpha, double* Hacc, const Split& s) {
  // whole: 2 stages x 3 planes x 256 rows of 80 bytes; quarter: 128 rows of 144
  constexpr size_t lds = 2 * 3 * 256 * 80;
  static_assert(lds >= 2 * 3 * 128 * 144 && lds >= (4096 + 4 * 32 * 33) * sizeof(double), "LDS");
  static std::atomic<unsigned long long> lds_set{0};
  const hipError_t e = allow_dynamic_lds((const void*)syrk_f32_kernel<CROSS, HALVES>, lds, lds_set);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((syrk_f32_kernel<CROSS, HALVES>), dim3(s.big + s.small), dim3(512), lds, st,
                     Xq, X, m, d, alpha, Hacc, s);
  return hipGetLastError();
}

template <bool CROSS>
static hipError_t launch_syrk_f32(hipStream_t st, const float* Xq, const float* X, int m, int d,
                                  double alpha, double* Hacc) {
  // The last round of whole tiles (256 at a time, one on a CU) whole, in halves or
  // in quarters, whichever takes the least time together with the diagonal's
  // quarters: a round of whole tiles takes 2.2 times, one of halves 1.7 times as
  // long as one of quarters (4096 tokens: 221, 168 and 98 us; cross term 262, 202 and
  // 127).  66 whole tiles (1536 channels) 220, 168 and 197 us, 120 of them (2048) 221 in
  // one round, 293 in three of quarters, 20 left over (3072) 446 whole and 328.
  Split s = split_of(d, !CROSS);
  const int last = s.big % 256;
  auto rounds = [&](int parts) { return (parts * last + s.small + 255) / 256; };
  const double whole = 2.2, half = 1.7 * rounds(2), quarter = rounds(4);
  if (quarter <= half && quarter < whole)
    cut_last(s, last, 4);
  else if (half < whole)
    cut_last(s, last, 2);
  if (s.parts == 2) return launch_syrk_f32_split<CROSS, true>(st, Xq, X, m, d, alpha, Hacc, s);
  return launch_syrk_f32_split<CROSS, false>(st, Xq, X, m, d, alpha, Hacc, s);
}

hipError_t launch_hessian_update(hipStream_t st, const float* X, int m, int d, double alpha,
                                 double* Hacc) {
  return launch_syrk_f32<false>(st, X, X, m, d, alpha, Hacc);
}

hipError_t launch_cross_update(hipStream_t st, const float* Xq, const float* X, int m, int d,
                               double alpha, double* Dacc) {
  return launch_syrk_f32<true>(st, Xq, X, m, d, alpha, Dacc);
}

}  // namespace jarq
