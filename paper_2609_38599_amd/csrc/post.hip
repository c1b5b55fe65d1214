// After refinement: negative-scale canonicalization (App. E.3), dequantized
// weights in a floating-point dtype, packed b-bit codes, and the activation
// ordering a GPTQ host may use (refinement keeps its groups in the reordered
// coordinates and the weights return to the original ones on write-back,
// App. A.1 and App. E.2).
#include "jarq_internal.h"

namespace jarq {

namespace {
unsigned grid_of(long long n) {
  const long long b = (n + 255) / 256;
  return (unsigned)(b < 16384 ? b : 16384);
}
}  // namespace

// eq. (canonicalization): for s < 0, s' = -s, q' = qmax - q, z' = qmax - z,
// which represents the same weights.  One thread per group; few scales are
// negative, so a launch lasts as long as one group's code update, whose
// 16-byte loads all go out together (8 us for 11008 x 4096 with one scale in
// fifty negative; word by word, each load behind the last store, 17).
template <int g>
__global__ __launch_bounds__(256) void canonicalize_kernel(int rows, int cols, int bits,
                                                           uint8_t* __restrict__ codes,
                                                           float* __restrict__ scales,
                                                           int32_t* __restrict__ zeros) {
  const int G = cols / g;
  const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= (long long)rows * G) return;
  const float s = scales[e];
  if (!(s < 0.f)) return;
  const int qmax = (1 << bits) - 1;
  const long long row = e / G, grp = e % G;
  uint8_t* q = codes + row * cols + grp * g;
  uint4 v[g / 16];
#pragma unroll
  for (int c = 0; c < g / 16; ++c) v[c] = *(const uint4*)(q + 16 * c);
  // byte by byte modulo 256, as (qmax - q) & 0xff of any code
  auto flip = [&](uint32_t w) {
    uint32_t out = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) out |= (uint32_t)((qmax - (int)((w >> (8 * i)) & 0xFF)) & 0xFF) << (8 * i);
    return out;
  };
#pragma unroll
  for (int c = 0; c < g / 16; ++c)
    *(uint4*)(q + 16 * c) = make_uint4(flip(v[c].x), flip(v[c].y), flip(v[c].z), flip(v[c].w));
  scales[e] = -s;
  zeros[e] = qmax - zeros[e];
}

hipError_t launch_canonicalize(hipStream_t st, int rows, int cols, int g, int bits,
                               uint8_t* codes, float* scales, int32_t* zeros) {
  const long long n = (long long)rows * (cols / g);
  const dim3 grid((unsigned)((n + 255) / 256));
  switch (g) {
    case 32: hipLaunchKernelGGL(canonicalize_kernel<32>, grid, dim3(256), 0, st, rows, cols, bits, codes, scales, zeros); break;
    case 64: hipLaunchKernelGGL(canonicalize_kernel<64>, grid, dim3(256), 0, st, rows, cols, bits, codes, scales, zeros); break;
    case 128: hipLaunchKernelGGL(canonicalize_kernel<128>, grid, dim3(256), 0, st, rows, cols, bits, codes, scales, zeros); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Round-to-nearest-even fp32 -> bf16 bits (NaN kept quiet).
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float x) {
  const uint32_t u = __float_as_uint(x);
  if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (uint16_t)((u >> 16) | 0x40);
  const uint32_t r = u + 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(r >> 16);
}

__device__ __forceinline__ void to_dtype(float v, float& o) { o = v; }
__device__ __forceinline__ void to_dtype(float v, _Float16& o) { o = (_Float16)v; }
__device__ __forceinline__ void to_dtype(float v, uint16_t& o) { o = f32_to_bf16_bits(v); }

// Sixteen weights s (q - z) of one group from its codes.
template <typename T>
__device__ __forceinline__ void dequant16(const uint4& q, float s, int z, T (&o)[16]) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int i = 0; i < 16; ++i)
    to_dtype(s * (float)((int)((w[i >> 2] >> (8 * (i & 3))) & 0xFFu) - z), o[i]);
}

// out[r][c] = s (q - z) in fp32, rounded once to the output dtype: sixteen
// weights of a group per thread and step (16-byte aligned codes and out).
// Bound by memory traffic.
template <typename T>
__global__ __launch_bounds__(256) void dequantize_kernel(long long pieces, int g,
                                                         const uint8_t* __restrict__ codes,
                                                         const float* __restrict__ scales,
                                                         const int32_t* __restrict__ zeros,
                                                         T* __restrict__ out) {
  const int sh = __ffs(g) - 5;   // g / 16 pieces a group, a power of two
  for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < pieces;
       e += (long long)gridDim.x * 256) {
    const long long sg = e >> sh;
    __attribute__((aligned(16))) T o[16];
    dequant16(*(const uint4*)(codes + 16 * e), scales[sg], zeros[sg], o);
#pragma unroll
    for (int i = 0; i < (int)sizeof(T); ++i) ((uint4*)(out + 16 * e))[i] = ((const uint4*)o)[i];
  }
}

// The same with a permutation: position k of the refined layer is original
// column perm[k] (entries outside [0, cols) are skipped, columns no entry names
// are left alone).  A work-group inverts the permutation into LDS once, then
// takes rows in turn: the row's weights in the refined order go to LDS, and
// the output is written along the row, gathered from there.  (Scattering
// each weight to its column wrote two bytes at a time: 199 us for
// 11008 x 4096 in bf16, now 42, 3.2 TB/s.)
template <typename T>
__global__ __launch_bounds__(512) void dequantize_perm_kernel(int rows, int cols, int g,
                                                              const uint8_t* __restrict__ codes,
                                                              const float* __restrict__ scales,
                                                              const int32_t* __restrict__ zeros,
                                                              const int32_t* __restrict__ perm,
                                                              T* __restrict__ out) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  uint16_t* inv = (uint16_t*)smem;                 // [cols], 0xffff = no position
  T* w_s = (T*)(smem + 2 * (size_t)cols);          // [cols]
  const int G = cols / g;
  for (int c = threadIdx.x; c < cols; c += 512) inv[c] = 0xffffu;
  __syncthreads();
  for (int k = threadIdx.x; k < cols; k += 512) {
    const int c = perm[k];
    if (c >= 0 && c < cols) inv[c] = (uint16_t)k;
  }
  for (int r = blockIdx.x; r < rows; r += gridDim.x) {
    __syncthreads();   // inv, or the previous row's reads of w_s
    for (int p = threadIdx.x; p < cols / 16; p += 512) {
      const long long sg = (long long)r * G + 16 * p / g;
      __attribute__((aligned(16))) T o[16];
      dequant16(*(const uint4*)(codes + (size_t)r * cols + 16 * p), scales[sg], zeros[sg], o);
#pragma unroll
      for (int i = 0; i < (int)sizeof(T); ++i) ((uint4*)(w_s + 16 * p))[i] = ((const uint4*)o)[i];
    }
    __syncthreads();
    T* dst = out + (size_t)r * cols;
    for (int p = threadIdx.x; p < cols / 8; p += 512) {
      const uint4 kv = *(const uint4*)(inv + 8 * p);
      const uint32_t kw[4] = {kv.x, kv.y, kv.z, kv.w};
      __attribute__((aligned(16))) T o[8];
      bool all = true;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t k = (kw[i >> 1] >> (16 * (i & 1))) & 0xffffu;
        all &= k != 0xffffu;
        o[i] = w_s[k == 0xffffu ? 0 : k];
      }
      if (all) {
#pragma unroll
        for (int i = 0; i < (int)sizeof(T) / 2; ++i) ((uint4*)(dst + 8 * p))[i] = ((const uint4*)o)[i];
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (((kw[i >> 1] >> (16 * (i & 1))) & 0xffffu) != 0xffffu) dst[8 * p + i] = o[i];
      }
    }
  }
}

// Either form for pointers without 16-byte alignment, and the permuted one for
// few rows, a weight per thread and step.
__global__ __launch_bounds__(256) void dequantize_any_kernel(int rows, int cols, int g,
                                                             const uint8_t* __restrict__ codes,
                                                             const float* __restrict__ scales,
                                                             const int32_t* __restrict__ zeros,
                                                             const int32_t* __restrict__ perm,
                                                             int dtype, void* __restrict__ out) {
  const long long n = (long long)rows * cols;
  const int G = cols / g;
  for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < n;
       e += (long long)gridDim.x * 256) {
    const long long r = e / cols;
    const int k = (int)(e % cols);
    const long long sg = r * G + k / g;
    const float v = scales[sg] * (float)((int)codes[e] - zeros[sg]);
    long long dst = e;
    if (perm != nullptr) {
      const int c = perm[k];
      if (c < 0 || c >= cols) continue;
      dst = r * cols + c;
    }
    if (dtype == 0)
      ((float*)out)[dst] = v;
    else if (dtype == 1)
      ((_Float16*)out)[dst] = (_Float16)v;
    else
      ((uint16_t*)out)[dst] = f32_to_bf16_bits(v);
  }
}

template <typename T>
static hipError_t launch_dequantize_t(hipStream_t st, int rows, int cols, int g,
                                      const uint8_t* codes, const float* scales,
                                      const int32_t* zeros, const int32_t* perm, T* out) {
  if (perm == nullptr) {
    const long long pieces = (long long)rows * (cols / 16);
    hipLaunchKernelGGL(dequantize_kernel<T>, dim3(grid_of(pieces)), dim3(256), 0, st, pieces, g,
                       codes, scales, zeros, out);
    return hipGetLastError();
  }
  const size_t lds = (size_t)cols * (2 + sizeof(T));
  static std::atomic<unsigned long long> lds_set{0};
  // the most a layer can have: 16384 columns
  const hipError_t e = allow_dynamic_lds((const void*)dequantize_perm_kernel<T>,
                                         16384 * (2 + sizeof(T)), lds_set);
  if (e != hipSuccess) return e;
  // four work-groups (all 32 wavefronts) a CU where LDS allows, rows in turn
  hipLaunchKernelGGL(dequantize_perm_kernel<T>, dim3(rows < 1024 ? rows : 1024), dim3(512), lds,
                     st, rows, cols, g, codes, scales, zeros, perm, out);
  return hipGetLastError();
}

hipError_t launch_dequantize(hipStream_t st, int rows, int cols, int g, const uint8_t* codes,
                             const float* scales, const int32_t* zeros, const int32_t* perm,
                             int dtype, void* out) {
  // Up to 64 rows the permuted form scatters its weights: a work-group a row, each
  // inverting the permutation first, leaves most of the chip idle (16 x 11008 in
  // bf16: 3.8 and 8.3 us; at 64 rows of 4096, 8192 and 16384 columns 4.2, 5.7, 9.2
  // and 4.7, 6.5, 10.8; at 128 rows 5.4, 9.0, 14.4 and 4.7, 6.8, 11.0).
  const bool few = perm != nullptr && rows <= 64;
  if (few || (((uintptr_t)codes | (uintptr_t)out) & 15) != 0) {
    hipLaunchKernelGGL(dequantize_any_kernel, dim3(grid_of((long long)rows * cols)), dim3(256), 0,
                       st, rows, cols, g, codes, scales, zeros, perm, dtype, out);
    return hipGetLastError();
  }
  if (dtype == 0)
    return launch_dequantize_t(st, rows, cols, g, codes, scales, zeros, perm, (float*)out);
  if (dtype == 1)
    return launch_dequantize_t(st, rows, cols, g, codes, scales, zeros, perm, (_Float16*)out);
  return launch_dequantize_t(st, rows, cols, g, codes, scales, zeros, perm, (uint16_t*)out);
}

// Row r's codes as one little-endian bit stream: code k occupies stream bits
// [k b, k b + b), stream bit t is bit t % 32 of word t / 32 of the row, rows
// start on a word boundary (cols is a multiple of 32, so a row is cols b / 32
// whole words).  A thread takes 32 codes, which are b words: 16-byte accesses
// to the codes where they are aligned, byte accesses otherwise.
template <int B, bool ALIGNED>
__global__ __launch_bounds__(256) void pack_kernel(long long pieces,
                                                   const uint8_t* __restrict__ codes,
                                                   uint32_t* __restrict__ packed) {
  for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < pieces;
       e += (long long)gridDim.x * 256) {
    uint32_t q[8];
    if (ALIGNED) {
      const uint4 a = ((const uint4*)(codes + 32 * e))[0], b = ((const uint4*)(codes + 32 * e))[1];
      q[0] = a.x, q[1] = a.y, q[2] = a.z, q[3] = a.w;
      q[4] = b.x, q[5] = b.y, q[6] = b.z, q[7] = b.w;
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        q[i] = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) q[i] |= (uint32_t)codes[32 * e + 4 * i + u] << (8 * u);
      }
    }
    uint32_t w[B];
#pragma unroll
    for (int i = 0; i < B; ++i) w[i] = 0;
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const uint32_t c = (q[k >> 2] >> (8 * (k & 3))) & ((1u << B) - 1u);
      const int t = k * B;
      w[t / 32] |= c << (t % 32);
      if (t % 32 + B > 32) w[t / 32 + 1] |= c >> (32 - t % 32);
    }
#pragma unroll
    for (int i = 0; i < B; ++i) packed[(long long)B * e + i] = w[i];
  }
}

template <int B, bool ALIGNED>
__global__ __launch_bounds__(256) void unpack_kernel(long long pieces,
                                                     const uint32_t* __restrict__ packed,
                                                     uint8_t* __restrict__ codes) {
  for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < pieces;
       e += (long long)gridDim.x * 256) {
    uint32_t w[B + 1];
#pragma unroll
    for (int i = 0; i < B; ++i) w[i] = packed[(long long)B * e + i];
    w[B] = 0;
    uint32_t q[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) q[i] = 0;
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const int t = k * B;
      uint32_t c = w[t / 32] >> (t % 32);
      if (t % 32 + B > 32) c |= w[t / 32 + 1] << (32 - t % 32);
      q[k >> 2] |= (c & ((1u << B) - 1u)) << (8 * (k & 3));
    }
    if (ALIGNED) {
      ((uint4*)(codes + 32 * e))[0] = make_uint4(q[0], q[1], q[2], q[3]);
      ((uint4*)(codes + 32 * e))[1] = make_uint4(q[4], q[5], q[6], q[7]);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int u = 0; u < 4; ++u) codes[32 * e + 4 * i + u] = (uint8_t)(q[i] >> (8 * u));
    }
  }
}

template <int B>
static hipError_t launch_pack_t(hipStream_t st, long long pieces, const uint8_t* codes,
                                uint32_t* packed) {
  if (((uintptr_t)codes & 15) == 0)
    hipLaunchKernelGGL((pack_kernel<B, true>), dim3(grid_of(pieces)), dim3(256), 0, st, pieces, codes, packed);
  else
    hipLaunchKernelGGL((pack_kernel<B, false>), dim3(grid_of(pieces)), dim3(256), 0, st, pieces, codes, packed);
  return hipGetLastError();
}
template <int B>
static hipError_t launch_unpack_t(hipStream_t st, long long pieces, const uint32_t* packed,
                                  uint8_t* codes) {
  if (((uintptr_t)codes & 15) == 0)
    hipLaunchKernelGGL((unpack_kernel<B, true>), dim3(grid_of(pieces)), dim3(256), 0, st, pieces, packed, codes);
  else
    hipLaunchKernelGGL((unpack_kernel<B, false>), dim3(grid_of(pieces)), dim3(256), 0, st, pieces, packed, codes);
  return hipGetLastError();
}

hipError_t launch_pack(hipStream_t st, int rows, int cols, int bits, const uint8_t* codes,
                       uint32_t* packed) {
  const long long pieces = (long long)rows * (cols / 32);
  switch (bits) {
    case 1: return launch_pack_t<1>(st, pieces, codes, packed);
    case 2: return launch_pack_t<2>(st, pieces, codes, packed);
    case 3: return launch_pack_t<3>(st, pieces, codes, packed);
    case 4: return launch_pack_t<4>(st, pieces, codes, packed);
    case 5: return launch_pack_t<5>(st, pieces, codes, packed);
    case 6: return launch_pack_t<6>(st, pieces, codes, packed);
    case 7: return launch_pack_t<7>(st, pieces, codes, packed);
    case 8: return launch_pack_t<8>(st, pieces, codes, packed);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_unpack(hipStream_t st, int rows, int cols, int bits, const uint32_t* packed,
                         uint8_t* codes) {
  const long long pieces = (long long)rows * (cols / 32);
  switch (bits) {
    case 1: return launch_unpack_t<1>(st, pieces, packed, codes);
    case 2: return launch_unpack_t<2>(st, pieces, packed, codes);
    case 3: return launch_unpack_t<3>(st, pieces, packed, codes);
    case 4: return launch_unpack_t<4>(st, pieces, packed, codes);
    case 5: return launch_unpack_t<5>(st, pieces, packed, codes);
    case 6: return launch_unpack_t<6>(st, pieces, packed, codes);
    case 7: return launch_unpack_t<7>(st, pieces, packed, codes);
    case 8: return launch_unpack_t<8>(st, pieces, packed, codes);
    default: return hipErrorInvalidValue;
  }
}

// Activation ordering: channels by decreasing diag(H), ties by increasing
// index (a stable sort): rank(i) = #{j : h_j > h_i or (h_j == h_i and j < i)},
// perm[rank(i)] = i.  Sixteen channels per work-group, sixteen threads each
// counting every sixteenth j; the diagonal is staged in LDS in pieces of 4096.
// (One thread per channel against the whole diagonal ran on d / 256
// work-groups and 256 strided loads at a time: 204 us at 2752 channels, now
// 20.)
constexpr int kActChunk = 4096;
__global__ __launch_bounds__(256) void act_order_kernel(const float* __restrict__ H, int d,
                                                        int32_t* __restrict__ perm) {
  __shared__ float hs[kActChunk];
  const int part = threadIdx.x & 15;
  const int i = blockIdx.x * 16 + (threadIdx.x >> 4);
  const float hi = i < d ? H[(long long)i * d + i] : 0.f;
  int rank = 0;
  for (int j0 = 0; j0 < d; j0 += kActChunk) {
    const int nj = min(kActChunk, d - j0);
    __syncthreads();
    for (int t0 = threadIdx.x; t0 < nj; t0 += 8 * 256) {
      float v[8];   // eight strided loads in flight
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int j = j0 + min(t0 + 256 * u, nj - 1);
        v[u] = H[(long long)j * d + j];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (t0 + 256 * u < nj) hs[t0 + 256 * u] = v[u];
    }
    __syncthreads();
    for (int t = part; t < nj; t += 16) {
      const float hj = hs[t];
      rank += (hj > hi || (hj == hi && j0 + t < i)) ? 1 : 0;
    }
  }
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) rank += __shfl_xor(rank, off);
  if (i < d && part == 0) perm[rank] = i;
}

hipError_t launch_act_order(hipStream_t st, const float* H, int d, int32_t* perm) {
  hipLaunchKernelGGL(act_order_kernel, dim3((d + 15) / 16), dim3(256), 0, st, H, d, perm);
  return hipGetLastError();
}

// Wp[r][k] = W[r][perm[k]], Hp[k][l] = H[perm[k]][perm[l]] (0 where an entry of
// perm is outside [0, d)).
// One work-group per output row: the source row is read along itself into LDS
// and gathered from there.
__global__ __launch_bounds__(256) void permute_kernel(int rows, int d,
                                                      const int32_t* __restrict__ perm,
                                                      const float* __restrict__ W,
                                                      const float* __restrict__ H,
                                                      float* __restrict__ Wp,
                                                      float* __restrict__ Hp) {
  extern __shared__ float row_s[];
  const bool is_w = (int)blockIdx.x < rows;
  const long long r = is_w ? blockIdx.x : blockIdx.x - rows;
  const int from = is_w ? 0 : perm[r];
  const bool live = is_w || (from >= 0 && from < d);
  const float* src = is_w ? W + r * d : H + (long long)(live ? from : 0) * d;
  float* dst = (is_w ? Wp : Hp) + r * d;
  for (int k = threadIdx.x; k < d; k += 256) row_s[k] = src[k];
  __syncthreads();
  for (int k = threadIdx.x; k < d; k += 256) {
    const int c = perm[k];
    dst[k] = live && c >= 0 && c < d ? row_s[c] : 0.f;
  }
}

hipError_t launch_permute(hipStream_t st, int rows, int d, const int32_t* perm, const float* W,
                          const float* H, float* Wp, float* Hp) {
  static std::atomic<unsigned long long> lds_set{0};
  // the most a layer can have: 16384 columns
  const hipError_t e = allow_dynamic_lds((const void*)permute_kernel, 16384 * sizeof(float), lds_set);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(permute_kernel, dim3(rows + d), dim3(256), (size_t)d * sizeof(float), st, rows,
                     d, perm, W, H, Wp, Hp);
  return hipGetLastError();
}

}  // namespace jarq
