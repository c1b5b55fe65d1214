// Joint scale solve of the scale update (paper eq. (6), App. E.2), in fp64.
//
// The G x G Gram matrix (upper triangle from the Gram kernel, symmetrised by
// construction) and the right-hand side r_a = c_a^T (W H)_a are factored by a
// right-looking Cholesky, one wavefront per row of the layer, in panels of 16
// columns: the 16 x 16 blocks of the lower triangle sit in registers in the
// layout of v_mfma_f64_16x16x4_f64's result, a panel goes through LDS to one
// row of the system per lane (two for G > 64), its columns are eliminated
// there, and the blocks right of it are updated on the fp64 matrix cores.
// Bound by the chain of columns and, beside it, the fp64 units; 32 to 128
// systems of a sweep's rows a CU hide it.  14336 rows of G = 64: 226 us (the
// matrix in 4 x 4 register tiles spread over the lanes, updated on the vector
// units: 551); 4096 rows of G = 32: 28 us (a row per lane: 33), of G = 88: 211 (411),
// of G = 128 0.88 ms (in LDS, two wavefronts a row: 7.0).  For G > 80 the blocks
// do not all fit: T = 6, 7 and 8 keep 16, 200 and 560 bytes a lane in scratch.
// The stabilised branch of
// App. E.2 (add lambda I and factor again) is taken when an entry is not
// finite, a pivot is not positive, the smallest pivot is at most
// r_cond * max(largest diagonal, 2^-23), or the smallest eigenvalue is at
// most t = r_cond * max(||A||_F, 2^-23).  Every Cholesky pivot is a Schur
// complement and bounded below by the smallest eigenvalue, and the largest
// diagonal bounds the largest eigenvalue from below, so the pivot test only
// fires where the paper's eigenvalue test fires; it can miss a nearly
// singular matrix whose pivots all stay large, which the last test catches.
// ||A||_F bounds the largest eigenvalue from above, so the last test fires
// wherever the paper's does, and beyond it only where the smallest
// eigenvalue lies in (r_cond lambda_max, t].  It is settled cheaply where it
// clearly does not fire: with L's comparison matrix C (|diagonal|, minus
// |off-diagonal|), C^{-1} >= |L^{-1}| entrywise, so x = C^{-1} 1 (solved
// beside the forward substitution) gives ||L^{-1}||_inf <= max x and
// lambda_min = 1 / ||L^{-1}||_2^2 >= 1 / (G (max x)^2).  Only where that
// bound is not above t is A - t I factored: it is positive definite exactly
// when lambda_min > t.  A second failure after lambda I leaves the row's
// scales unchanged and is counted.
#include "chol64.h"

namespace jarq {

// Right-hand sides of the scale systems, r_i = c_i^T (W H)_i for group i of a
// row (eq. (6)), in fp64.  They depend on the row's codes of group i only, so
// the sweep keeps them in `cache` ([layer rows][G]): the first scale solve of
// a run (ctl->valid == 0, or no ctl) forms them from W H and the codes and
// stores them; later ones read them, the code update having added
// d^T (W H)_i for every change d it made since.
struct RhsSrc {
  const float* wh;
  const uint8_t* codes;
  const int32_t* zeros;
  double* cache;
  const GramCtl* ctl;
};

// The right-hand sides of layer row grow into out[0 .. G) (LDS), by one
// wavefront: g / 8 lanes a group, so that its reads are whole cache lines (a
// lane per group: 25 us more at 4096 x 11008, g = 128).
__device__ __forceinline__ void rhs_form(const RhsSrc& rs, int grow, int cols, int g, int G,
                                         double* out) {
  const int lane = threadIdx.x;
  const int lpg = g >> 3, per = 64 / lpg, sub = lane / lpg;   // lpg = 4, 8 or 16
  const size_t at = (size_t)grow * cols + 8 * (lane % lpg);
  for (int i0 = 0; i0 < G; i0 += 4 * per) {   // four groups' loads in flight a lane
    uint2 qv[4];
    f32x4 wv[4][2];
    int zv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = min(i0 + u * per + sub, G - 1);
      const size_t e = at + (size_t)i * g;
      qv[u] = *(const uint2*)(rs.codes + e);
      wv[u][0] = *(const f32x4*)(rs.wh + e);
      wv[u][1] = *(const f32x4*)(rs.wh + e + 4);
      zv[u] = rs.zeros[(size_t)grow * G + i];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      double r = 0.0;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int q = (int)(((k < 4 ? qv[u].x : qv[u].y) >> (8 * (k & 3))) & 0xffu);
        r = fma((double)(q - zv[u]), (double)wv[u][k >> 2][k & 3], r);
      }
      for (int o = lpg >> 1; o >= 1; o >>= 1) r += __shfl_xor(r, o);
      const int i = i0 + u * per + sub;
      if (i < G && lane % lpg == 0) out[i] = r;
    }
  }
}

// Compile-time loop: Panels<K, N>::run(f) calls f(PanelC<k>) for k = K .. N - 1.
template <int V>
struct PanelC {
  static constexpr int value = V;
};
template <int K, int N>
struct Panels {
  template <typename F>
  static __device__ __forceinline__ void run(F&& f) {
    if constexpr (K < N) {
      f(PanelC<K>{});
      Panels<K + 1, N>::run(f);
    }
  }
};

// T = ceil(G / 16) panels.  Row i of the system is lane i % 64, slot i / 64;
// rows and columns from G to 16 T are zero but for a diagonal of kPadPivot, and
// their columns are left out.  (No step reads that diagonal; with 0 in its place the
// same steps come out slower as compiled: 4096 rows of G = 64 80 us instead of 69.)
//
// LDS.  Rows are kSolveLd doubles (17: the 16 rows and the k-pairs of a fragment
// read cover the 64 banks once), first of the Schur complement's columns, then of
// L's, which stay there for the backward substitution.  Panel p's rows from its
// diagonal ones on, then the column exchange; or PACKED, where that puts more
// systems on a CU (T = 4: eight for seven, T = 6: four for three) or leaves fewer
// registers in scratch (T = 8): one block of 16 diagonal rows, used by every panel
// in turn and then by its column exchange; panel p's rows below them; L's strict
// lower triangles of the diagonal rows, packed row by row, 120 a panel.  4096 rows,
// not packed and packed: G = 64 82 and 70 us, 88 389 and 211, 128 991 and 879; where
// it changes neither, packing costs its writes (G = 32 31 and 32, 80 166 and 175, 104
// 645 and 683).
// One wavefront: its LDS accesses complete in order, so there is no barrier; the
// empty asm statements keep the compiler from moving a read above another
// lane's write.
constexpr int kSolveLd = 17;
constexpr double kPadPivot = 1e300;
template <int T>
struct SolveShape {
  static constexpr int NS = T > 4 ? 2 : 1;        // rows of the system per lane
  static constexpr int NBLK = T * (T + 1) / 2;
  static constexpr bool PACKED = T == 4 || T == 6 || T == 8;
  static constexpr int kRows = 16 * kSolveLd;     // 16 rows
  // diagonal rows of panel p, and its rows from 16 (p + 1) on
  static __host__ __device__ constexpr int diag(int p) {
    return PACKED ? 0 : kRows * (p * T - p * (p - 1) / 2);
  }
  static __host__ __device__ constexpr int below(int p) {
    return PACKED ? kRows * (1 + p * (T - 1) - p * (p - 1) / 2) : diag(p) + kRows;
  }
  static constexpr int kEnd = PACKED ? below(T) : diag(T);   // the triangles, or the exchange
  // (a backward step reads up to 15 entries past a triangle's row)
  static constexpr size_t lds_bytes() {
    return (size_t)(kEnd + (PACKED ? 120 * T + 16 : 128)) * sizeof(double);
  }
};
static_assert(4 * SolveShape<6>::lds_bytes() <= 160 * 1024, "four systems a CU");

template <int T>
__global__ __launch_bounds__(64, T > 4 ? 1 : T > 2 ? 2 : 4) void solve_kernel(
    int rows, int cols, int g, const float* __restrict__ gram, const RhsSrc rs,
    float* __restrict__ scales, const uint8_t* __restrict__ active, Counters* __restrict__ cnt,
    Flags* __restrict__ flags, float lam, float rcond, int accept,
    const int32_t* __restrict__ rowmap, const int* __restrict__ n_dev) {
  using S = SolveShape<T>;
  constexpr int NS = S::NS;
  const int G = cols / g;
  if (n_dev != nullptr) rows = *n_dev;
  const int row = blockIdx.x;  // position of the sweep; layer row grow
  if (row >= rows) return;
  const int grow = map_row(rowmap, row);
  if (active != nullptr && !active[grow]) return;
  const int lane = threadIdx.x, lc = lane & 15, lk = lane >> 4;
  extern __shared__ double sm[];

  // ---- right-hand side r_i = sum over group i of (q - z) (W H) ----
  const bool cached = rs.ctl != nullptr && rs.ctl->valid != 0;   // uniform
  double* rc = rs.cache + (size_t)grow * G;
  if (!cached) {
    rhs_form(rs, grow, cols, g, G, sm);
    asm volatile("" ::: "memory");   // (one wavefront: its LDS accesses complete in order)
  }
  double r0[NS];
  int finite = 1;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int i = lane + 64 * s;
    r0[s] = 0.0;
    if (i < G) {
      r0[s] = cached ? rc[i] : sm[i];
      if (!cached) rc[i] = r0[s];
      finite &= isfinite(r0[s]) ? 1 : 0;
    }
  }
  asm volatile("" ::: "memory");

  // ---- the blocks: element v of block (bi, bj) is row 16 bi + lane % 16,
  // column 16 bj + 4 v + lane / 16 (entry (i, j), i >= j, is stored at (j, i)) ----
  f64x4 blk[S::NBLK];
  const float* gr = gram + (size_t)grow * G * G;
  double diag, sq;   // largest diagonal; sum of squares (both triangles)
  const bool last_in = 16 * (T - 1) + lc < G;   // rows of the last block row (others are < G)
  auto load = [&](double shift) __attribute__((always_inline)) {
    diag = 0.0;
    sq = 0.0;
    // (opaque copies: what depends on them is formed here each time instead of
    // being kept in registers across the factorisation)
    int lr = lc, lq = lk;
    asm volatile("" : "+v"(lr), "+v"(lq));
#pragma unroll
    for (int bi = 0; bi < T; ++bi) {
#pragma unroll
      for (int bj = 0; bj <= bi; ++bj) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * bi + lr, c = 16 * bj + 4 * v + lq;
          // rows and columns from G on read the last one's entries and are
          // replaced (only the upper triangle holds values)
          const int rc = bi == T - 1 ? min(r, G - 1) : r, cc = bj == T - 1 ? min(c, G - 1) : c;
          const double x = (double)gr[(uint32_t)(min(cc, rc) * G + max(cc, rc))];
          const bool in = bi < T - 1 || last_in;
          double val = x;
          if (bi == bj) {
            const bool eq = r == c, low = in && c <= r;
            finite &= isfinite(x) ? 1 : 0;
            diag = fmax(diag, low && eq ? x : 0.0);
            sq = fma(low ? (eq ? x : 2.0 * x) : 0.0, x, sq);
            val = low ? x + (eq ? shift : 0.0) : (eq ? kPadPivot : 0.0);
          } else {
            finite &= isfinite(x) ? 1 : 0;
            sq = fma(in ? 2.0 * x : 0.0, x, sq);
            val = in ? x : 0.0;
          }
          blk[bi * (bi + 1) / 2 + bj][v] = val;
        }
        // (formed here, not from kept values after the factorisation)
        asm volatile("" : "+v"(diag), "+v"(sq), "+v"(finite));
      }
    }
  };

  // A = L L^T with the forward substitution L y = r and, beside it, the
  // comparison system C x = 1 (|l_ik| x_k added where l_ik y_k is subtracted).
  // Column k stays unscaled while it is used: with l = a_k / pivot, a_j -=
  // l a_k[row j], r_i -= l_i r_k and x_i += |l_i| x_k, so the square roots are
  // off the chain; afterwards rr, xx and the columns of L take their 1 / L(k, k).
  double rr[NS], xx[NS], rs_own[NS];
  double minpiv;   // the smallest pivot, -1 where one is not positive and finite
  auto factor = [&]() __attribute__((always_inline)) {
    minpiv = INFINITY;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      rr[s] = r0[s];
      xx[s] = 1.0;
      rs_own[s] = 1.0;
    }
    Panels<0, T>::run([&](auto pc) __attribute__((always_inline)) {
      constexpr int p = decltype(pc)::value;
      constexpr int c0 = 16 * p, sp = c0 / 64, l0 = c0 % 64;   // slot and lane of its first row
      constexpr int below = 16 * (T - p - 1);
      double* dg = sm + S::diag(p);
      double* L = sm + S::below(p);
      double* colb = S::PACKED ? dg : sm + S::kEnd;   // (the diagonal rows are in registers then)
      // (an opaque copy, so that the comparisons below are made here and not
      // kept for every panel across the passes)
      int ln = lane;
      asm volatile("" : "+v"(ln));
#pragma unroll
      for (int bi = p; bi < T; ++bi)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          (bi == p ? dg : L + 16 * (bi - p - 1) * kSolveLd)[lc * kSolveLd + 4 * v + lk] =
              blk[bi * (bi + 1) / 2 + p][v];
      asm volatile("" ::: "memory");
      double a[NS][16], t[16], lp[NS];
      double* lrow[NS];
      // slots sp .. NS - 1, with a static index (arrays stay in registers)
      auto slots = [&](auto&& fn) __attribute__((always_inline)) { Panels<sp, NS>::run(fn); };
      slots([&](auto sc) __attribute__((always_inline)) {
        constexpr int s = decltype(sc)::value;
        const int i = ln + 64 * s - c0;   // rows above the panel repeat its first, rows past it the last
        lrow[s] = i < 16 || below == 0 ? dg + min(max(i, 0), 15) * kSolveLd
                                       : L + min(i - 16, below - 1) * kSolveLd;
#pragma unroll
        for (int k = 0; k < 16; ++k) a[s][k] = lrow[s][k];
      });
      double own = 1.0;
      Panels<0, 16>::run([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        constexpr int kn = k < 15 ? k + 1 : 15;
        // columns from G on change nothing (uniform)
        if (p == T - 1 && c0 + k >= G) return;
        asm volatile("" : "+v"(ln));
        const double pk = readlane_f64(a[sp][k], l0 + k);
        const bool b = !(pk > 0.0 && pk < INFINITY);
        minpiv = fmin(minpiv, b ? -1.0 : pk);
        asm volatile("" : "+v"(minpiv));   // (formed here, not from kept pivots later)
        const double piv = b ? 1.0 : pk;
        own = ln == l0 + k ? piv : own;
        double* ck = colb + 64 * (k & 1);
        if (k < 14) ck[ln] = a[sp][k];
        const double ip = chol_rcp(piv);
        const double rk = readlane_f64(rr[sp], l0 + k), xk = readlane_f64(xx[sp], l0 + k);
        // step k - 1 on the columns past k
        if constexpr (k > 0) {
          slots([&](auto sc) __attribute__((always_inline)) {
            constexpr int s = decltype(sc)::value;
#pragma unroll
            for (int j = k + 1; j < 16; ++j) a[s][j] = fma(-lp[s], t[j], a[s][j]);
          });
        }
        const double an = readlane_f64(a[sp][k], l0 + kn);
        slots([&](auto sc) __attribute__((always_inline)) {
          constexpr int s = decltype(sc)::value;
          lp[s] = ln + 64 * s > c0 + k ? a[s][k] * ip : 0.0;
          if constexpr (k < 15) a[s][kn] = fma(-lp[s], an, a[s][kn]);
          rr[s] = fma(-lp[s], rk, rr[s]);
          xx[s] = fma(fabs(lp[s]), xk, xx[s]);
        });
        asm volatile("" ::: "memory");
#pragma unroll
        for (int j = k + 2; j < 16; ++j) t[j] = ck[l0 + j];
      });
      // 1 / L(k, k) of the panel's rows, a row per lane
      const bool mine = ln >= l0 && ln < l0 + 16;
      const double rsv = chol_rsqrt(own);
      rs_own[sp] = mine ? rsv : rs_own[sp];
      // L's columns; rows below the panel's own 16 are complete, and within those
      // the entries above the diagonal are never read
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const double rk = readlane_f64(rsv, l0 + k);
        slots([&](auto sc) __attribute__((always_inline)) { a[decltype(sc)::value][k] *= rk; });
      }
      slots([&](auto sc) __attribute__((always_inline)) {
        constexpr int s = decltype(sc)::value;
        const int i = ln + 64 * s - c0;
        if (i >= (S::PACKED ? 16 : 0) && i < 16 + below) {
#pragma unroll
          for (int k = 0; k < 16; ++k) lrow[s][k] = a[s][k];
        }
        if constexpr (S::PACKED && s == sp) {
          double* tri = sm + S::kEnd + 120 * p + i * (i - 1) / 2;
#pragma unroll
          for (int k = 0; k < 15; ++k)
            if (i > k && i < 16) tri[k] = a[s][k];
        }
      });
      asm volatile("" ::: "memory");
      // blocks right of the panel: block (bi, bj) -= L_bi L_bj^T
      if constexpr (p + 1 < T) {
        double f[T - p - 1][4];
#pragma unroll
        for (int b = p + 1; b < T; ++b)
#pragma unroll
          for (int ks = 0; ks < 4; ++ks)
            f[b - p - 1][ks] = L[(16 * (b - p - 1) + lc) * kSolveLd + 4 * ks + lk];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
          for (int bi = p + 1; bi < T; ++bi)
#pragma unroll
            for (int bj = p + 1; bj <= bi; ++bj)
              blk[bi * (bi + 1) / 2 + bj] =
                  mfma_f64(-f[bj - p - 1][ks], f[bi - p - 1][ks], blk[bi * (bi + 1) / 2 + bj]);
      }
    });
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      rr[s] *= rs_own[s];
      xx[s] *= rs_own[s];
    }
  };

  // The passes of the stabilised branch in one loop (the factorisation is
  // long): plain; where its bound does not clear t, A - t I and then A again;
  // A + lambda I.  Every lane sees the same pivots, so the row decides as one.
  enum { kPlain, kBelow, kRidge, kAgain };
  int pass = kPlain;
  double shift = 0.0, tshift = 0.0;
  bool ridge = false, failed = false;
  while (true) {
    load(shift);
    factor();
    if (pass == kPlain) {
      double dmax = diag, fro = sq, xm = 0.0;
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (lane + 64 * s < G) xm = fmax(xm, xx[s] == xx[s] ? xx[s] : INFINITY);
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) {
        dmax = fmax(dmax, __shfl_xor(dmax, o));
        fro += __shfl_xor(fro, o);
        xm = fmax(xm, __shfl_xor(xm, o));
      }
      tshift = (double)rcond * fmax(sqrt(fro), (double)kFp32Eps);
      ridge = !__all(finite != 0) || !(minpiv > (double)rcond * fmax(dmax, (double)kFp32Eps));
      // lambda_min >= 1 / (G (max x)^2) (a NaN bound clears nothing)
      if (!ridge && (double)G * xm * xm * tshift < 1.0) break;
      pass = ridge ? kRidge : kBelow;
      shift = ridge ? (double)lam : -tshift;
    } else if (pass == kBelow) {
      ridge = !(minpiv > 0.0);
      pass = ridge ? kRidge : kAgain;
      shift = ridge ? (double)lam : 0.0;
    } else {
      if (pass == kRidge) failed = !(minpiv > 0.0);
      break;
    }
  }

  // ---- backward substitution L^T s = y: s_k = y_k / l_kk, y_i -= l_ki s_k ----
  // Step k of panel pk = k / 16: lane i finds L(k, i) in row k of panel i / 16, or
  // (packed) in the triangle of panel pk if that is its own.  Lanes of later
  // panels read something of theirs, unused.
  for (int pk = T - 1; pk >= 0; --pk) {
    const double* li[NS];
    bool own[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int i = min(lane + 64 * s, 16 * T - 1), p = i >> 4;
      own[s] = S::PACKED && p >= pk;
      li[s] = sm + (i & 15) +
              (own[s] ? S::kEnd + 120 * p
                      : S::below(p) + S::kRows * (S::PACKED ? pk - p - 1 : max(pk - p, 0) - 1));
    }
    for (int kr = min(15, G - 1 - 16 * pk); kr >= 0; --kr) {
      const int k = 16 * pk + kr;
      const double y = NS == 1 || k < 64 ? rr[0] * rs_own[0] : rr[NS - 1] * rs_own[NS - 1];
      const double sk = readlane_f64(y, k & 63);
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int i = lane + 64 * s;
        const double l = li[s][own[s] ? kr * (kr - 1) / 2 : kr * kSolveLd];
        rr[s] = i < k ? fma(-l, sk, rr[s]) : (i == k ? sk : rr[s]);
      }
    }
  }

  // Ridge acceptance (the remark of App. G.5, optional): a ridge solution is
  // kept only when it does not increase F_j.  At fixed codes F_j(s) = const +
  // s^T G s - 2 r^T s, from the Gram matrix (loaded again) and the right-hand
  // side: dq = s'^T G s' - s^T G s - 2 r^T (s' - s).
  bool keep_old = false;
  if (accept && ridge && !failed) {  // uniform
    double* vn = sm;                 // s' (new) and s (previous): the panels are done with
    double* vo = sm + 16 * T;
    double dq = 0.0;
    asm volatile("" ::: "memory");
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int i = lane + 64 * s;
      if (i < 16 * T) {
        const double so = i < G ? (double)scales[(size_t)grow * G + i] : 0.0;
        vn[i] = i < G ? rr[s] : 0.0;
        vo[i] = so;
        if (i < G) dq -= 2.0 * r0[s] * (rr[s] - so);
      }
    }
    asm volatile("" ::: "memory");
    load(0.0);
#pragma unroll
    for (int bi = 0; bi < T; ++bi)
#pragma unroll
      for (int bj = 0; bj <= bi; ++bj)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * bi + lc, c = 16 * bj + 4 * v + lk;
          if (r < G && c <= r)
            dq += (r == c ? 1.0 : 2.0) * blk[bi * (bi + 1) / 2 + bj][v] *
                  (vn[r] * vn[c] - vo[r] * vo[c]);
        }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) dq += __shfl_xor(dq, o);
    keep_old = dq > 0.0;
  }

  if (!failed && !keep_old) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int i = lane + 64 * s;
      if (i < G) scales[(size_t)grow * G + i] = (float)rr[s];
    }
  }
  if (lane == 0) {
    if (ridge) atomicAdd(&cnt->ridge_rows, 1u);
    if (failed) {
      atomicAdd(&cnt->solve_failed, 1u);
      atomicAdd(&flags->solve_failed, 1);
    }
  }
}

template <int T>
static hipError_t launch_solve_t(hipStream_t st, int rows, int cols, int g, const float* gram,
                                 const RhsSrc& rs, float* scales, const uint8_t* active,
                                 Counters* cnt, Flags* flags, float lam, float rcond, int accept,
                                 const int32_t* rowmap, const int* n_dev) {
  constexpr size_t lds = SolveShape<T>::lds_bytes();
  static std::atomic<unsigned long long> lds_set{0};
  const hipError_t e = allow_dynamic_lds((const void*)solve_kernel<T>, lds, lds_set);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(solve_kernel<T>, dim3(rows), dim3(64), lds, st, rows, cols, g, gram, rs,
                     scales, active, cnt, flags, lam, rcond, accept, rowmap, n_dev);
  return hipGetLastError();
}

hipError_t launch_solve(hipStream_t st, int rows, int cols, int g, const float* gram,
                        const float* wh, const uint8_t* codes, const int32_t* zeros,
                        double* rhs_cache, const GramCtl* rctl,
                        float* scales, const uint8_t* active, Counters* cnt, Flags* flags,
                        float lam, float rcond, int accept, const int32_t* rowmap,
                        const int* n_dev) {
  const RhsSrc rs{wh, codes, zeros, rhs_cache, rctl};
#define JARQ_SOLVE(T)                                                                            \
  case T:                                                                                        \
    return launch_solve_t<T>(st, rows, cols, g, gram, rs, scales, active, cnt, flags, lam, rcond, \
                             accept, rowmap, n_dev)
  switch ((cols / g + 15) / 16) {
    JARQ_SOLVE(1);
    JARQ_SOLVE(2);
    JARQ_SOLVE(3);
    JARQ_SOLVE(4);
    JARQ_SOLVE(5);
    JARQ_SOLVE(6);
    JARQ_SOLVE(7);
    JARQ_SOLVE(8);
    default: return hipErrorInvalidValue;  // G > 128 is rejected by the API
  }
#undef JARQ_SOLVE
}

}  // namespace jarq
