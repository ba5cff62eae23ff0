// Panel kernels of the tile Cholesky (gfx950): the factorisation of a diagonal
// tile, the solves with it (panel tiles, inverse) and the updates between its
// blocks.  They carry the critical path.
//
// k_potrf_block factors one 128 x 128 block on the diagonal of an FP64 tile
// with one workgroup and is built for latency, not for flops (the block's 0.7
// MFLOP are 2.3 us of one CU's FP64 MFMA rate).
#include <type_traits>

#include "mpcr_internal.h"

namespace mpcr {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int SB = 128;  // diagonal block
constexpr int PB = 16;   // panel width inside it
constexpr int PW = 32;   // inverted diagonal blocks handed to the panel solves
constexpr int NP = SB / PB;
constexpr int BLD = PB + 1;  // LDS row of a 16 x 16 block (doubles)

__device__ __forceinline__ int tri_blk(int i, int j) { return i * (i + 1) / 2 + j; }

// 1 / sqrt(d) for d > 0 (normal): the hardware estimate refined by two
// Newton steps y <- y + (y / 2)(1 - d y^2), each of which squares the relative
// error (about 3/2 e^2), so an estimate good to 2^-14 or better ends within a
// few units in the last place.
__device__ __forceinline__ double rsqrt_f64(double d) {
  double y = __builtin_amdgcn_rsq(d);
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const double e = fma(-d * y, y, 1.0);
    y = fma(0.5 * y, e, y);
  }
  return y;
}

// Column steps with lane N of every 16-lane row broadcast to that row inside
// the operation (DPP row_newbcast; no trip through scalar registers).  A DPP
// operand must have been written two wait states before its use, and a result
// of v_rsq one before: every block sees to that itself.
//   steps of rsqrt_f64 of the next pivot, each with N of the column's remaining
//   updates d[q] -= d_C[q] d_C, x[q] -= d_C[q] x_C, q = Q .. Q + N - 1 (s = d_C,
//   t = x_C) behind it.  Written out so, because the compiler puts the whole
//   dependent chain behind the updates that are there to hide it.
#define MPCR_BCAST_PAIR(a, b, q)                                                                 \
  "v_fmac_f64_dpp %[" a "], -%[s], %[s] row_newbcast:%c[" q "] row_mask:0xf bank_mask:0xf\n\t" \
  "v_fmac_f64_dpp %[" b "], -%[s], %[t] row_newbcast:%c[" q "] row_mask:0xf bank_mask:0xf\n\t"
#define MPCR_PIVOT_STEP(NAME, OPS)                                                                           \
  template <int Q, int N>                                                                                    \
  __device__ __forceinline__ void NAME(double (&d)[PB], double (&x)[PB], double s, double t, double piv,     \
                                       double& y, double& e, double& h) {                                    \
    if constexpr (N == 0)                                                                                    \
      asm volatile(OPS : [y] "+v"(y), [e] "+v"(e), [h] "+v"(h) : [p] "v"(piv));                              \
    else if constexpr (N == 1)                                                                               \
      asm volatile(OPS MPCR_BCAST_PAIR("d0", "x0", "q0")                                                     \
                   : [y] "+v"(y), [e] "+v"(e), [h] "+v"(h), [d0] "+v"(d[Q]), [x0] "+v"(x[Q])                 \
                   : [p] "v"(piv), [s] "v"(s), [t] "v"(t), [q0] "n"(Q));                                     \
    else                                                                                                     \
      asm volatile(OPS MPCR_BCAST_PAIR("d0", "x0", "q0") MPCR_BCAST_PAIR("d1", "x1", "q1")                   \
                   : [y] "+v"(y), [e] "+v"(e), [h] "+v"(h), [d0] "+v"(d[Q]), [x0] "+v"(x[Q]),                \
                     [d1] "+v"(d[Q + 1]), [x1] "+v"(x[Q + 1])                                                \
                   : [p] "v"(piv), [s] "v"(s), [t] "v"(t), [q0] "n"(Q), [q1] "n"(Q + 1));                    \
  }
MPCR_PIVOT_STEP(pivot_rsq, "v_rsq_f64 %[y], %[p]\n\ts_nop 0\n\t")
MPCR_PIVOT_STEP(pivot_mul, "v_mul_f64 %[e], -%[p], %[y]\n\tv_mul_f64 %[h], 0.5, %[y]\n\t")
MPCR_PIVOT_STEP(pivot_err, "v_fma_f64 %[e], %[e], %[y], 1.0\n\ts_nop 0\n\t")
MPCR_PIVOT_STEP(pivot_fix, "v_fma_f64 %[y], %[h], %[e], %[y]\n\ts_nop 0\n\t")
// 1 / sqrt(piv), with the updates q = C + 2 .. 15 of column C
template <int C>
__device__ __forceinline__ double pivot_updates(double (&d)[PB], double (&x)[PB], double piv) {
  constexpr int n = PB - 2 - C;  // updates, spread over the seven steps
  constexpr int Q1 = C + 2 + (n + 6) / 7, Q2 = Q1 + (n + 5) / 7, Q3 = Q2 + (n + 4) / 7, Q4 = Q3 + (n + 3) / 7;
  constexpr int Q5 = Q4 + (n + 2) / 7, Q6 = Q5 + (n + 1) / 7;
  const double s = d[C], t = x[C];
  double y = 0.0, e = 0.0, h = 0.0;
  pivot_rsq<C + 2, Q1 - C - 2>(d, x, s, t, piv, y, e, h);
  pivot_mul<Q1, Q2 - Q1>(d, x, s, t, piv, y, e, h);
  pivot_err<Q2, Q3 - Q2>(d, x, s, t, piv, y, e, h);
  pivot_fix<Q3, Q4 - Q3>(d, x, s, t, piv, y, e, h);
  pivot_mul<Q4, Q5 - Q4>(d, x, s, t, piv, y, e, h);
  pivot_err<Q5, Q6 - Q5>(d, x, s, t, piv, y, e, h);
  pivot_fix<Q6, PB - Q6>(d, x, s, t, piv, y, e, h);
  return y;
}
#undef MPCR_PIVOT_STEP
#undef MPCR_BCAST_PAIR
//   fma_bcast<Q>    a[q] -= s[q] t for q = Q .. 15 (s[q] is lane q's value)
template <int Q>
__device__ __forceinline__ void fma_bcast(double (&a)[PB], double s, double t) {
  if constexpr (Q + 8 <= PB) {
    asm volatile(
        "s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%8, %9 row_newbcast:%c10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, -%8, %9 row_newbcast:%c11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, -%8, %9 row_newbcast:%c12 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, -%8, %9 row_newbcast:%c13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %4, -%8, %9 row_newbcast:%c14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %5, -%8, %9 row_newbcast:%c15 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %6, -%8, %9 row_newbcast:%c16 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %7, -%8, %9 row_newbcast:%c17 row_mask:0xf bank_mask:0xf"
        : "+v"(a[Q]), "+v"(a[Q + 1]), "+v"(a[Q + 2]), "+v"(a[Q + 3]), "+v"(a[Q + 4]), "+v"(a[Q + 5]), "+v"(a[Q + 6]), "+v"(a[Q + 7])
        : "v"(s), "v"(t), "n"(Q), "n"(Q + 1), "n"(Q + 2), "n"(Q + 3), "n"(Q + 4), "n"(Q + 5), "n"(Q + 6), "n"(Q + 7));
    fma_bcast<Q + 8>(a, s, t);
  } else if constexpr (Q + 4 <= PB) {
    asm volatile(
        "s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%4, %5 row_newbcast:%c6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, -%4, %5 row_newbcast:%c7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, -%4, %5 row_newbcast:%c8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, -%4, %5 row_newbcast:%c9 row_mask:0xf bank_mask:0xf"
        : "+v"(a[Q]), "+v"(a[Q + 1]), "+v"(a[Q + 2]), "+v"(a[Q + 3])
        : "v"(s), "v"(t), "n"(Q), "n"(Q + 1), "n"(Q + 2), "n"(Q + 3));
    fma_bcast<Q + 4>(a, s, t);
  } else if constexpr (Q + 2 <= PB) {
    asm volatile(
        "s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%2, %3 row_newbcast:%c4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, -%2, %3 row_newbcast:%c5 row_mask:0xf bank_mask:0xf"
        : "+v"(a[Q]), "+v"(a[Q + 1])
        : "v"(s), "v"(t), "n"(Q), "n"(Q + 1));
    fma_bcast<Q + 2>(a, s, t);
  } else if constexpr (Q + 1 <= PB) {
    asm volatile(
        "s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%c3 row_mask:0xf bank_mask:0xf"
        : "+v"(a[Q])
        : "v"(s), "v"(t), "n"(Q));
    fma_bcast<Q + 1>(a, s, t);
  }
}
//   column<C>       d_C *= r, x_C *= r, their products with lane C + 1 from d[C + 1]
//                   and x[C + 1], and returns lane C + 1 of the new d[C + 1]: the next pivot
template <int C>
__device__ __forceinline__ double column(double (&d)[PB], double (&x)[PB], double r) {
  double piv;
  asm volatile(
        "v_mul_f64 %0, %0, %5\n\t"
        "v_mul_f64 %1, %1, %5\n\t"
        "s_nop 0\n\t"
        "v_fmac_f64_dpp %2, -%0, %0 row_newbcast:%c6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, -%0, %1 row_newbcast:%c6 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_mov_b64_dpp %4, %2 row_newbcast:%c6 row_mask:0xf bank_mask:0xf"
        : "+v"(d[C]), "+v"(x[C]), "+v"(d[C + 1]), "+v"(x[C + 1]), "=&v"(piv)
        : "v"(r), "n"(C + 1));
  return piv;
}

// Column C and the following ones of a right-looking Cholesky of a 16 x 16
// block and of the inversion of its factor: d[c] is element c of row lane % 16
// of the block, x[c] starts as element c of row lane % 16 of the unit matrix
// (every 16-lane row of the wave holds a copy of both).  The unit rows are
// solved by the same column steps that factor the block and end as the columns
// of the inverse.  Elements above the diagonal are carried along and never
// used.  r is 1 / sqrt of column C's pivot; the next pivot and its reciprocal
// square root come first in a column, so that their latency lies behind the
// column's other updates, and no branch separates the columns.  A pivot that is
// not positive (or infinite) makes r and everything after it NaN, which the
// last r, returned, shows.  TRACK: bad collects the columns whose pivot is not
// positive as bits; without it, the workgroup's barrier in mid-phase is met in
// column MID.
constexpr int MID = 4;
template <int C, bool TRACK>
__device__ __forceinline__ double factor_rows16(double (&d)[PB], double (&x)[PB], double r, uint32_t& bad) {
  if constexpr (C + 1 < PB) {
    const double piv = column<C>(d, x, r);
    if (TRACK) bad |= (uint32_t)(__builtin_amdgcn_ballot_w64(!(piv > 0.0)) & 1u) << (C + 1);
    if (!TRACK && C == MID) __syncthreads();
    const double rn = pivot_updates<C>(d, x, piv);
    return factor_rows16<C + 1, TRACK>(d, x, rn, bad);
  } else {
    d[C] *= r;
    x[C] *= r;
    return r;
  }
}

// Rows 16 .. 31 of column lane % 16 of the inverse of [[A, 0], [B, C]] by forward
// substitution: y -= B a (a: that column of A^{-1}), then the column steps of C
// (b[m], c[m]: element m of this lane's row; r: the reciprocals of C's diagonal;
// a and r by eights).
template <int M, int END>
__device__ __forceinline__ void substitute_left(double (&y)[PB], const double (&b)[PB], const double (&a)[8]) {
  if constexpr (M < END) {
    fma_bcast<0>(y, b[M], a[M % 8]);
    substitute_left<M + 1, END>(y, b, a);
  }
}
template <int M, int END>
__device__ __forceinline__ void substitute_diag(double (&y)[PB], const double (&c)[PB], const double (&r)[8]) {
  if constexpr (M < END) {
    y[M] *= r[M % 8];
    fma_bcast<M + 1>(y, c[M], y[M]);
    substitute_diag<M + 1, END>(y, c, r);
  }
}
// values that are to be in registers from here on
template <int N>
__device__ __forceinline__ void keep(double (&v)[N]) {
#pragma unroll
  for (int c = 0; c < N; ++c) asm volatile("" : "+v"(v[c]));
}
// element 4 (lane / 16) + C of v, which every 16-lane row holds a copy of
template <int ROW>
__device__ __forceinline__ int in_row(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, 0xe4, 1 << ROW, 0xf, false);
}
template <int C>
__device__ __forceinline__ double own_quarter(const double (&v)[PB]) {
  int2 t = __builtin_bit_cast(int2, v[C]);
  const int2 v1 = __builtin_bit_cast(int2, v[4 + C]), v2 = __builtin_bit_cast(int2, v[8 + C]);
  const int2 v3 = __builtin_bit_cast(int2, v[12 + C]);
  t = {in_row<1>(t.x, v1.x), in_row<1>(t.y, v1.y)};
  t = {in_row<2>(t.x, v2.x), in_row<2>(t.y, v2.y)};
  t = {in_row<3>(t.x, v3.x), in_row<3>(t.y, v3.y)};
  return __builtin_bit_cast(double, t);
}

struct PotrfLds {
  double L[NP * (NP + 1) / 2][PB][BLD];  // the lower 16 x 16 blocks
  double Di[4][PB][BLD];                 // inverses of the factored diagonal blocks p (slot p % 4)
  int fail;
};

// The block's 36 lower 16 x 16 blocks live in LDS.  In phase p
//   wave 0 forms the panel's top block L_{p,p-1}, updates block (p, p) with it,
//       factors that block and inverts its factor;
//   one wave per row block i > p forms L_{i,p-1} = A_{i,p-1} times the inverse's
//       transpose and subtracts panels 0 .. p - 1 from block (i, p) (one more
//       wave: from block (p + 1, p + 1)), the last panel after a barrier, which
//       wave 0 meets between two columns of its factorisation; the panel p - 1
//       is then stored;
//   wave 7 forms dinv, the inverses of the four 32 x 32 diagonal blocks, by
//       forward substitution on unit vectors.
// Wave 4, which shares wave 0's SIMD, is the last to get a matrix product (they
// hold up wave 0's FP64 operations).
// Products are FP64 MFMA.  The panel's are formed transposed (inverse times
// A^T): that result layout is the operand layout of the next product.  The chain
// per phase is wave 0's: two products of four MFMAs and sixteen columns, nearly
// all of it instruction issue.  Updating block columns from the left keeps every
// phase's products (at most 16 blocks, 27 from the right) shorter than that.
// Nothing above the diagonal is written (no kernel reads it).
// 87 KB of LDS and at most 128 VGPRs: with the tile updates resident on every
// CU (two workgroups of 74 KB), it fits as soon as one of them retires.  (The
// LDS is given at the launch: counted by the compiler, it would make it spend
// 256 VGPRs.)
// Measured alone: 24 us a block; 87 us for the version whose diagonal
// blocks were factored with scalar-register broadcasts and lane masks, inverted
// in a second pass and followed by the trailing update before the next one.
__global__ __launch_bounds__(512, 4) void k_potrf_block(TileView tv, int k, int j, double* dinv) {
  __builtin_amdgcn_s_setprio(2);
  const int info0 = *tv.info;
  const int nb = tv.nb, c0 = j * SB;
  double* A = (double*)tv.tile(k, k) + (int64_t)c0 * nb + c0;
  extern __shared__ __attribute__((aligned(16))) char potrf_lds[];
  PotrfLds& sm = *(PotrfLds*)potrf_lds;
  auto& L = sm.L;
  auto& Di = sm.Di;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int lr = lane >> 4, lc = lane & 15;  // MFMA result: rows lr + 4 r, column lc

  // load: one wave per column, two rows per lane (column pieces of 1 KB).  The
  // first panel goes to LDS at once, the columns behind it (waves 1 .. 7) beside
  // the first factorisation; the info word is looked at only once the loads are
  // on their way.
  constexpr int NLATER = (SB - PB) / 7;
  double2 later[NLATER];
  const int lbi = lane >> 3, lrow = 2 * (lane & 7);
  {
    double2 v[2];
#pragma unroll
    for (int g = 0; g < 2; ++g) v[g] = *(const double2*)(A + (int64_t)(wave + 8 * g) * nb + 2 * lane);
#pragma unroll
    for (int g = 0; g < NLATER; ++g) {
      const int c = PB + wave - 1 + 7 * g;
      if (wave > 0 && lbi >= c / PB) later[g] = *(const double2*)(A + (int64_t)c * nb + 2 * lane);
    }
    if (info0) return;
    if (tid == 0) sm.fail = 0;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      L[tri_blk(lbi, 0)][lrow][wave + 8 * g] = v[g].x;
      L[tri_blk(lbi, 0)][lrow + 1][wave + 8 * g] = v[g].y;
    }
  }
  __syncthreads();
  if (wave > 0) {
#pragma unroll
    for (int g = 0; g < NLATER; ++g) {
      const int c = PB + wave - 1 + 7 * g, bj = c / PB;
      if (lbi >= bj) {
        L[tri_blk(lbi, bj)][lrow][c % PB] = later[g].x;
        L[tri_blk(lbi, bj)][lrow + 1][c % PB] = later[g].y;
      }
    }
  }

  // acc -= L(i, q) L(j, q)^T, q = q0 .. q1 - 1
  auto update = [&](d4 acc, int i, int j, int q0, int q1) {
    for (int q = q0; q < q1; ++q) {
      const double(*P)[BLD] = L[tri_blk(i, q)], (*Q)[BLD] = L[tri_blk(j, q)];
      double a[4], b[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        a[u] = -P[lc][4 * u + lr];
        b[u] = Q[lc][4 * u + lr];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], acc, 0, 0, 0);
    }
    return acc;
  };
  // (elements u in row lr + 4 u, column lc)
  auto load_block = [&](int i, int j) {
    d4 v;
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = L[tri_blk(i, j)][lr + 4 * u][lc];
    return v;
  };
  auto store_block = [&](int i, int j, d4 v) {
#pragma unroll
    for (int u = 0; u < 4; ++u) L[tri_blk(i, j)][lr + 4 * u][lc] = v[u];
  };
  // L_ip[lc][4 u + lr] of block row i in register u
  auto panel_block = [&](int i, int p) {
    double(*P)[BLD] = L[tri_blk(i, p)];
    double di[4], a[4];
    d4 x = {0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      di[u] = Di[p & 3][lc][4 * u + lr];
      a[u] = P[lc][4 * u + lr];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) x = __builtin_amdgcn_mfma_f64_16x16x4f64(di[u], a[u], x, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < 4; ++u) P[lc][4 * u + lr] = x[u];
    return x;
  };

#pragma unroll 1
  for (int p = 0; p <= NP; ++p) {
    asm volatile("" : "+v"(lr), "+v"(lc));  // what derives from them is not to be kept in registers from phase to phase
    if (wave == 0 && p < NP) {
      __builtin_amdgcn_s_setprio(3);
      double(*D)[BLD] = L[tri_blk(p, p)];
      if (p > 0) {
        d4 acc = load_block(p, p);
        const d4 v = panel_block(p, p - 1);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-v[u], v[u], acc, 0, 0, 0);
        store_block(p, p, acc);
        __builtin_amdgcn_wave_barrier();
      }
      double d[PB], x[PB];
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        d[c] = D[lc][c];
        x[c] = c == lc ? 1.0 : 0.0;
      }
      uint32_t bad = 0;
      const double rl = factor_rows16<0, false>(d, x, rsqrt_f64(D[0][0]), bad);
      if (!(rl > 0.0)) {  // (uniform) find the first column whose pivot is not positive
#pragma unroll
        for (int c = 0; c < PB; ++c) {
          d[c] = D[lc][c];
          x[c] = c == lc ? 1.0 : 0.0;
        }
        const double piv = D[0][0];
        bad = __builtin_amdgcn_ballot_w64(!(piv > 0.0)) & 1u;
        factor_rows16<0, true>(d, x, rsqrt_f64(piv), bad);
        if (bad && tid == 0) {
          sm.fail = 1;
          *tv.info = k * nb + c0 + PB * p + __builtin_ctz(bad) + 1;
        }
      }
      // every 16-lane row stores four columns of its copies
      const double dq[4] = {own_quarter<0>(d), own_quarter<1>(d), own_quarter<2>(d), own_quarter<3>(d)};
      const double xq[4] = {own_quarter<0>(x), own_quarter<1>(x), own_quarter<2>(x), own_quarter<3>(x)};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        D[lc][4 * lr + c] = dq[c];
        Di[p & 3][4 * lr + c][lc] = xq[c];
      }
      __builtin_amdgcn_s_setprio(2);
    } else {
      if (wave == 7 && p > 0 && p % 2 == 0) {  // (dinv below, second half)
        const double(*A0)[BLD] = Di[(p - 2) & 3], (*C0)[BLD] = Di[(p - 1) & 3], (*Y)[BLD] = Di[(p + 1) & 3];
        const double(*Cl)[BLD] = L[tri_blk(p - 1, p - 1)];
        double y[PB], u[PB], v[8];
#pragma unroll
        for (int c = 0; c < PB; ++c) {
          y[c] = Y[c][lc];
          u[c] = Cl[lc][c];
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = C0[c][c];
        keep(y);
        keep(u);
        keep(v);
        substitute_diag<0, 8>(y, u, v);
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = C0[8 + c][8 + c];
        keep(v);
        substitute_diag<8, 16>(y, u, v);
        const double yq[4] = {own_quarter<0>(y), own_quarter<1>(y), own_quarter<2>(y), own_quarter<3>(y)};
        double* o = dinv + (int64_t)(c0 + PB * (p - 2)) * PW + lc * PW;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int R = 4 * lr + c;
          o[R] = R >= lc ? A0[R][lc] : 0.0;
          o[PB + R] = yq[c];
          o[PB * PW + R] = 0.0;
          o[PB * PW + PB + R] = R >= lc ? C0[R][lc] : 0.0;
        }
      }
      if (p < NP) {
        // task t: block (p + 1 + t, p), behind them block (p + 1, p + 1); the
        // sixth and seventh are there only for p <= 2
        const int t = wave == 4 ? 5 : wave == 7 ? 6 : wave < 4 ? wave - 1 : wave - 2, nrow = NP - 1 - p;
        const bool row = t < nrow, task = p > 0 && t <= nrow && nrow > 0;
        const int i = row ? p + 1 + t : p + 1, j = row ? p : p + 1;
        d4 acc;
        if (task) {
          acc = load_block(i, j);
          if (row) panel_block(i, p - 1);
          acc = update(acc, i, j, 0, p - 1);
        }
        __syncthreads();
        if (task) store_block(i, j, update(acc, i, j, p - 1, p));
      }
      // dinv (column-major): the inverted 32 x 32 block [[A', 0], [N, C']] of two
      // panels, N column by column (column lc in every 16-lane row, which stores
      // its quarter): the rows above C in the second panel's phase, C's in the
      // next (in between in a slot of Di that is not in use)
      if (wave == 7 && p % 2) {
        const double(*Bl)[BLD] = L[tri_blk(p, p - 1)], (*A0)[BLD] = Di[(p - 1) & 3];
        double y[PB], u[PB], v[8];
#pragma unroll
        for (int c = 0; c < PB; ++c) {
          u[c] = Bl[lc][c];
          y[c] = 0.0;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = c >= lc ? A0[c][lc] : 0.0;
        keep(u);
        keep(v);
        substitute_left<0, 8>(y, u, v);
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = 8 + c >= lc ? A0[8 + c][lc] : 0.0;
        keep(v);
        substitute_left<8, 16>(y, u, v);
        const double yq[4] = {own_quarter<0>(y), own_quarter<1>(y), own_quarter<2>(y), own_quarter<3>(y)};
#pragma unroll
        for (int c = 0; c < 4; ++c) Di[(p + 2) & 3][4 * lr + c][lc] = yq[c];
      }
      // panel p - 1 to memory: one wave per column, two rows per lane
      if (p > 0 && wave != 7) {
        const int R = PB * (p - 1) + 2 * lane, rb = R < SB ? R / PB : p - 1;
        const int w0 = p < NP ? 1 : 0;  // (wave 0 stores the last one too)
        const double(*b)[BLD] = L[tri_blk(rb, p - 1)];
        double2 v[3];
#pragma unroll
        for (int g = 0; g < 3; ++g) {
          const int c = min(wave - w0 + g * (7 - w0), PB - 1);
          v[g] = {b[R % PB][c], b[R % PB + 1][c]};
        }
#pragma unroll
        for (int g = 0; g < 3; ++g) {
          const int c = wave - w0 + g * (7 - w0);
          double* o = A + (int64_t)(PB * (p - 1) + c) * nb + R;
          if (c >= PB || R >= SB) continue;
          if (2 * lane >= c) *(double2*)o = v[g];
          else if (2 * lane + 1 == c) o[1] = v[g].y;
        }
      }
    }
    if (p == NP) break;
    __syncthreads();
    if (sm.fail) return;
  }
}

hipError_t launch_potrf_block(const TileView& tv, int k, int j, double* dinv, hipStream_t s) {
  k_potrf_block<<<1, 512, sizeof(PotrfLds), s>>>(tv, k, j, dinv);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Panel solves and inverses of tiles above 512 (k_trsm, k_trsm4, k_trtri).
// ---------------------------------------------------------------------------
// acc0/acc1 (16 x 16 each) += A[R0.., K0:K1] * B[C0.., K0:K1]^T, operands read
// straight from column-major FP64 storage (lda = ldb = ld).  Software
// pipelined: the twelve loads of the next 16-wide k batch are issued before the
// eight MFMAs of the current one.  K1 - K0 is a multiple of 4.
__device__ __forceinline__ void mfma_rows16x32(const double* A, const double* B, int64_t ld, int R0, int C0, int K0,
                                               int K1, int lane, d4& acc0, d4& acc1) {
  const int r = lane & 15, q = lane >> 4;
  auto ld12 = [&](int kk, double* a, double* b0, double* b1) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t col = kk + 4 * u + q;
      a[u] = A[col * ld + R0 + r];
      b0[u] = B[col * ld + C0 + r];
      b1[u] = B[col * ld + C0 + 16 + r];
    }
  };
  int kk = K0;
  const int full_end = K0 + ((K1 - K0) / 16) * 16;
  if (kk < full_end) {
    double a[4], b0[4], b1[4];
    ld12(kk, a, b0, b1);
    for (; kk < full_end; kk += 16) {
      double na[4], nb0[4], nb1[4];
      const bool more = kk + 16 < full_end;
      if (more) ld12(kk + 16, na, nb0, nb1);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b0[u], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b1[u], acc1, 0, 0, 0);
      }
      if (more) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          a[u] = na[u];
          b0[u] = nb0[u];
          b1[u] = nb1[u];
        }
      }
    }
  }
  for (; kk < K1; kk += 4) {
    const int64_t col = kk + q;
    double a = A[col * ld + R0 + r], b0 = B[col * ld + C0 + r], b1 = B[col * ld + C0 + 16 + r];
    acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b0, acc0, 0, 0, 0);
    acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b1, acc1, 0, 0, 0);
  }
}

// ---------------------------------------------------------------------------
// Triangular solves by one wave with inverted 32 x 32 diagonal blocks.
//
// trsm_rows16_inv solves X L^T = A for 16 rows r0 .. r0+15 over the columns
// [c0, c1), left-looking over 32-column chunks J:
//   T   = A[rows, J] - X[rows, c0:J] L[J, c0:J]^T     (FP64 MFMA)
//   X_J = T D_J^{-T}                                 (FP64 MFMA, D_J^{-1} given)
// X (ld ldx) holds the solved columns of these rows, L the factor (ld ldl);
// load_a(idx) and store_x(idx, v) read A and write X_J at a column-major index
// of the rows' storage.  Each wave works alone (no barriers): the chunk goes
// from the MFMA result layout to the operand layout through Ts (16 x 33
// doubles of LDS per wave), and X is re-read by the same wave after a
// workgroup-scope fence.
// ---------------------------------------------------------------------------
template <class LoadA, class StoreX>
__device__ __forceinline__ void trsm_rows16_inv(const double* X, const double* L, int64_t ld, const double* dinv,
                                                int c0, int c1, int r0, double (*Ts)[PW + 1], int lane, LoadA load_a,
                                                StoreX store_x) {
  const int q = lane >> 4, c = lane & 15;
  // A and D_J^{-1} of the next chunk are requested before the current chunk's
  // product, so their latency hides behind it
  double av[8], dv[PW / 2];
  auto fetch = [&](int J0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int R = q + 4 * r;
      av[2 * r] = load_a((int64_t)(J0 + c) * ld + r0 + R);
      av[2 * r + 1] = load_a((int64_t)(J0 + c + 16) * ld + r0 + R);
    }
    const double* Di = dinv + (int64_t)(J0 / PW) * PW * PW;  // Di[kk * 32 + n] = D_J^{-1}[n][kk]
#pragma unroll
    for (int u = 0; u < PW / 4; ++u) {
      dv[2 * u] = Di[(4 * u + q) * PW + c];
      dv[2 * u + 1] = Di[(4 * u + q) * PW + 16 + c];
    }
  };
  fetch(c0);
#pragma unroll 1
  for (int J0 = c0; J0 < c1; J0 += PW) {
    double ca[8], cd[PW / 2];
#pragma unroll
    for (int e = 0; e < 8; ++e) ca[e] = av[e];
#pragma unroll
    for (int e = 0; e < PW / 2; ++e) cd[e] = dv[e];
    if (J0 + PW < c1) fetch(J0 + PW);
    d4 acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
    mfma_rows16x32(X, L, ld, r0, J0, c0, J0, lane, acc0, acc1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int R = q + 4 * r;
      Ts[R][c] = ca[2 * r] - acc0[r];
      Ts[R][c + 16] = ca[2 * r + 1] - acc1[r];
    }
    __builtin_amdgcn_wave_barrier();
    d4 x0 = {0, 0, 0, 0}, x1 = {0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < PW / 4; ++u) {
      const int kk = 4 * u + q;
      const double a = Ts[c][kk];
      x0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, cd[2 * u], x0, 0, 0, 0);
      x1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, cd[2 * u + 1], x1, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t i0 = (int64_t)(J0 + c) * ld + r0 + q + 4 * r;
      store_x(i0, x0[r]);
      store_x(i0 + 16 * ld, x1[r]);
    }
    __threadfence_block();
    __builtin_amdgcn_wave_barrier();
  }
}

// ---------------------------------------------------------------------------
// Blocked POTRF of the FP64 diagonal tile k, spread over several workgroups:
// the tile is split into SB x SB blocks and, for each block column j,
//   (a) k_potrf_block  one workgroup factors the diagonal block D_jj and
//                      inverts its four 32 x 32 diagonal blocks into dinv for
//                      the solves below,
//   (b) k_potrf_panel  the rows below solve X D_jj^T = A, one workgroup per
//                      16 rows (solve_rows16),
//   (c) k_potrf_syrk   the lower trailing part loses L_{:,j} L_{:,j}^T
//                      (FP64 MFMA).
// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
// Triangular solves X L^T = A for 16 rows over 128 T columns (T <= 4), right-
// looking, by eight waves.  Column tile ct (16 wide) belongs to wave ct % 8, so
// that a 32-column chunk J belongs to one pair of waves; per chunk
//   (1) its pair forms T = A - acc and exchanges the two halves,
//   (2) each of the two multiplies T by its half of the inverted diagonal block
//       (X_J = T D_J^{-T}) and publishes it; meanwhile the other waves subtract
//       the earlier chunks from their own tiles,
//   (3) the next chunk's pair subtracts X_J first, which leads to its (1).
// Two barriers per chunk.  All products are formed transposed (the fragment of L
// or of D_J^{-1} first): a lane's results are then the operands of the next
// product, so T and X_J pass through LDS register by register without a layout
// change, and loads and stores touch 16 consecutive rows.  What is read from
// memory (L, D_J^{-1}, A) is requested one step ahead; nothing solved is read
// back from memory.  load_a(e, own) and store_x(e, own, v) take element e + own of
// the rows' column-major storage (leading dimension ld), e uniform in the wave.
// Every tile's products are added in ascending k.  QUARTERS: as four sums over
// the quarters of its contraction, added in order.
// Bound: the chain of (1) .. (3), sixteen dependent MFMAs and two exchanges per
// chunk.  At most 128 VGPRs and 86 KB of LDS, so that a workgroup fits where one
// of a tile update's retires.  Measured, one launch alone, against a left-looking
// solve that read X back from memory chunk by chunk: 3 panel tiles of 256 38 ->
// 18 us, 128 columns of the diagonal tile 15 -> 7.5 us, inverse of a 256 tile
// 48 -> 17 us.
// ---------------------------------------------------------------------------
// the element a 32-bit number of bytes behind a uniform address (one address register per lane)
template <class E>
__device__ __forceinline__ E& at(E* p, unsigned bytes) {
  return *(E*)((char*)p + bytes);
}

// a tile's address in scalar registers
__device__ __forceinline__ char* uniform_tile(const TileView& tv, int i, int j) {
  const uint64_t o = (uint64_t)tv.off[tri_index(i, j)];
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)o), hi = __builtin_amdgcn_readfirstlane((int)(o >> 32));
  return (char*)tv.base + (int64_t)((uint64_t)hi << 32 | lo);
}

template <int T, bool QUARTERS>
struct SolveLds {
  double X[4][8][64];      // chunk % 4 (a wave lags at most two behind), k step, lane
  double t[2][4][64];      // half of the chunk, register, lane
  double sum[QUARTERS ? 8 * T : 1][4][64];  // column tile's finished quarters
};

template <int T, bool QUARTERS, class LoadA, class StoreX>
__device__ __forceinline__ void solve_rows16(const double* L, int ld, const double* dinv, SolveLds<T, QUARTERS>& sm,
                                             LoadA load_a, StoreX store_x) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pair = wave >> 1, h = wave & 1, q = lane >> 4, i = lane & 15;
  const unsigned own = q * ld + i;  // the lane's element behind a uniform address
  d4 cur[T];
  int bound[T];
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int t = 0; t < T; ++t) {
    cur[t] = d4{0, 0, 0, 0};
    bound[t] = 8 * (4 * t + pair);
    if (QUARTERS) {
#pragma unroll
      for (int r = 0; r < 4; ++r) sm.sum[8 * t + wave][r][lane] = 0.0;
    }
  }
  auto load_l = [&](double (&v)[8], int t, int p) {  // the fragment of tile t's rows of L at chunk p
    const double* o = L + (int64_t)(32 * p) * ld + 16 * (8 * t + wave);
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = at(o + (int64_t)(4 * u) * ld, 8 * own);
  };
  // cur[t] += the product with chunk p
  auto apply = [&](auto tt, const double (&l)[8], int p) {
    constexpr int t = decltype(tt)::value;
    double x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = sm.X[p & 3][u][lane];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (QUARTERS && u % 2 == 0 && 32 * p + 4 * u == bound[t]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) sm.sum[8 * t + wave][r][lane] += cur[t][r];
        cur[t] = d4{0, 0, 0, 0};
        bound[t] += 8 * (4 * t + pair);
      }
      cur[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(l[u], x[u], cur[t], 0, 0, 0);
    }
  };
  int J = 0;     // the chunk being solved
  int done = 0;  // chunks subtracted from all of the wave's tiles
  // The wave's part of n chunks that are not its own: the earlier chunks are
  // subtracted from its tiles FIRST .. T - 1 in turn, the next one's fragment in
  // flight.
  auto others = [&](auto ff, int n) {
    constexpr int FIRST = decltype(ff)::value;
#pragma unroll 1
    for (; n > 0; --n) {
      __syncthreads();
      if constexpr (FIRST < T) {
        double l[8];
        if (done < J) load_l(l, FIRST, done);
#pragma unroll 1
        for (; done < J; ++done) {
          auto step = [&](auto ss) {
            constexpr int s = decltype(ss)::value;
            if constexpr (s >= FIRST && s < T) {
              double now[8];
#pragma unroll
              for (int u = 0; u < 8; ++u) now[u] = l[u];
              if (s + 1 < T) load_l(l, s + 1, done);
              else if (done + 1 < J) load_l(l, FIRST, done + 1);
              apply(ss, now, done);
            }
          };
          step(std::integral_constant<int, 0>{});
          step(std::integral_constant<int, 1>{});
          step(std::integral_constant<int, 2>{});
          step(std::integral_constant<int, 3>{});
        }
      }
      if (n > 1) {  // (the last one's second barrier comes behind what the caller requests)
        __syncthreads();
        ++J;
      }
    }
  };
  // the chunks between the wave's chunks 4 (t - 1) + pair and 4 t + pair, and its own
  auto group = [&](auto tt) {
    constexpr int t = decltype(tt)::value;
    double dv[8], av[4];
    auto fetch = [&] {
      const double* Di = dinv + (4 * t + pair) * PW * PW + 16 * h;
#pragma unroll
      for (int u = 0; u < 8; ++u) dv[u] = at(Di + 4 * u * PW, 8 * (unsigned)(q * PW + i));
#pragma unroll
      for (int r = 0; r < 4; ++r) av[r] = load_a((int64_t)(16 * (8 * t + wave) + 4 * r) * ld, own);
    };
    const int between = t > 0 ? 3 : pair;
    if (between > 0) {
      others(tt, between);
      double l[8];
      load_l(l, t, J);
      __syncthreads();
      __builtin_amdgcn_s_setprio(3);
      fetch();
      apply(tt, l, J);
      ++J;
    } else {
      fetch();
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) sm.t[h][r][lane] = av[r] - (QUARTERS ? sm.sum[8 * t + wave][r][lane] + cur[t][r] : cur[t][r]);
    __syncthreads();
    d4 x = {0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < 8; ++u) x = __builtin_amdgcn_mfma_f64_16x16x4f64(dv[u], sm.t[u >> 2][u & 3][lane], x, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) sm.X[J & 3][4 * h + r][lane] = x[r];
    __builtin_amdgcn_s_setprio(1);
    __syncthreads();
    ++J;
#pragma unroll
    for (int r = 0; r < 4; ++r) store_x((int64_t)(16 * (8 * t + wave) + 4 * r) * ld, own, x[r]);
  };
  group(std::integral_constant<int, 0>{});
  if constexpr (T > 1) group(std::integral_constant<int, 1>{});
  if constexpr (T > 2) group(std::integral_constant<int, 2>{});
  if constexpr (T > 3) group(std::integral_constant<int, 3>{});
  if (pair < 3) {
    others(std::integral_constant<int, T>{}, 3 - pair);
    __syncthreads();
  }
}

// rows c1 .. nb of block column j: X D_jj^T = A in place, 16 rows per workgroup
__global__ __launch_bounds__(512, 4) void k_potrf_panel(TileView tv, int k, int j, const double* dinv) {
  if (*tv.info) return;
  const int nb = tv.nb, c0 = j * SB;
  double* D = (double*)uniform_tile(tv, k, k) + (int64_t)c0 * nb + c0;  // the factored diagonal block
  double* A = D + SB + blockIdx.x * 16;                        // these rows
  __shared__ SolveLds<1, false> sm;
  solve_rows16<1, false>(D, nb, dinv + (int64_t)c0 * PW, sm, [&](int64_t e, unsigned own) { return at(A + e, 8 * own); },
                         [&](int64_t e, unsigned own, double v) { at(A + e, 8 * own) = v; });
}

// C[R, C] -= P[R, 0:K] P[C, 0:K]^T over the lower triangle of a matrix: half of a
// 32 x 32 block on or below the diagonal per workgroup, four waves, two per 16 x
// 16 tile, each over one half of the contraction; the second half's sums are
// added to the first's through LDS.  These updates sit on the critical path and
// occupy few CUs, so the blocks are small and the contraction is split: a wave's
// chain is K / 8 dependent MFMAs.  Operands come straight from memory, 32 k per
// batch with the next batch's loads in flight.  Four waves of at most 128 VGPRs
// fit wherever a workgroup of a tile update retires; with eight, or more VGPRs,
// they wait for the whole update.  Measured alone, before (64 x 64 blocks, eight
// waves) and after: K = 128, 128 rows 13 -> 4.2 us; a 256 tile, K = 256, 20 -> 5.6 us.
constexpr int SYRK_WGS = 2;  // workgroups per 32 x 32 block
__device__ __forceinline__ void syrk_block32(const double* P, double* C, int ld, int K, double (*red)[4][64]) {
  __builtin_amdgcn_s_setprio(2);
  int bi = 0, rem = blockIdx.x / SYRK_WGS;
  while (rem > bi) { rem -= bi + 1; ++bi; }
  const int bj = rem;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = wave & 1, kh = wave >> 1, q = lane >> 4, i = lane & 15;
  const int R0 = bi * 32 + 16 * tile, C0 = bj * 32 + 16 * (blockIdx.x % SYRK_WGS);
  const bool live = R0 >= C0;
  d4 acc = {0, 0, 0, 0};
  double old[4];
  if (live) {
    const unsigned own = 8 * (q * ld + i);
    const double* a = P + (int64_t)(kh * (K / 2)) * ld + R0;
    const double* b = P + (int64_t)(kh * (K / 2)) * ld + C0;
    if (kh == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) old[r] = at(C + (int64_t)(C0 + 4 * r) * ld + R0, own);
    }
    double va[2][8], vb[2][8];
    auto load = [&](int s) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        va[s][u] = at(a + (int64_t)(4 * u) * ld, own);
        vb[s][u] = at(b + (int64_t)(4 * u) * ld, own);
      }
      a += (int64_t)32 * ld;
      b += (int64_t)32 * ld;
    };
    auto product = [&](int s) {
#pragma unroll
      for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(vb[s][u], va[s][u], acc, 0, 0, 0);
    };
    load(0);
    load(1);
    for (int n = 0; n < K / 128; ++n) {  // 64 k of this half
      product(0);
      if (n + 1 < K / 128) load(0);
      product(1);
      if (n + 1 < K / 128) load(1);
    }
    if (kh == 1) {
#pragma unroll
      for (int r = 0; r < 4; ++r) red[tile][r][lane] = acc[r];
    }
  }
  __syncthreads();
  if (live && kh == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = C0 + q + 4 * r;
      if (R0 + i >= c) C[(int64_t)c * ld + R0 + i] = old[r] - (acc[r] + red[tile][r][lane]);
    }
  }
}

// the trailing part of the diagonal tile k behind block column j
__global__ __launch_bounds__(256, 4) void k_potrf_syrk(TileView tv, int k, int j) {
  if (*tv.info) return;
  const int nb = tv.nb, c0 = j * SB, c1 = c0 + SB;
  double* A = (double*)tv.tile(k, k);
  __shared__ double red[2][4][64];
  syrk_block32(A + (int64_t)c0 * nb + c1, A + (int64_t)c1 * nb + c1, nb, SB, red);
}

// A_jj -= L_jk L_jk^T for one diagonal tile with an FP64 panel tile
__global__ __launch_bounds__(256, 4) void k_syrk_tile(TileView tv, int k, int j) {
  if (*tv.info) return;
  __shared__ double red[2][4][64];
  syrk_block32((const double*)tv.tile(j, k), (double*)tv.tile(j, j), tv.nb, tv.nb, red);
}

hipError_t launch_syrk_tile(const TileView& tv, int k, int j, hipStream_t s) {
  const int nbk = tv.nb / 32;
  k_syrk_tile<<<SYRK_WGS * nbk * (nbk + 1) / 2, 256, 0, s>>>(tv, k, j);
  return hipGetLastError();
}

hipError_t launch_potrf_tile(const TileView& tv, int k, double* dinv, hipStream_t s) {
  const int nsb = tv.nb / SB;
  for (int j = 0; j < nsb; ++j) {
    if (const hipError_t e = launch_potrf_block(tv, k, j, dinv, s); e != hipSuccess) return e;
    const int rest = (tv.nb - (j + 1) * SB) / 32;  // 32-row blocks below block j
    if (rest > 0) {
      k_potrf_panel<<<rest * 2, 512, 0, s>>>(tv, k, j, dinv);
      k_potrf_syrk<<<SYRK_WGS * rest * (rest + 1) / 2, 256, 0, s>>>(tv, k, j);
    }
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Panel TRSM: for i > k, X = A_ik L_kk^{-T} in FP64, rounded once to p(i,k).
// Tiles above 512: one wave per 16 rows of a panel tile (trsm_rows16_inv with the
// inverted diagonal blocks of L_kk from its POTRF); the FP64 X goes to the
// workspace ws ((nt-k-1) tiles of nb x nb) and the tile receives one rounding of
// it.  Smaller ones: k_trsm_rows below.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_trsm(TileView tv, int k, double* ws, const double* dinv) {
  if (*tv.info) return;
  const int nb = tv.nb, rblocks = nb / 16;
  const int ti = k + 1 + blockIdx.x / rblocks;
  const int r0 = (blockIdx.x % rblocks) * 16;
  void* Ap = tv.tile(ti, k);
  const int fa = tv.tfmt(ti, k);
  const double ma = tv.tmul(ti, k);
  double* X = ws + (int64_t)(ti - k - 1) * nb * nb;
  __shared__ double Ts[16][PW + 1];
  // FP8 tiles are rounded by k_quant_panel_f8 once the whole tile's largest magnitude is known
  trsm_rows16_inv(X, (const double*)tv.tile(k, k), nb, dinv, 0, nb, r0, Ts, threadIdx.x,
                  [&](int64_t i) { return load_wide(Ap, fa, i) * ma; },
                  [&](int64_t i, double v) {
                    X[i] = v;
                    if (fa != F8) store_round(Ap, fa, i, v);
                  });
}

// FP8 panel tiles after k_trsm: scale from the solved tile's largest magnitude,
// then one rounding of every value (one workgroup per panel tile)
__global__ __launch_bounds__(256) void k_quant_panel_f8(TileView tv, int k, const double* ws) {
  const int ti = k + 1 + blockIdx.x;
  if (*tv.info || tv.tfmt(ti, k) != F8) return;
  const int nb = tv.nb;
  const double* X = ws + (int64_t)blockIdx.x * nb * nb;
  __shared__ double red[256];
  double m = 0.0;
  for (int64_t e = threadIdx.x; e < (int64_t)nb * nb; e += 256) m = fmax(m, fabs(X[e]));
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  const int sc = fp8_scale_exp(red[0]);
  uint8_t* P = (uint8_t*)tv.tile(ti, k);
  for (int64_t e = threadIdx.x; e < (int64_t)nb * nb; e += 256) P[e] = to_e4m3(ldexp(X[e], sc));
  if (threadIdx.x == 0) tv.sc[tri_index(ti, k)] = (int8_t)sc;
}

// The same panel solve with four waves per 16 rows, for steps with few panel
// tiles, where the solve sits alone on the critical path: the update of every
// 32-column chunk is split over the waves by quarters of its contraction
// (their partial products added in wave order through LDS), and wave 0 forms
// the chunk's columns with the inverted diagonal block.  Two barriers per
// chunk; the chunk's columns reach the other waves through global memory
// after a workgroup-scope fence.
constexpr int TRSM_SPLIT_MAX = 32;  // panel tiles up to which the split solve is used

__global__ __launch_bounds__(256) void k_trsm4(TileView tv, int k, double* ws, const double* dinv) {
  if (*tv.info) return;
  const int nb = tv.nb, rblocks = nb / 16;
  const int ti = k + 1 + blockIdx.x / rblocks;
  const int r0 = (blockIdx.x % rblocks) * 16;
  void* Ap = tv.tile(ti, k);
  const int fa = tv.tfmt(ti, k);
  const double ma = tv.tmul(ti, k);
  double* X = ws + (int64_t)(ti - k - 1) * nb * nb;
  const double* L = (const double*)tv.tile(k, k);
  __shared__ double red[4][16][PW + 1];
  __shared__ double Ts[16][PW + 1];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int q = lane >> 4, c = lane & 15;
#pragma unroll 1
  for (int J0 = 0; J0 < nb; J0 += PW) {
    const int part = J0 / 4;  // a multiple of 8
    d4 acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
    mfma_rows16x32(X, L, nb, r0, J0, w * part, (w + 1) * part, lane, acc0, acc1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      red[w][q + 4 * r][c] = acc0[r];
      red[w][q + 4 * r][c + 16] = acc1[r];
    }
    __syncthreads();
    if (w == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int R = q + 4 * r;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int cc = c + 16 * h;
          const double a = load_wide(Ap, fa, (int64_t)(J0 + cc) * nb + r0 + R) * ma;
          Ts[R][cc] = a - (((red[0][R][cc] + red[1][R][cc]) + red[2][R][cc]) + red[3][R][cc]);
        }
      }
      __builtin_amdgcn_wave_barrier();
      const double* Di = dinv + (int64_t)(J0 / PW) * PW * PW;  // Di[kk * 32 + n] = D_J^{-1}[n][kk]
      d4 x0 = {0, 0, 0, 0}, x1 = {0, 0, 0, 0};
#pragma unroll
      for (int u = 0; u < PW / 4; ++u) {
        const int kk = 4 * u + q;
        const double a = Ts[c][kk];
        x0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Di[kk * PW + c], x0, 0, 0, 0);
        x1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Di[kk * PW + 16 + c], x1, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t i0 = (int64_t)(J0 + c) * nb + r0 + q + 4 * r;
        X[i0] = x0[r];
        X[i0 + 16 * nb] = x1[r];
        // FP8 tiles are rounded by k_quant_panel_f8 once the whole tile's largest magnitude is known
        if (fa != F8) {
          store_round(Ap, fa, i0, x0[r]);
          store_round(Ap, fa, i0 + 16 * nb, x1[r]);
        }
      }
      __threadfence_block();
    }
    __syncthreads();
  }
}

// ... for tiles of up to 512: one workgroup per 16 rows (solve_rows16).  The FP64 X
// goes to ws only for FP8 tiles, which k_quant_panel_f8 rounds from it.
template <int T, bool QUARTERS>
__global__ __launch_bounds__(512, 4) void k_trsm_rows(TileView tv, int k, double* ws, const double* dinv) {
  if (*tv.info) return;
  const int nb = tv.nb, rblocks = nb / 16;
  const int ti = k + 1 + blockIdx.x / rblocks;
  const int r0 = (blockIdx.x % rblocks) * 16;
  const int fa = __builtin_amdgcn_readfirstlane(tv.tfmt(ti, k)), es = fmt_bytes(fa);
  char* Ap = uniform_tile(tv, ti, k) + r0 * es;
  const double ma = tv.tmul(ti, k);
  double* X = ws + (int64_t)(ti - k - 1) * nb * nb + r0;
  extern __shared__ __attribute__((aligned(16))) char solve_lds[];
  solve_rows16<T, QUARTERS>((const double*)uniform_tile(tv, k, k), nb, dinv, *(SolveLds<T, QUARTERS>*)solve_lds,
                            [&](int64_t e, unsigned own) { return load_wide(&at(Ap + e * es, own * es), fa, 0) * ma; },
                            [&](int64_t e, unsigned own, double v) {
                              if (fa == F8) at(X + e, 8 * own) = v;
                              else store_round(&at(Ap + e * es, own * es), fa, 0, v);
                            });
}

hipError_t launch_trsm_panel(const TileView& tv, int k, double* ws, const double* dinv, bool fp8_panel,
                             hipStream_t s) {
  int ntile = tv.nt - k - 1;
  if (ntile <= 0) return hipSuccess;
  const bool split = ntile <= TRSM_SPLIT_MAX;
  const int grid = ntile * (tv.nb / 16);
#define MPCR_TRSM(T)                                                                               \
  case T:                                                                                          \
    if (split) k_trsm_rows<T, true><<<grid, 512, sizeof(SolveLds<T, true>), s>>>(tv, k, ws, dinv);      \
    else k_trsm_rows<T, false><<<grid, 512, sizeof(SolveLds<T, false>), s>>>(tv, k, ws, dinv);    \
    break
  switch (tv.nb / 128) {
    MPCR_TRSM(1);
    MPCR_TRSM(2);
    MPCR_TRSM(3);
    MPCR_TRSM(4);
    default:
      if (split) k_trsm4<<<grid, 256, 0, s>>>(tv, k, ws, dinv);
      else k_trsm<<<grid, 64, 0, s>>>(tv, k, ws, dinv);
  }
#undef MPCR_TRSM
  if (fp8_panel) k_quant_panel_f8<<<ntile, 256, 0, s>>>(tv, k, ws);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Inverted diagonal tiles for the solves.  Row r of X = L_kk^{-T} (X L^T = I) is
// column r of L_kk^{-1}, so trsm_rows16_inv applied to the identity, one wave
// per 16 rows, gives L_kk^{-1} stored by rows (its transpose in column-major
// order) from the 32 x 32 block inverses that the tile's POTRF left in dinv;
// entries left of the rows' own 32-column chunk are zero.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_trtri(TileView tv, double* Linv, const double* dinv) {
  if (*tv.info) return;
  const int nb = tv.nb, rb = nb / 16;
  const int kt = blockIdx.x / rb, r0 = (blockIdx.x % rb) * 16;
  const int c0 = (r0 / PW) * PW;
  double* X = Linv + (int64_t)kt * nb * nb;
  __shared__ double Ts[16][PW + 1];
  const int lane = threadIdx.x;
  for (int e = lane; e < 16 * c0; e += 64) X[(int64_t)(e / 16) * nb + r0 + e % 16] = 0.0;
  trsm_rows16_inv(X, (const double*)tv.tile(kt, kt), nb, dinv + (int64_t)kt * nb * PW, c0, nb, r0, Ts, lane,
                  [&](int64_t i) { return (i % nb) == (i / nb) ? 1.0 : 0.0; }, [&](int64_t i, double v) { X[i] = v; });
}

// ... for tiles of up to 512 (solve_rows16)
template <int T>
__global__ __launch_bounds__(512, 4) void k_trtri_rows(TileView tv, double* Linv, const double* dinv) {
  if (*tv.info) return;
  const int nb = tv.nb, rb = nb / 16;
  const int kt = blockIdx.x / rb, r0 = (blockIdx.x % rb) * 16;
  double* X = Linv + (int64_t)kt * nb * nb;
  const int64_t diag = (int64_t)(r0 + (threadIdx.x & 15)) * nb + (threadIdx.x & 15);  // this lane's row's one
  extern __shared__ __attribute__((aligned(16))) char solve_lds[];
  solve_rows16<T, false>((const double*)uniform_tile(tv, kt, kt), nb, dinv + (int64_t)kt * nb * PW,
                         *(SolveLds<T, false>*)solve_lds, [&](int64_t e, unsigned own) { return e + own == diag ? 1.0 : 0.0; },
                         [&](int64_t e, unsigned own, double v) { at(X + r0 + e, 8 * own) = v; });
}

hipError_t launch_trtri_diag(const TileView& tv, double* Linv, const double* dinv, hipStream_t s) {
  const int grid = tv.nt * (tv.nb / 16);
  switch (tv.nb / 128) {
    case 1: k_trtri_rows<1><<<grid, 512, sizeof(SolveLds<1, false>), s>>>(tv, Linv, dinv); break;
    case 2: k_trtri_rows<2><<<grid, 512, sizeof(SolveLds<2, false>), s>>>(tv, Linv, dinv); break;
    case 3: k_trtri_rows<3><<<grid, 512, sizeof(SolveLds<3, false>), s>>>(tv, Linv, dinv); break;
    case 4: k_trtri_rows<4><<<grid, 512, sizeof(SolveLds<4, false>), s>>>(tv, Linv, dinv); break;
    default: k_trtri<<<grid, 64, 0, s>>>(tv, Linv, dinv);
  }
  return hipGetLastError();
}

}  // namespace mpcr
