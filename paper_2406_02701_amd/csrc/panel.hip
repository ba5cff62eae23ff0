// Diagonal block factorisation of the tile Cholesky (gfx950).
//
// k_potrf_block factors one 128 x 128 block on the diagonal of an FP64 tile
// with one workgroup.  It sits alone on the critical path of every
// factorisation, so it is built for latency, not for flops (the block's
// 0.7 MFLOP are 2.3 us of one CU's FP64 MFMA rate).
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
      __builtin_amdgcn_s_setprio(0);
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

}  // namespace mpcr
