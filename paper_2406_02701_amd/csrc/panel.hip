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

// 1 / sqrt(d) for d > 0 (normal): the hardware estimate y, then one step of
// third order, y (1 + e/2 + 3/8 e^2) with e = 1 - d y^2 (the series of
// (1 - e)^(-1/2)), whose relative error is about 5/16 e^3: an estimate good to
// 2^-18 or better ends within a few units in the last place.  Four dependent
// operations, where two Newton steps take six.
__device__ __forceinline__ double rsqrt_f64(double d) {
  const double y = __builtin_amdgcn_rsq(d);
  const double e = fma(-d * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// Column steps with lane N of every 16-lane row broadcast to that row inside
// the operation (DPP row_newbcast; no trip through scalar registers).  A DPP
// operand must have been written two wait states before its use: every block
// sees to that itself.
//   fma2_bcast<Q>   d[q] -= d_C[q] d_C,  x[q] -= d_C[q] x_C  for q = Q .. 15
//                   (s = d_C, t = x_C; d_C[q] is lane q's value)
template <int Q>
__device__ __forceinline__ void fma2_bcast(double (&d)[PB], double (&x)[PB], double s, double t) {
  if constexpr (Q + 5 <= PB) {
    asm volatile(
        "s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%10, %10 row_newbcast:%c12 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %5, -%10, %11 row_newbcast:%c12 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, -%10, %10 row_newbcast:%c13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %6, -%10, %11 row_newbcast:%c13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, -%10, %10 row_newbcast:%c14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %7, -%10, %11 row_newbcast:%c14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, -%10, %10 row_newbcast:%c15 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %8, -%10, %11 row_newbcast:%c15 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %4, -%10, %10 row_newbcast:%c16 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %9, -%10, %11 row_newbcast:%c16 row_mask:0xf bank_mask:0xf"
        : "+v"(d[Q]), "+v"(d[Q + 1]), "+v"(d[Q + 2]), "+v"(d[Q + 3]), "+v"(d[Q + 4]), "+v"(x[Q]), "+v"(x[Q + 1]), "+v"(x[Q + 2]), "+v"(x[Q + 3]), "+v"(x[Q + 4])
        : "v"(s), "v"(t), "n"(Q), "n"(Q + 1), "n"(Q + 2), "n"(Q + 3), "n"(Q + 4));
    fma2_bcast<Q + 5>(d, x, s, t);
  } else if constexpr (Q + 2 <= PB) {
    asm volatile(
        "s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%4, %4 row_newbcast:%c6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, -%4, %5 row_newbcast:%c6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, -%4, %4 row_newbcast:%c7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, -%4, %5 row_newbcast:%c7 row_mask:0xf bank_mask:0xf"
        : "+v"(d[Q]), "+v"(d[Q + 1]), "+v"(x[Q]), "+v"(x[Q + 1])
        : "v"(s), "v"(t), "n"(Q), "n"(Q + 1));
    fma2_bcast<Q + 2>(d, x, s, t);
  } else if constexpr (Q + 1 <= PB) {
    asm volatile(
        "s_nop 1\n\t"
        "v_fmac_f64_dpp %0, -%2, %2 row_newbcast:%c4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, -%2, %3 row_newbcast:%c4 row_mask:0xf bank_mask:0xf"
        : "+v"(d[Q]), "+v"(x[Q])
        : "v"(s), "v"(t), "n"(Q));
    fma2_bcast<Q + 1>(d, x, s, t);
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
// block with the solve of 64 rows below it: d[c] is element c of row lane % 16
// of the block (every 16-lane row of the wave holds a copy), x[c] element c of
// this lane's row below.  The rows below are solved by the same column steps
// that factor the block.  Elements above the diagonal are carried along and
// never used.  r is 1 / sqrt of column C's pivot; the next pivot and its
// reciprocal square root come first in a column, so that their latency lies
// behind the column's other updates, and no branch separates the columns.  A
// pivot that is not positive (or infinite) makes r and everything after it
// NaN, which the last r, returned, shows.  TRACK: bad collects the columns
// whose pivot is not positive as bits.
template <int C, bool TRACK>
__device__ __forceinline__ double factor_rows16(double (&d)[PB], double (&x)[PB], double r, uint32_t& bad) {
  if constexpr (C + 1 < PB) {
    const double piv = column<C>(d, x, r);
    const double rn = rsqrt_f64(piv);
    if (TRACK) bad |= (uint32_t)(__builtin_amdgcn_ballot_w64(!(piv > 0.0)) & 1u) << (C + 1);
    fma2_bcast<C + 2>(d, x, d[C], x[C]);
    return factor_rows16<C + 1, TRACK>(d, x, rn, bad);
  } else {
    d[C] *= r;
    x[C] *= r;
    return r;
  }
}

struct PotrfLds {
  double L[NP * (NP + 1) / 2][PB][BLD];  // the lower 16 x 16 blocks
  double Di[4][PB][BLD];                 // inverses of the factored diagonal blocks p (slot p % 4)
  int fail;
};

// The block's 36 lower 16 x 16 blocks live in LDS.  Per 16-column panel p:
//   (1) one or two waves factor it: each holds the diagonal block (p, p) and 64
//       rows to be solved with it (the factorisation of the diagonal block is
//       repeated in both, which needs no exchange between them).  The rows are
//       those of the panel below and, behind them, the 16 rows of a unit
//       matrix, whose solution is the inverse of the diagonal block.
//       Meanwhile the other waves finish the trailing update with panel p - 1
//       and store that panel;
//   (2) the blocks of column p + 1, the next panel, lose panel p's product
//       (FP64 MFMA, one wave each).
// Two barriers per panel; the chain per panel is the sixteen columns of (1)
// (about 150 cycles each, nearly all of it instruction issue) and one block
// product of (2).  Measured alone: 23 us a block (87 us for a version that
// inverted each diagonal block and solved the panel by MFMA afterwards).  dinv receives the inverses of the four 32 x 32 diagonal blocks,
// [[A', 0], [-C' B A', C']] from the 16 x 16 ones.  Nothing above the diagonal
// is written (no kernel reads it).
// 87 KB of LDS and at most 128 VGPRs: with the tile updates resident on every
// CU (two workgroups of 74 KB), it fits as soon as one of them retires.  (The
// LDS is given at the launch: counted by the compiler, it would make it spend
// 256 VGPRs.)
__global__ __launch_bounds__(512, 4) void k_potrf_block(TileView tv, int k, int j, double* dinv) {
  const int info0 = *tv.info;
  const int nb = tv.nb, c0 = j * SB;
  double* A = (double*)tv.tile(k, k) + (int64_t)c0 * nb + c0;
  extern __shared__ __attribute__((aligned(16))) char potrf_lds[];
  PotrfLds& sm = *(PotrfLds*)potrf_lds;
  auto& L = sm.L;
  auto& Di = sm.Di;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane >> 4, lc = lane & 15;  // MFMA result: rows lr + 4 r, column lc

  // load: one wave per column, two rows per lane (column pieces of 1 KB); the
  // info word is looked at only once these loads are on their way
  {
    double2 v[SB / 8];
    const int bi = lane >> 3, r = 2 * (lane & 7);
#pragma unroll
    for (int g = 0; g < SB / 8; ++g) {
      const int c = wave + 8 * g;
      if (bi >= c / PB) v[g] = *(const double2*)(A + (int64_t)c * nb + 2 * lane);
    }
    if (info0) return;
    if (tid == 0) sm.fail = 0;
#pragma unroll
    for (int g = 0; g < SB / 8; ++g) {
      const int c = wave + 8 * g, bj = c / PB;
      if (bi >= bj) {
        L[tri_blk(bi, bj)][r][c % PB] = v[g].x;
        L[tri_blk(bi, bj)][r + 1][c % PB] = v[g].y;
      }
    }
  }
  __syncthreads();

  // blocks (bi, bj) -= L(bi, p) L(bj, p)^T for the N given blocks
  auto update = [&](auto ntag, const int (&bi)[2], const int (&bj)[2], int p) {
    constexpr int N = decltype(ntag)::value;
    d4 acc[N];
    double a[N][4], b[N][4];
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        a[n][u] = -L[tri_blk(bi[n], p)][lc][4 * u + lr];
        b[n][u] = L[tri_blk(bj[n], p)][lc][4 * u + lr];
        acc[n][u] = L[tri_blk(bi[n], bj[n])][lr + 4 * u][lc];
      }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int n = 0; n < N; ++n) acc[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[n][u], b[n][u], acc[n], 0, 0, 0);
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
      for (int u = 0; u < 4; ++u) L[tri_blk(bi[n], bj[n])][lr + 4 * u][lc] = acc[n][u];
  };
  constexpr std::integral_constant<int, 1> one{};
  constexpr std::integral_constant<int, 2> two{};

#pragma unroll 1
  for (int p = 0; p <= NP; ++p) {
    const int below = SB - PB * (p + 1);                 // rows below the diagonal block
    const int nw = p == NP ? 0 : below >= 64 ? 2 : 1;    // waves that factor the panel
    double d[PB], x[PB];
    const int t = wave * 64 + lane;                      // row below the diagonal block
    if (wave < nw) {
      __builtin_amdgcn_s_setprio(3);
      const double* drow = L[tri_blk(p, p)][lc];
      const double* row = L[tri_blk(p + (t < below ? 1 + t / PB : 0), p)][lc];
#pragma unroll
      for (int c = 0; c < PB; ++c) d[c] = drow[c];
#pragma unroll
      for (int c = 0; c < PB; ++c) x[c] = row[c];
      if (t >= below) {
#pragma unroll
        for (int c = 0; c < PB; ++c) x[c] = t - below == c ? 1.0 : 0.0;
      }
      uint32_t bad = 0;
      const double rl = factor_rows16<0, false>(d, x, rsqrt_f64(L[tri_blk(p, p)][0][0]), bad);
      if (!(rl > 0.0)) {  // (uniform) find the first column whose pivot is not positive
#pragma unroll
        for (int c = 0; c < PB; ++c) d[c] = drow[c];
        const double piv = L[tri_blk(p, p)][0][0];
        bad = __builtin_amdgcn_ballot_w64(!(piv > 0.0)) & 1u;
        factor_rows16<0, true>(d, x, rsqrt_f64(piv), bad);
        if (bad && tid == 0) {
          sm.fail = 1;
          *tv.info = k * nb + c0 + PB * p + __builtin_ctz(bad) + 1;
        }
      }
      if (t < below) {
        double* o = L[tri_blk(p + 1 + t / PB, p)][lc];
#pragma unroll
        for (int c = 0; c < PB; ++c) o[c] = x[c];
      } else if (t < below + PB) {
#pragma unroll
        for (int c = 0; c < PB; ++c) Di[p & 3][c][t - below] = x[c];
      }
      __builtin_amdgcn_s_setprio(0);
    } else if (p > 0) {
      // the inverted 32 x 32 block of the panels p - 2, p - 1 into dinv (column-major)
      if (wave == 7 && p % 2 == 0) {
        const double(*B)[BLD] = L[tri_blk(p - 1, p - 2)];
        const double(*A0)[BLD] = Di[(p - 2) & 3], (*C0)[BLD] = Di[(p - 1) & 3];
        d4 s = {0, 0, 0, 0}, m = {0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < 4; ++u) s = __builtin_amdgcn_mfma_f64_16x16x4f64(B[lc][4 * u + lr], A0[4 * u + lr][lc], s, 0, 0, 0);
        // the result layout of s (rows lr + 4 u) is the operand layout of its u-th k step
#pragma unroll
        for (int u = 0; u < 4; ++u) m = __builtin_amdgcn_mfma_f64_16x16x4f64(-C0[lc][4 * u + lr], s[u], m, 0, 0, 0);
        double* o = dinv + (int64_t)(c0 + PB * (p - 2)) * PW + lc * PW;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int R = lr + 4 * r;
          o[R] = R >= lc ? A0[R][lc] : 0.0;
          o[PB + R] = m[r];
          o[PB * PW + R] = 0.0;
          o[PB * PW + PB + R] = R >= lc ? C0[R][lc] : 0.0;
        }
      }
      // trailing blocks (bi, bj), p < bj <= bi, with panel p - 1
      const int m = NP - 1 - p, nblk = m * (m + 1) / 2, step = 8 - nw;
#pragma unroll 1
      for (int b = wave - nw; b < nblk; b += 2 * step) {
        int bi[2], bj[2];
        const bool both = b + step < nblk;
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          int i = 0, rem = n && both ? b + step : b;
          while (rem > i) { rem -= i + 1; ++i; }
          bi[n] = p + 1 + i;
          bj[n] = p + 1 + rem;
        }
        if (both) update(two, bi, bj, p - 1);
        else update(one, bi, bj, p - 1);
      }
      // panel p - 1 to memory: one wave per column, two rows per lane
      const int R = PB * (p - 1) + 2 * lane, rb = R < SB ? R / PB : 0;
      for (int c = wave - nw; c < PB; c += step) {
        const double v0 = L[tri_blk(rb >= p - 1 ? rb : p - 1, p - 1)][R % PB][c];
        const double v1 = L[tri_blk(rb >= p - 1 ? rb : p - 1, p - 1)][R % PB + 1][c];
        double* o = A + (int64_t)(PB * (p - 1) + c) * nb + R;
        if (R < SB && 2 * lane >= c) *(double2*)o = double2{v0, v1};
        else if (R < SB && 2 * lane + 1 == c) o[1] = v1;
      }
    }
    if (p == NP) break;
    __syncthreads();
    if (sm.fail) return;
    if (wave > 0 && p + wave < NP) {
      const int bi[2] = {p + wave, 0}, bj[2] = {p + 1, 0};
      update(one, bi, bj, p);
    }
    if (wave == 0) {
      // the factored diagonal block, only now that no wave reads the old one:
      // every 16-lane row stores four columns of its copy
#pragma unroll
      for (int c = 0; c < 4; ++c)
        L[tri_blk(p, p)][lc][4 * lr + c] = lr == 0 ? d[c] : lr == 1 ? d[4 + c] : lr == 2 ? d[8 + c] : d[12 + c];
    }
    __syncthreads();
  }
}

hipError_t launch_potrf_block(const TileView& tv, int k, int j, double* dinv, hipStream_t s) {
  k_potrf_block<<<1, 512, sizeof(PotrfLds), s>>>(tv, k, j, dinv);
  return hipGetLastError();
}

}  // namespace mpcr
