// Diagonal block factorisation of the tile Cholesky (gfx950).
//
// k_potrf_block factors one 128 x 128 block on the diagonal of an FP64 tile
// with one workgroup.  It sits alone on the critical path of every
// factorisation, so it is built for latency, not for flops (the block's
// 0.7 MFLOP are 2.3 us of one CU's FP64 MFMA rate).
#include "mpcr_internal.h"

namespace mpcr {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int SB = 128;  // diagonal block
constexpr int PB = 16;   // panel width inside it
constexpr int PW = 32;   // inverted diagonal blocks handed to the panel solves
constexpr int NP = SB / PB;
constexpr int BLD = PB + 1;  // LDS row of a 16 x 16 block (doubles)

__device__ __forceinline__ int tri_blk(int i, int j) { return i * (i + 1) / 2 + j; }

// 64-bit lane broadcast: the value v of lane src, read as a wave-uniform scalar.
__device__ __forceinline__ double lane_f64(double v, int src) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, src);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), src);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

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

// Sixteen columns of a right-looking Cholesky with one matrix row per lane:
// lanes 0..15 hold the rows of the 16 x 16 diagonal block, lanes 16..63 rows
// below it (x[c] = element c of the row), so the rows below are solved by the
// same operations that factor the block.  The elements above the diagonal are
// carried along and never used.  rs receives 1 / L[l][l] in lane l < 16.
// Returns the first column whose pivot is not positive, or -1.
__device__ __forceinline__ int factor_rows16(double (&x)[PB], int lane, double& rs) {
#pragma unroll
  for (int c = 0; c < PB; ++c) {
    const double d = lane_f64(x[c], c);
    if (!(d > 0.0)) return c;
    const double r = rsqrt_f64(d);
    rs = lane == c ? r : rs;
    const double lc = x[c] * r;
    x[c] = lc;
#pragma unroll
    for (int q = c + 1; q < PB; ++q) x[q] = fma(-lc, lane_f64(lc, q), x[q]);
  }
  return -1;
}

// The block's 36 lower 16 x 16 blocks live in LDS.  Per 16-column panel p:
//   (1) up to three waves factor it: every one of them holds the 16 rows of
//       the diagonal block (p, p) in lanes 0..15 and 48 rows below it in lanes
//       16..63 (the factorisation of the diagonal block is repeated in each,
//       which costs nothing and needs no exchange between waves); meanwhile
//       the other waves finish the trailing update with panel p - 1 and the
//       inverses of the diagonal blocks;
//   (2) all waves subtract panel p's product from the blocks of column p + 1
//       (FP64 MFMA), the next panel to be factored.
// Two barriers per panel; the chain per panel is the sixteen columns of (1)
// and one block product of (2).  dinv receives the inverses of the four
// 32 x 32 diagonal blocks, [[A', 0], [-C' B A', C']] from the 16 x 16 ones.
// 86 KB of LDS and at most 128 VGPRs: with the tile updates resident on every
// CU (two workgroups of 74 KB), it fits as soon as one of them retires.
__global__ __launch_bounds__(512) __attribute__((amdgpu_num_vgpr(128))) void k_potrf_block(TileView tv, int k, int j,
                                                                                           double* dinv) {
  if (*tv.info) return;
  const int nb = tv.nb, c0 = j * SB;
  double* A = (double*)tv.tile(k, k) + (int64_t)c0 * nb + c0;
  __shared__ __attribute__((aligned(16))) double L[NP * (NP + 1) / 2][PB][BLD];
  __shared__ double Dg[PB][BLD];     // the diagonal block that the panel's first wave has factored
  __shared__ double Di[2][PB][BLD];  // inverses of the diagonal blocks p (slot p % 2)
  __shared__ double Dr[SB];          // 1 / L[c][c]
  __shared__ int fail;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane >> 4, lc = lane & 15;  // MFMA result: rows lr + 4 r, column lc
  if (tid == 0) fail = 0;

  // load: one wave per column, two rows per lane (column pieces of 1 KB)
  {
    double2 v[SB / 8];
    const int bi = lane >> 3, r = 2 * (lane & 7);
#pragma unroll
    for (int g = 0; g < SB / 8; ++g) {
      const int c = wave + 8 * g;
      if (bi >= c / PB) v[g] = *(const double2*)(A + (int64_t)c * nb + 2 * lane);
    }
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

  // block (bi, bj) -= L(bi, p) L(bj, p)^T
  auto update = [&](int bi, int bj, int p) {
    double(*C)[BLD] = L[tri_blk(bi, bj)];
    const double(*P)[BLD] = L[tri_blk(bi, p)];
    const double(*Q)[BLD] = L[tri_blk(bj, p)];
    double a[4], b[4];
    d4 acc;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = C[lr + 4 * r][lc];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = -P[lc][4 * u + lr];
      b[u] = Q[lc][4 * u + lr];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) C[lr + 4 * r][lc] = acc[r];
  };
  // Di[p % 2] = L(p, p)^{-1}, column `lane` by forward substitution (one wave)
  auto invert16 = [&](int p) {
    const double(*D)[BLD] = L[tri_blk(p, p)];
    if (lane < PB) {
      double y[PB];
#pragma unroll
      for (int r = 0; r < PB; ++r) y[r] = r == lane ? 1.0 : 0.0;
#pragma unroll
      for (int r = 0; r < PB; ++r) {
        y[r] *= Dr[PB * p + r];
#pragma unroll
        for (int q = r + 1; q < PB; ++q) y[q] = fma(-D[q][r], y[r], y[q]);
      }
#pragma unroll
      for (int r = 0; r < PB; ++r) Di[p & 1][r][lane] = y[r];
    }
  };
  // the inverted 32 x 32 block of the panels p - 1, p (p odd) into dinv (column-major; one wave)
  auto invert32 = [&](int p) {
    const double(*B)[BLD] = L[tri_blk(p, p - 1)];
    d4 t = {0, 0, 0, 0}, m = {0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < 4; ++u) t = __builtin_amdgcn_mfma_f64_16x16x4f64(B[lc][4 * u + lr], Di[0][4 * u + lr][lc], t, 0, 0, 0);
    // the result layout of t (rows lr + 4 u) is the operand layout of its u-th k step
#pragma unroll
    for (int u = 0; u < 4; ++u) m = __builtin_amdgcn_mfma_f64_16x16x4f64(-Di[1][lc][4 * u + lr], t[u], m, 0, 0, 0);
    double* o = dinv + (int64_t)(c0 + PB * (p - 1)) * PW + lc * PW;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int R = lr + 4 * r;
      o[R] = Di[0][R][lc];
      o[PB + R] = m[r];
      o[PB * PW + R] = 0.0;
      o[PB * PW + PB + R] = Di[1][R][lc];
    }
  };

#pragma unroll 1
  for (int p = 0; p < NP; ++p) {
    const int below = SB - PB * (p + 1);                     // rows below the diagonal block
    const int nw = below > 96 ? 3 : below > 48 ? 2 : 1;      // waves that factor the panel
    if (wave < nw) {
      __builtin_amdgcn_s_setprio(3);
      const int t = wave * 48 + lane - PB;  // row below the diagonal block (lanes 16 ..)
      const bool live = lane < PB || t < below;
      double(*row)[BLD] = lane < PB ? L[tri_blk(p, p)] + lane : L[tri_blk(p + 1 + (live ? t : 0) / PB, p)] + (live ? t : 0) % PB;
      if (!live) row = L[tri_blk(p, p)];
      double x[PB], rs = 0.0;
#pragma unroll
      for (int c = 0; c < PB; ++c) x[c] = (*row)[c];
      const int bad = factor_rows16(x, lane, rs);
      if (bad >= 0) {
        if (tid == 0) {
          fail = 1;
          if (*tv.info == 0) *tv.info = k * nb + c0 + PB * p + bad + 1;
        }
      } else {
        if (lane >= PB && live) {
#pragma unroll
          for (int c = 0; c < PB; ++c) (*row)[c] = x[c];
        } else if (lane < PB && wave == 0) {  // (the other waves may still be reading block (p, p))
#pragma unroll
          for (int c = 0; c < PB; ++c) Dg[lane][c] = c <= lane ? x[c] : 0.0;
          Dr[PB * p + lane] = rs;
        }
      }
      __builtin_amdgcn_s_setprio(0);
    } else if (p > 0) {
      // trailing blocks (bi, bj), p < bj <= bi, with panel p - 1; the last wave
      // first inverts the diagonal block p - 1
      if (wave == 7) {
        invert16(p - 1);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if ((p - 1) & 1) invert32(p - 1);
      }
      const int m = NP - 1 - p, nblk = m * (m + 1) / 2;
      for (int b = wave - nw; b < nblk; b += 8 - nw) {
        int i = 0, rem = b;
        while (rem > i) { rem -= i + 1; ++i; }
        update(p + 1 + i, p + 1 + rem, p - 1);
      }
    }
    __syncthreads();
    if (fail) return;
    const int bi = p + 1 + wave;
    if (bi < NP) update(bi, p + 1, p);
    if (wave == 7) {  // never has a block above: the factored diagonal block takes its place
#pragma unroll
      for (int e = lane; e < PB * PB; e += 64) L[tri_blk(p, p)][e / PB][e % PB] = Dg[e / PB][e % PB];
    }
    __syncthreads();
  }

  if (wave == 7) {
    invert16(NP - 1);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    invert32(NP - 1);
  }
  // store: one wave per column, two rows per lane; nothing above the diagonal
  // is written (no kernel reads it)
  {
    const int bi = lane >> 3, r = 2 * (lane & 7);
    for (int c = wave; c < SB; c += 8) {
      const int bj = c / PB;
      if (2 * lane + 1 < c) continue;
      double* o = A + (int64_t)c * nb + 2 * lane;
      const double v0 = L[tri_blk(bi, bj)][r][c % PB], v1 = L[tri_blk(bi, bj)][r + 1][c % PB];
      if (2 * lane >= c) *(double2*)o = double2{v0, v1};
      else o[1] = v1;
    }
  }
}

hipError_t launch_potrf_block(const TileView& tv, int k, int j, double* dinv, hipStream_t s) {
  k_potrf_block<<<1, 512, 0, s>>>(tv, k, j, dinv);
  return hipGetLastError();
}

}  // namespace mpcr
