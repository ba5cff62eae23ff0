// Multi-format matrix product C = alpha op(A) op(B) + beta C.
//
// The paper's section "Linear Algebra Functions Performance" multiplies the
// same matrices in double, single and half precision; here each input format
// has its own MFMA path on gfx950:
//   FP64  v_mfma_f64_16x16x4f64      (FP64 accumulation)
//   FP32  v_mfma_f32_16x16x4f32      (FP32 accumulation)
//   BF16  v_mfma_f32_16x16x32_bf16   (FP32 accumulation)
//   FP16  v_mfma_f32_16x16x32_f16    (FP32 accumulation)
//   FP8   v_mfma_f32_16x16x32_fp8_fp8 (FP32 accumulation); each 128-wide k block
//         is accumulated separately and added with its factor 2^-(sA + sB)
// One workgroup computes a 128 x 128 block of C with four waves (2 x 2), each
// 64 x 64 = 4 x 4 MFMA tiles; operands are staged through LDS, k-major for the
// FP64/FP32 paths and row-major (k contiguous per row) for the 16/8-bit paths.
// The FP8 k blocks of 128 are those of the block scaling (one exponent per
// 128 x 128 block of each operand).
#include <type_traits>

#include "mpcr_internal.h"

namespace mpcr {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

constexpr int GB = 128;  // block of C per workgroup

// FP64 uses 8 waves of 64 x 32 (more waves per CU hide the staging of the
// slow FP64 MFMA better than more work per wave), FP32 4 waves of 64 x 64;
// both stage 16 k per chunk, double-buffered with one barrier per chunk (the
// shapes of the factorisation's tile-update loop).
template <int P> struct GTraits;
template <> struct GTraits<F64> { using S = double; static constexpr int BK = 16, NW = 8, WPE = 2; };
template <> struct GTraits<F32> { using S = float; static constexpr int BK = 16, NW = 4, WPE = 2; };

// FP64 / FP32 path: operands staged k-major ([BK][GB + pad]) through LDS.
template <int P>
__global__ __launch_bounds__(GTraits<P>::NW * 64) __attribute__((amdgpu_waves_per_eu(GTraits<P>::WPE))) void
k_gemm(int transA, int transB, int64_t M, int64_t N, int64_t K, double alpha, const void* Av, int64_t lda,
       const void* Bv, int64_t ldb, double beta, void* Cv, int64_t ldc, int cprec) {
  using S = typename GTraits<P>::S;
  constexpr int BK = GTraits<P>::BK, NW = GTraits<P>::NW, NT = NW * 64;
  constexpr int WM = 2, WN = NW / WM, TM = GB / WM, TN = GB / WN, FM = TM / 16, FN = TN / 16;
  constexpr int PADK = 16;  // rows k, k+1 (FP64) or k .. k+3 (FP32) of a fragment on disjoint banks
  __shared__ __attribute__((aligned(16))) S As[2][BK][GB + PADK];
  __shared__ __attribute__((aligned(16))) S Bs[2][BK][GB + PADK];

  const S* A = (const S*)Av;
  const S* B = (const S*)Bv;
  // XCD-aware order: each XCD sweeps a contiguous run of blocks, grouped 8 block
  // rows high so that the blocks in flight on one XCD share A and B panels
  const int gm = gridDim.x, gn = gridDim.y;
  const int lb = xcd_remap(blockIdx.y * gm + blockIdx.x, gm * gn);
  constexpr int GROUP = 8;
  const int group = lb / (GROUP * gn), first = group * GROUP;
  const int rows = (gm - first) < GROUP ? (gm - first) : GROUP;
  const int bi = first + (lb % (GROUP * gn)) % rows, bj = (lb % (GROUP * gn)) / rows;
  const int64_t r0 = (int64_t)bi * GB, c0 = (int64_t)bj * GB;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WM, wn = wave / WM;

  constexpr int PER = GB * BK / NT;  // elements per thread per operand
  constexpr int V = 16 / sizeof(S);  // elements per 16-byte vector
  constexpr int PV = PER / V;        // vectors per thread per operand
  S ra[PER], rb[PER];
  // Whole blocks with 16-byte aligned columns move 16-byte vectors (V
  // consecutive elements of the stored matrix: rows of a column, or k values
  // of a transposed operand's column); other blocks move single elements with
  // bounds checks.  Consecutive threads read consecutive addresses.
  const bool vec = (r0 + GB <= M) && (c0 + GB <= N) && (K % BK == 0) && ((lda * (int64_t)sizeof(S)) % 16 == 0) &&
                   ((ldb * (int64_t)sizeof(S)) % 16 == 0) && ((uintptr_t)A % 16 == 0) && ((uintptr_t)B % 16 == 0);
  // vector v of a thread: (row-or-column index, k index) of its first element
  auto avec = [&](int v, int& r, int& kk) {
    const int e = tid + NT * v;
    if (!transA) { r = (e % (GB / V)) * V; kk = e / (GB / V); } else { kk = (e % (BK / V)) * V; r = e / (BK / V); }
  };
  auto bvec = [&](int v, int& c, int& kb) {
    const int e = tid + NT * v;
    if (transB) { c = (e % (GB / V)) * V; kb = e / (GB / V); } else { kb = (e % (BK / V)) * V; c = e / (BK / V); }
  };
  auto gload = [&](int64_t k0) {
    if (vec) {
#pragma unroll
      for (int v = 0; v < PV; ++v) {
        int r, kk, c, kb;
        avec(v, r, kk);
        bvec(v, c, kb);
        const S* pa = A + (transA ? (r0 + r) * lda + k0 + kk : (k0 + kk) * lda + r0 + r);
        const S* pb = B + (transB ? (k0 + kb) * ldb + c0 + c : (c0 + c) * ldb + k0 + kb);
        *(uint4*)&ra[V * v] = *(const uint4*)pa;
        *(uint4*)&rb[V * v] = *(const uint4*)pb;
      }
      return;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int e = tid + NT * q;
      int r, kk;
      if (!transA) { r = e % GB; kk = e / GB; } else { kk = e % BK; r = e / BK; }
      const int64_t gr = r0 + r, gk = k0 + kk;
      ra[q] = (gr < M && gk < K) ? A[transA ? gr * lda + gk : gk * lda + gr] : (S)0;
      int c, kb;
      if (transB) { c = e % GB; kb = e / GB; } else { kb = e % BK; c = e / BK; }
      const int64_t gc = c0 + c, gkb = k0 + kb;
      rb[q] = (gc < N && gkb < K) ? B[transB ? gkb * ldb + gc : gc * ldb + gkb] : (S)0;
    }
  };
  auto sstore = [&](int buf) {
    if (vec) {
#pragma unroll
      for (int v = 0; v < PV; ++v) {
        int r, kk, c, kb;
        avec(v, r, kk);
        bvec(v, c, kb);
#pragma unroll
        for (int u = 0; u < V; ++u) {
          if (!transA) As[buf][kk][r + u] = ra[V * v + u]; else As[buf][kk + u][r] = ra[V * v + u];
          if (transB) Bs[buf][kb][c + u] = rb[V * v + u]; else Bs[buf][kb + u][c] = rb[V * v + u];
        }
      }
      return;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int e = tid + NT * q;
      int r, kk;
      if (!transA) { r = e % GB; kk = e / GB; } else { kk = e % BK; r = e / BK; }
      As[buf][kk][r] = ra[q];
      int c, kb;
      if (transB) { c = e % GB; kb = e / GB; } else { kb = e % BK; c = e / BK; }
      Bs[buf][kb][c] = rb[q];
    }
  };

  using Acc = typename std::conditional<P == F64, d4, f4>::type;
  Acc acc[FM][FN];
#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b) acc[a][b] = Acc{0, 0, 0, 0};

  if (K > 0) {
    gload(0);
    sstore(0);
  }
  __syncthreads();
  int cur = 0;
  for (int64_t k0 = 0; k0 < K; k0 += BK) {
    const bool more = k0 + BK < K;
    if (more) gload(k0 + BK);
#pragma unroll
    for (int k4 = 0; k4 < BK; k4 += 4) {
      S av[FM], bv[FN];
#pragma unroll
      for (int a = 0; a < FM; ++a) av[a] = As[cur][k4 + (lane >> 4)][wm * TM + a * 16 + (lane & 15)];
#pragma unroll
      for (int b = 0; b < FN; ++b) bv[b] = Bs[cur][k4 + (lane >> 4)][wn * TN + b * 16 + (lane & 15)];
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) {
          if constexpr (P == F64)
            acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
          else
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[b], acc[a][b], 0, 0, 0);
        }
    }
    if (more) sstore(cur ^ 1);
    __syncthreads();
    cur ^= 1;
  }

#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = (P == F64) ? ((lane >> 4) + 4 * r) : (4 * (lane >> 4) + r);
        const int64_t R = r0 + wm * TM + a * 16 + row;
        const int64_t C = c0 + wn * TN + b * 16 + (lane & 15);
        if (R >= M || C >= N) continue;
        const int64_t idx = C * ldc + R;
        double v = alpha * (double)acc[a][b][r];
        if (cprec == F64) {
          double* Cp = (double*)Cv;
          if (beta != 0.0) v += beta * Cp[idx];
          Cp[idx] = v;
        } else {
          float* Cp = (float*)Cv;
          if (beta != 0.0) v += beta * (double)Cp[idx];
          Cp[idx] = (float)v;
        }
      }
}

// ---------------------------------------------------------------------------
// 16- and 8-bit path.  Both operands are read "k-contiguous": A as an m x k
// row-major array (AT, leading dimension ldat) and B as the usual k x n
// column-major array, with 16-byte aligned rows and k a multiple of the stage.
// Operands in another layout are first packed into that one, k padded with
// zeros (k_pack); rows past m or n are read as the last row and their products
// not stored, so ragged and whole shapes run the same loop.
//
// One workgroup of WM x WN waves computes a (16 TA WM) x (16 TB WN) block of C,
// a wave TA x TB tiles of 16 x 16.  Stages of 128 bytes of k: both operands'
// rows are moved global -> registers -> LDS (padded rows, so the 16-byte
// fragment reads of 16 consecutive rows hit disjoint banks), double-buffered
// with one barrier per stage; the next stage's global loads are in flight
// during the current stage's MFMAs.  The MFMA takes the B fragment as its first
// operand, so a lane's four results are four columns of one row of C: for each
// register the 16 lanes of a group store 16 consecutive rows of a column.
//
// FP8: a stage is one block of the power-of-two scaling, and each 16 x 16 tile
// of a stage one gfx950 block-scaled MFMA (v_mfma_scale_f32_16x16x128_f8f6f4,
// E4M3 operands): its E8M0 scales undo the operands' block exponents inside
// the instruction (exact powers of two), so the stages accumulate straight
// into the FP32 results.  A lane supplies 32 consecutive k of one row or
// column; the same lane-to-k assignment for both operands makes the sum
// correct for any internal order of the 128 products.
// ---------------------------------------------------------------------------
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int STAGE = 128;  // bytes of k per stage

template <int P, int WM, int WN, int TA, int TB, int PAD>
__global__ __launch_bounds__(64 * WM * WN) void k_gemm_lowp(int64_t M, int64_t N, int64_t K, double alpha,
                                                            const void* ATv, int64_t ldat, const int8_t* sA,
                                                            int64_t mbA, int sa_kmajor, const void* Bv, int64_t ldb,
                                                            const int8_t* sB, int64_t mbB, int sb_kmajor, double beta,
                                                            void* Cv, int64_t ldc, int cprec) {
  constexpr int ES = (P == F8) ? 1 : 2;            // element bytes
  constexpr int BK = STAGE / ES;                   // k per stage
  constexpr int NT = 64 * WM * WN;                 // threads
  constexpr int BM = 16 * TA * WM, BN = 16 * TB * WN;
  constexpr int RPL = NT / 8;                      // rows per load instruction
  constexpr int NVA = BM / RPL, NVB = BN / RPL;    // 16-byte vectors per thread and operand
  constexpr int LDR = STAGE + PAD;                 // LDS row
  __shared__ __attribute__((aligned(16))) uint8_t As[2][BM * LDR];
  __shared__ __attribute__((aligned(16))) uint8_t Bs[2][BN * LDR];
  // XCD-aware order, grouped 8 block rows high (blocks in flight on one XCD share panels)
  const int gm = gridDim.x, gn = gridDim.y;
  const int lb = xcd_remap(blockIdx.y * gm + blockIdx.x, gm * gn);
  constexpr int GROUP = 8;
  const int group = lb / (GROUP * gn), first = group * GROUP;
  const int rows = (gm - first) < GROUP ? (gm - first) : GROUP;
  const int bi = first + (lb % (GROUP * gn)) % rows, bj = (lb % (GROUP * gn)) / rows;
  const int64_t r0 = (int64_t)bi * BM, c0 = (int64_t)bj * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WM, wn = wave / WM;
  const int g16 = lane & 15, q = lane >> 4;

  // loader: thread t moves 16-byte vectors (row t / 8 + RPL v, chunk t % 8) of
  // both operands.  The last stage reloads itself (no branch around the
  // staging, so the staged vectors stay in registers); its copies are never
  // read.
  const int lrow = tid >> 3, lchunk = tid & 7;
  const uint8_t* AT = (const uint8_t*)ATv;
  const uint8_t* B = (const uint8_t*)Bv;
  const uint8_t *pa[NVA], *pb[NVB];
#pragma unroll
  for (int v = 0; v < NVA; ++v) {
    const int64_t r = r0 + lrow + RPL * v;
    pa[v] = AT + (r < M ? r : M - 1) * ldat * ES + lchunk * 16;
  }
#pragma unroll
  for (int v = 0; v < NVB; ++v) {
    const int64_t c = c0 + lrow + RPL * v;
    pb[v] = B + (c < N ? c : N - 1) * ldb * ES + lchunk * 16;
  }
  const int soff = lrow * LDR + lchunk * 16;
  u32x4 ga[NVA], gb[NVB];
  auto gload = [&](int64_t kb) {
#pragma unroll
    for (int v = 0; v < NVA; ++v) ga[v] = *(const u32x4*)(pa[v] + kb);
#pragma unroll
    for (int v = 0; v < NVB; ++v) gb[v] = *(const u32x4*)(pb[v] + kb);
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int v = 0; v < NVA; ++v) *(u32x4*)&As[buf][soff + v * RPL * LDR] = ga[v];
#pragma unroll
    for (int v = 0; v < NVB; ++v) *(u32x4*)&Bs[buf][soff + v * RPL * LDR] = gb[v];
  };

  f4 acc[TA][TB];
#pragma unroll
  for (int a = 0; a < TA; ++a)
#pragma unroll
    for (int b = 0; b < TB; ++b) acc[a][b] = f4{0, 0, 0, 0};

  const int64_t KB = K * ES;
  if (K > 0) {
    gload(0);
    sstore(0);
  }
  __syncthreads();
  int cur = 0;
  if constexpr (P == F8) {
    auto frag = [&](const uint8_t* p) {  // 32 consecutive bytes
      const u32x4 lo = *(const u32x4*)p, hi = *(const u32x4*)(p + 16);
      return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
    };
    // the scale blocks of this wave's rows and columns
    const int64_t ra = r0 + 16 * TA * wm, cb = c0 + 16 * TB * wn;
    const int64_t ib = (ra < M ? ra : M - 1) / 128, jb = (cb < N ? cb : N - 1) / 128;
    for (int64_t k0 = 0; k0 < KB; k0 += STAGE) {
      gload(k0 + STAGE < KB ? k0 + STAGE : k0);
      const int64_t kb = k0 / 128;
      const int ea = sa_kmajor ? sA[ib * mbA + kb] : sA[kb * mbA + ib];
      const int eb = sb_kmajor ? sB[kb * mbB + jb] : sB[jb * mbB + kb];
      // E8M0 scale bytes of 2^-ea and 2^-eb; 255 (ea = -128) is no scale: one step goes to the other operand's
      int sca = 127 - ea, scb = 127 - eb;
      if (sca > 254) { sca = 254; scb = scb < 254 ? scb + 1 : 254; }
      if (scb > 254) { scb = 254; sca = sca < 254 ? sca + 1 : 254; }
      const uint8_t* Ab = &As[cur][(wm * TA * 16 + g16) * LDR + 32 * q];
      const uint8_t* Bb = &Bs[cur][(wn * TB * 16 + g16) * LDR + 32 * q];
      i32x8 fb[TB];
#pragma unroll
      for (int b = 0; b < TB; ++b) fb[b] = frag(Bb + b * 16 * LDR);
      i32x8 fa = frag(Ab);
#pragma unroll
      for (int a = 0; a < TA; ++a) {
        const i32x8 fan = frag(Ab + ((a + 1) % TA) * 16 * LDR);  // the next row block's fragment
#pragma unroll
        for (int b = 0; b < TB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fb[b], fa, acc[a][b], 0, 0, 0, scb, 0, sca);
        fa = fan;
      }
      sstore(cur ^ 1);
      __syncthreads();
      cur ^= 1;
    }
  } else {
    // fragments of one 32-wide k step: A rows 16 a + g16, B columns 16 b + g16,
    // k values 8 q .. 8 q + 7 of the step
    u16x8 fa0[TA], fb0[TB], fa1[TA], fb1[TB];
    auto frag = [&](int buf, int k32, u16x8* fa, u16x8* fb) {
      const uint8_t* Ab = &As[buf][(wm * TA * 16 + g16) * LDR + (k32 + 8 * q) * ES];
      const uint8_t* Bb = &Bs[buf][(wn * TB * 16 + g16) * LDR + (k32 + 8 * q) * ES];
#pragma unroll
      for (int b = 0; b < TB; ++b) fb[b] = *(const u16x8*)(Bb + b * 16 * LDR);
#pragma unroll
      for (int a = 0; a < TA; ++a) fa[a] = *(const u16x8*)(Ab + a * 16 * LDR);
    };
    auto mma = [&](const u16x8* fa, const u16x8* fb) {
#pragma unroll
      for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b) {
          if constexpr (P == BF16)
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fb[b]),
                                                                 __builtin_bit_cast(bf16x8, fa[a]), acc[a][b], 0, 0, 0);
          else
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, fb[b]),
                                                                __builtin_bit_cast(f16x8, fa[a]), acc[a][b], 0, 0, 0);
        }
    };
    // per stage: the next stage's A and B are requested at its start and stored
    // to the other LDS buffer at its end; the second step's fragments are read
    // while the first step's MFMAs run; after the barrier the next stage's first
    // fragments are read
    if (K > 0) frag(0, 0, fa0, fb0);
    for (int64_t k0 = 0; k0 < KB; k0 += STAGE) {
      gload(k0 + STAGE < KB ? k0 + STAGE : k0);
      frag(cur, 32, fa1, fb1);
      mma(fa0, fb0);
      mma(fa1, fb1);
      sstore(cur ^ 1);
      __syncthreads();
      cur ^= 1;
      frag(cur, 0, fa0, fb0);
    }
  }

  // lane (g16, q), register r of tile (a, b): C[r0 + 16 (TA wm + a) + g16][c0 + 16 (TB wn + b) + 4 q + r]
#pragma unroll
  for (int a = 0; a < TA; ++a)
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t R = r0 + (wm * TA + a) * 16 + g16;
        const int64_t Cc = c0 + (wn * TB + b) * 16 + 4 * q + r;
        if (R >= M || Cc >= N) continue;
        const int64_t idx = Cc * ldc + R;
        double v = alpha * (double)acc[a][b][r];
        if (cprec == F64) {
          double* Cp = (double*)Cv;
          if (beta != 0.0) v += beta * Cp[idx];
          Cp[idx] = v;
        } else {
          float* Cp = (float*)Cv;
          if (beta != 0.0) v += beta * (double)Cp[idx];
          Cp[idx] = (float)v;
        }
      }
}

// Packs a rows x cols operand into a k-contiguous array: out[r * ldo + c] =
// element (r, c), read from in[c * ldi + r] (TR) or in[r * ldi + c] (!TR), and 0
// for cols <= c < ldo.  64 x 64 pieces go through LDS so that both the reads
// and the writes move 16-byte vectors (reads at the elements' own alignment,
// which global memory serves; single elements at the edges).
template <typename T, bool TR>
__global__ __launch_bounds__(256) void k_pack(int64_t rows, int64_t cols, const T* in, int64_t ldi, T* out,
                                              int64_t ldo) {
  constexpr int V = 16 / sizeof(T), VPL = 64 / V;  // elements per vector, vectors per line of a piece
  constexpr int LD = 64 + 4 / sizeof(T);
  __shared__ __attribute__((aligned(16))) T t[64][LD];  // [r][c]
  const int64_t rb = (int64_t)blockIdx.x * 64, cb = (int64_t)blockIdx.y * 64;
  for (int e = threadIdx.x; e < 64 * VPL; e += 256) {
    const int line = e / VPL, f = (e % VPL) * V;  // f .. f + V - 1: rows (TR) or columns (!TR) of the piece
    const int64_t slow = (TR ? cb : rb) + line, fast = (TR ? rb : cb) + f;
    const int64_t nslow = TR ? cols : rows, nfast = TR ? rows : cols;
    T v[V];
    if (slow < nslow && fast + V <= nfast) {
      __builtin_memcpy(v, in + slow * ldi + fast, 16);
    } else {
#pragma unroll
      for (int u = 0; u < V; ++u) v[u] = (slow < nslow && fast + u < nfast) ? in[slow * ldi + fast + u] : T(0);
    }
#pragma unroll
    for (int u = 0; u < V; ++u) {
      if (TR) t[f + u][line] = v[u];
      else t[line][f + u] = v[u];
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * VPL; e += 256) {
    const int r = e / VPL, c = (e % VPL) * V;
    if (rb + r >= rows || cb + c >= ldo) continue;  // ldo is a multiple of V
    T v[V];
#pragma unroll
    for (int u = 0; u < V; ++u) v[u] = t[r][c + u];
    __builtin_memcpy(__builtin_assume_aligned(out + (rb + r) * ldo + cb + c, 16), v, 16);
  }
}

// ldo: a multiple of 16 bytes, out 16-byte aligned
hipError_t launch_pack(int es, int trans, int64_t rows, int64_t cols, const void* in, int64_t ldi, void* out,
                       int64_t ldo, hipStream_t s) {
  if (rows == 0 || cols == 0) return hipSuccess;
  dim3 grid((unsigned)((rows + 63) / 64), (unsigned)((ldo + 63) / 64));
  if (es == 1) {
    if (trans) k_pack<uint8_t, true><<<grid, 256, 0, s>>>(rows, cols, (const uint8_t*)in, ldi, (uint8_t*)out, ldo);
    else k_pack<uint8_t, false><<<grid, 256, 0, s>>>(rows, cols, (const uint8_t*)in, ldi, (uint8_t*)out, ldo);
  } else {
    if (trans) k_pack<uint16_t, true><<<grid, 256, 0, s>>>(rows, cols, (const uint16_t*)in, ldi, (uint16_t*)out, ldo);
    else k_pack<uint16_t, false><<<grid, 256, 0, s>>>(rows, cols, (const uint16_t*)in, ldi, (uint16_t*)out, ldo);
  }
  return hipGetLastError();
}

// 256 x 256 blocks (eight waves of 128 x 64, half the LDS traffic per product
// of the 128 x 128 ones) once they fill the chip; a launch that leaves more
// than a fifth of its last round of 256 CUs idle runs 128 x 128 blocks (four
// waves of 64 x 64, two workgroups per CU).
static bool large_blocks(int64_t m, int64_t n) {
  const int64_t blocks = ((m + 255) / 256) * ((n + 255) / 256), rounds = (blocks + 255) / 256;
  return blocks * 5 >= rounds * 256 * 4;
}

// k per stage of the 16/8-bit product: its operands' k is a multiple of it
int gemm_lowp_kstage(int prec) { return STAGE / (prec == F8 ? 1 : 2); }

hipError_t launch_gemm_lowp(int prec, int64_t m, int64_t n, int64_t k, double alpha, const void* AT, int64_t ldat,
                            const int8_t* sA, int64_t mbA, int sa_kmajor, const void* B, int64_t ldb,
                            const int8_t* sB, int64_t mbB, int sb_kmajor, double beta, void* C, int64_t ldc, int cprec,
                            hipStream_t s) {
  const int es = prec == F8 ? 1 : 2;
  if (k % (STAGE / es) != 0 || (ldat * es) % 16 != 0 || (ldb * es) % 16 != 0 || (uintptr_t)AT % 16 != 0 ||
      (uintptr_t)B % 16 != 0)
    return hipErrorInvalidValue;
#define MPCR_LOWP(P, WM, WN, TA, TB, PAD)                                                                             \
  k_gemm_lowp<P, WM, WN, TA, TB, PAD>                                                                                 \
      <<<dim3((unsigned)((m + 16 * TA * WM - 1) / (16 * TA * WM)), (unsigned)((n + 16 * TB * WN - 1) / (16 * TB * WN))), \
         64 * WM * WN, 0, s>>>(m, n, k, alpha, AT, ldat, sA, mbA, sa_kmajor, B, ldb, sB, mbB, sb_kmajor, beta, C, ldc, \
                               cprec)
  if (large_blocks(m, n)) {
    switch (prec) {
      case BF16: MPCR_LOWP(BF16, 2, 4, 8, 4, 32); break;
      case F16: MPCR_LOWP(F16, 2, 4, 8, 4, 32); break;
      case F8: MPCR_LOWP(F8, 2, 4, 8, 4, 16); break;
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (prec) {
      case BF16: MPCR_LOWP(BF16, 2, 2, 4, 4, 16); break;
      case F16: MPCR_LOWP(F16, 2, 2, 4, 4, 16); break;
      case F8: MPCR_LOWP(F8, 2, 2, 4, 4, 16); break;
      default: return hipErrorInvalidValue;
    }
  }
#undef MPCR_LOWP
  return hipGetLastError();
}

hipError_t launch_gemm(int prec, int transA, int transB, int64_t m, int64_t n, int64_t k, double alpha, const void* A,
                       int64_t lda, const void* B, int64_t ldb, double beta, void* C, int64_t ldc, int cprec,
                       hipStream_t s) {
  dim3 grid((unsigned)((m + GB - 1) / GB), (unsigned)((n + GB - 1) / GB));
  switch (prec) {
    case F64: k_gemm<F64><<<grid, GTraits<F64>::NW * 64, 0, s>>>(transA, transB, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, cprec); break;
    case F32: k_gemm<F32><<<grid, GTraits<F32>::NW * 64, 0, s>>>(transA, transB, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, cprec); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace mpcr
