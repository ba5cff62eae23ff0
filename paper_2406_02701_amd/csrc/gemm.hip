// Multi-format matrix product C = alpha op(A) op(B) + beta C.
//
// The paper's section "Linear Algebra Functions Performance" multiplies the
// same matrices in double, single and half precision; here each input format
// has its own MFMA path on gfx950:
//   FP64  v_mfma_f64_16x16x4f64                 (FP64 accumulation)
//   FP32  v_mfma_f32_16x16x4f32                 (FP32 accumulation)
//   BF16  v_mfma_f32_16x16x32_bf16              (FP32 accumulation)
//   FP16  v_mfma_f32_16x16x32_f16               (FP32 accumulation)
//   FP8   v_mfma_scale_f32_16x16x128_f8f6f4     (FP32 accumulation), the block
//         exponents as the instruction's scales
// Operands are staged through LDS, k-major for FP64/FP32 and row-major (k
// contiguous per row) for the 16/8-bit formats.  The FP8 k blocks of 128 are
// those of the block scaling (one exponent per 128 x 128 block of each operand).
#include <type_traits>

#include "mpcr_internal.h"

namespace mpcr {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

// FP64 / FP32 path: blocks of (16 FM WM) x (16 FN WN) of C by WM x WN waves of
// FM x FN MFMA tiles; both operands are staged k-major through LDS, 16 k per
// chunk, double-buffered with one barrier per chunk, the next chunk's loads in
// flight during the current one's MFMAs.
//   Loads are 16-byte vectors along the stored columns at the elements' own
// alignment, whatever the sizes and leading dimensions: a vector that crosses
// the last row or column is read element by element with clamped indexes (what
// lies past the edge only feeds results that are not stored), and only a last
// chunk of fewer than 16 k takes a checked path, which fills up with zeros.
//   A transposed operand's vector is four (FP64: two) k of one row and is
// scattered to as many LDS rows; the row index is exclusive-or'ed with 16
// (FP64: 4) times the k group, which puts a wave's 64 stores on 64 different
// banks and leaves the fragment reads, which stay inside a group (FP64: inside
// 16 rows), free of conflicts.
//   FP64 takes the B fragment first, so that a store instruction writes 16
// consecutive rows; FP32 stores a lane's four consecutive rows as one vector.
// Bound by the matrix cores (133 of 157 TF/s FP32, 62 of 79 FP64 at 8192^3) once
// the blocks fill the chip.  Measured, whole call, against 128 x 128 blocks that
// took a ragged size or k element by element: FP32 NT 3000^3 1370 -> 541 us, NN
// 8192^3 10.1 -> 8.3 ms, TN 1000^3 243 -> 49 us; FP64 NT 3000^3 1513 -> 1035 us,
// NN 8192^3 22.0 -> 17.7 ms.
template <int P> struct GTraits;
template <> struct GTraits<F64> {
  using S = double;
  using Acc = d4;
  typedef double Vec __attribute__((ext_vector_type(2), aligned(8)));
};
template <> struct GTraits<F32> {
  using S = float;
  using Acc = f4;
  typedef float Vec __attribute__((ext_vector_type(4), aligned(4)));
};
constexpr int GPAD = 16;  // rows k, k+1 (FP64) or k .. k+3 (FP32) of a fragment on disjoint banks

// One operand's way into LDS.  TR: the stored matrix is k x rows (a row's k are
// contiguous), else rows x k.
template <int P, int NT, int BR, int BK, bool TR>
struct GOperand {
  using S = typename GTraits<P>::S;
  using Vec = typename GTraits<P>::Vec;
  static constexpr int V = 16 / sizeof(S), NV = BR * BK / V / NT, LD = BR + GPAD;
  static_assert(NV * NT * V == BR * BK, "whole vectors per thread");
  const S* p[NV];  // each vector's first element in chunk 0 (row clamped)
  int64_t step;    // elements from one chunk to the next
  bool cross[NV];  // (not TR) the vector crosses the last row
  int last[NV];    // ... the offset of the last row's element
  Vec v[NV];

  static __device__ __forceinline__ int row(int e) { return TR ? e / (BK / V) : (e % (BR / V)) * V; }
  static __device__ __forceinline__ int kk(int e) { return TR ? (e % (BK / V)) * V : e / (BR / V); }
  // LDS column of row r, k
  static __device__ __forceinline__ int col(int r, int k) {
    constexpr int SPREAD = (P == F64 ? 32 : 64) / (BK / V);
    return TR ? r ^ (SPREAD * (k / V)) : r;
  }
  __device__ __forceinline__ void init(const S* A, int64_t ld, int64_t r0, int64_t rows, int tid) {
    step = TR ? BK : BK * ld;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int e = tid + NT * i;
      const int64_t r = r0 + row(e), rc = r < rows ? r : rows - 1;
      p[i] = TR ? A + rc * ld + kk(e) : A + rc + kk(e) * ld;
      cross[i] = !TR && rc + V > rows;
      last[i] = (int)(rows - 1 - rc < V ? rows - 1 - rc : V);
    }
  }
  __device__ __forceinline__ void load() {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (!cross[i]) {
        v[i] = *(const Vec*)p[i];
      } else {
#pragma unroll
        for (int u = 0; u < V; ++u) v[i][u] = p[i][u < last[i] ? u : last[i]];
      }
      p[i] += step;
    }
  }
  __device__ __forceinline__ void load_tail(int left, int tid) {  // left < BK k
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int k = kk(tid + NT * i);
#pragma unroll
      for (int u = 0; u < V; ++u) {
        const int o = TR ? u : (u < last[i] ? u : last[i]);
        v[i][u] = (TR ? k + u : k) < left ? p[i][o] : (S)0;
      }
    }
  }
  __device__ __forceinline__ void store(S (*lds)[LD], int tid) const {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int e = tid + NT * i, r = row(e), k = kk(e);
      if constexpr (TR) {
#pragma unroll
        for (int u = 0; u < V; ++u) lds[k + u][col(r, k)] = v[i][u];
      } else {
        typedef S VecA __attribute__((ext_vector_type(16 / sizeof(S))));
        *(VecA*)&lds[k][r] = (VecA)v[i];
      }
    }
  }
};

template <int P, int WM, int WN, int FM, int FN, int BK, bool TA, bool TB>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2))) void
k_gemm(int64_t M, int64_t N, int64_t K, double alpha, const void* Av, int64_t lda, const void* Bv, int64_t ldb,
       double beta, void* Cv, int64_t ldc, int cprec) {
  using S = typename GTraits<P>::S;
  using Acc = typename GTraits<P>::Acc;
  constexpr int NT = 64 * WM * WN, BM = 16 * FM * WM, BN = 16 * FN * WN;
  using OpA = GOperand<P, NT, BM, BK, TA>;
  using OpB = GOperand<P, NT, BN, BK, !TB>;
  __shared__ __attribute__((aligned(16))) S As[2][BK][OpA::LD];
  __shared__ __attribute__((aligned(16))) S Bs[2][BK][OpB::LD];

  // XCD-aware order: each XCD sweeps a contiguous run of blocks, grouped 8 block
  // rows high so that the blocks in flight on one XCD share A and B panels
  const int gm = gridDim.x, gn = gridDim.y;
  const int lb = xcd_remap(blockIdx.y * gm + blockIdx.x, gm * gn);
  constexpr int GROUP = 8;
  const int group = lb / (GROUP * gn), first = group * GROUP;
  const int rows = (gm - first) < GROUP ? (gm - first) : GROUP;
  const int bi = first + (lb % (GROUP * gn)) % rows, bj = (lb % (GROUP * gn)) / rows;
  const int64_t r0 = (int64_t)bi * BM, c0 = (int64_t)bj * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WM, wn = wave / WM, g16 = lane & 15, q = lane >> 4;

  OpA a;
  OpB b;
  a.init((const S*)Av, lda, r0, M, tid);
  b.init((const S*)Bv, ldb, c0, N, tid);
  Acc acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = Acc{0, 0, 0, 0};

  const int64_t chunks = (K + BK - 1) / BK;
  const int left = (int)(K % BK);
  auto gload = [&](int64_t t) {
    if (t + 1 < chunks || left == 0) {
      a.load();
      b.load();
    } else {
      a.load_tail(left, tid);
      b.load_tail(left, tid);
    }
  };
  if (chunks > 0) {
    gload(0);
    a.store(As[0], tid);
    b.store(Bs[0], tid);
  }
  __syncthreads();
  int cur = 0;
  for (int64_t t = 0; t < chunks; ++t) {
    const bool more = t + 1 < chunks;
    if (more) gload(t + 1);
#pragma unroll
    for (int k4 = 0; k4 < BK; k4 += 4) {
      const int k = k4 + q;
      S av[FM], bv[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) av[i] = As[cur][k][OpA::col((wm * FM + i) * 16 + g16, P == F64 ? k : k4)];
#pragma unroll
      for (int j = 0; j < FN; ++j) bv[j] = Bs[cur][k][OpB::col((wn * FN + j) * 16 + g16, P == F64 ? k : k4)];
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          if constexpr (P == F64)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(bv[j], av[i], acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
    }
    if (more) {
      a.store(As[cur ^ 1], tid);
      b.store(Bs[cur ^ 1], tid);
    }
    __syncthreads();
    cur ^= 1;
  }

  auto put = [&](auto* Cp, int64_t idx, double x) {
    using T = std::remove_pointer_t<decltype(Cp)>;
    double v = alpha * x;
    if (beta != 0.0) v += beta * (double)Cp[idx];
    Cp[idx] = (T)v;
  };
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int64_t R = r0 + (wm * FM + i) * 16, C = c0 + (wn * FN + j) * 16;
      if constexpr (P == F64) {
        if (R + g16 >= M) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (C + q + 4 * r < N) put((double*)Cv, (C + q + 4 * r) * ldc + R + g16, acc[i][j][r]);
      } else {
        if (C + g16 >= N) continue;
        const int64_t idx = (C + g16) * ldc + R + 4 * q;
        if (cprec == F32 && R + 4 * q + 4 <= M) {
          using Vec = GTraits<F32>::Vec;
          Vec* o = (Vec*)((float*)Cv + idx);
          Vec old = {0, 0, 0, 0}, w;
          if (beta != 0.0) old = *o;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            double v = alpha * (double)acc[i][j][r];
            if (beta != 0.0) v += beta * (double)old[r];
            w[r] = (float)v;
          }
          *o = w;
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (R + 4 * q + r >= M) break;
            if (cprec == F64) put((double*)Cv, idx + r, (double)acc[i][j][r]);
            else put((float*)Cv, idx + r, (double)acc[i][j][r]);
          }
        }
      }
    }
}

// ---------------------------------------------------------------------------
// 16- and 8-bit path.  Both operands are read "k-contiguous": A as an m x k
// row-major array (AT, leading dimension ldat) and B as the usual k x n
// column-major array, with 16-byte aligned rows.  Operands in another layout are
// first packed into that one, k padded with zeros to whole stages (k_pack); rows
// past m or n are read as the last row and their products not stored, so ragged and
// whole shapes run the same loop.  A part of a stage at the end of k (TAIL: operands
// that are read where they are) is loaded behind the loop, zeros past the last k.
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
//
// Bound: FP8 at 8192^3 by LDS reads and the matrix cores together.  Whole calls,
// before -> after (kernels for whole shapes only, generic bytewise one for the
// rest, exponents requested behind the next stage's operands, bounds checks on
// every store): FP8 TN 8192^3 643 -> 630 us, NN 734 -> 658 us, TN 3001 x 2999 x
// 4003 560 -> 110 us, NN 2000^3 114 -> 47 us; BF16
// TN 3001 x 2999 x 4003 584 -> 127 us.
// ---------------------------------------------------------------------------
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int STAGE = 128;     // bytes of k per stage
constexpr int LOWP_BIG = 256;  // block of C of k_gemm_lowp_big

// XCD-aware order of the blocks, grouped 8 block rows high (blocks in flight on one XCD share panels)
__device__ __forceinline__ void lowp_block(int& bi, int& bj) {
  const int gm = gridDim.x, gn = gridDim.y;
  const int lb = xcd_remap(blockIdx.y * gm + blockIdx.x, gm * gn);
  constexpr int GROUP = 8;
  const int group = lb / (GROUP * gn), first = group * GROUP;
  const int rows = (gm - first) < GROUP ? (gm - first) : GROUP;
  bi = first + (lb % (GROUP * gn)) % rows;
  bj = (lb % (GROUP * gn)) / rows;
}

// lane (g16, q), register r of tile (a, b): C[R0 + 16 a][C0 + 16 b + r], R0 and C0 the lane's first row and column
template <int TA, int TB>
__device__ __forceinline__ void lowp_store(const f4 (&acc)[TA][TB], double alpha, double beta, void* Cv, int64_t ldc,
                                           int cprec, int64_t R0, int64_t C0, int64_t M, int64_t N, bool whole_block) {
  auto write = [&](auto* Cp, auto whole) {
    using T = std::remove_pointer_t<decltype(Cp)>;
    Cp += C0 * ldc + R0;
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        T* col = Cp + (b * 16 + r) * ldc;
#pragma unroll
        for (int a = 0; a < TA; ++a) {
          if (!decltype(whole)::value && (R0 + a * 16 >= M || C0 + b * 16 + r >= N)) continue;
          double v = alpha * (double)acc[a][b][r];
          if (beta != 0.0) v += beta * (double)col[a * 16];
          col[a * 16] = (T)v;
        }
      }
  };
  if (cprec == F64) {
    if (whole_block) write((double*)Cv, std::true_type{});
    else write((double*)Cv, std::false_type{});
  } else {
    if (whole_block) write((float*)Cv, std::true_type{});
    else write((float*)Cv, std::false_type{});
  }
}

template <int P, int WM, int WN, int TA, int TB, int PAD, bool TAIL>
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
  int bi, bj;
  lowp_block(bi, bj);
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

  const int64_t KB = TAIL ? K / BK * STAGE : K * ES;  // (whole stages, in bytes)
  if (KB > 0) {
    gload(0);
    sstore(0);
  }
  __syncthreads();
  int cur = 0;
  // the part of a stage behind the whole ones into the buffer that nobody reads any more
  auto load_tail = [&] {
    using E = std::conditional_t<ES == 1, uint8_t, uint16_t>;
    const int left = (int)(K * ES - KB) - lchunk * 16;  // bytes of this thread's vectors
    auto vec = [&](const uint8_t* p) {
      u32x4 v = {0, 0, 0, 0};
      if (left >= 16) return *(const u32x4*)p;
#pragma unroll
      for (int e = 0; e < 16 / ES; ++e)
        if (e * ES < left) v[e * ES / 4] |= (uint32_t)((const E*)p)[e] << (8 * ES * (e % (4 / ES)));
      return v;
    };
#pragma unroll
    for (int v = 0; v < NVA; ++v) ga[v] = vec(pa[v] + KB);
#pragma unroll
    for (int v = 0; v < NVB; ++v) gb[v] = vec(pb[v] + KB);
    sstore(cur ^ 1);
    __syncthreads();
    cur ^= 1;
  };
  if constexpr (P == F8) {
    auto frag = [&](const uint8_t* p) {  // 32 consecutive bytes
      const u32x4 lo = *(const u32x4*)p, hi = *(const u32x4*)(p + 16);
      return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
    };
    // the scale blocks of this wave's rows and columns
    const int64_t ra = r0 + 16 * TA * wm, cb = c0 + 16 * TB * wn;
    const int64_t ib = (ra < M ? ra : M - 1) / 128, jb = (cb < N ? cb : N - 1) / 128;
    // (the exponents of a stage are requested a stage ahead, before its operands:
    // loads return in order, so a later request would wait for all of those)
    const int8_t* pea = sa_kmajor ? sA + ib * mbA : sA + ib;
    const int8_t* peb = sb_kmajor ? sB + jb : sB + jb * mbB;
    const int64_t dea = sa_kmajor ? 1 : mbA, deb = sb_kmajor ? mbB : 1;
    int nea = KB > 0 ? *pea : 0, neb = KB > 0 ? *peb : 0;
    auto mma = [&](int ea, int eb) {
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
    };
    for (int64_t k0 = 0; k0 < KB; k0 += STAGE) {
      const int64_t kn = k0 + STAGE < KB ? k0 + STAGE : k0;
      const int ea = nea, eb = neb;
      nea = pea[(kn / 128) * dea];
      neb = peb[(kn / 128) * deb];
      gload(kn);
      mma(ea, eb);
      sstore(cur ^ 1);
      __syncthreads();
      cur ^= 1;
    }
    if constexpr (TAIL) {
      const int ea = pea[(KB / 128) * dea], eb = peb[(KB / 128) * deb];
      load_tail();
      mma(ea, eb);
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
    if (KB > 0) frag(0, 0, fa0, fb0);
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
    if constexpr (TAIL) {
      load_tail();
      frag(cur, 0, fa0, fb0);
      frag(cur, 32, fa1, fb1);
      mma(fa0, fb0);
      mma(fa1, fb1);
    }
  }

  lowp_store<TA, TB>(acc, alpha, beta, Cv, ldc, cprec, r0 + wm * TA * 16 + g16, c0 + wn * TB * 16 + 4 * q, M, N,
                     r0 + BM <= M && c0 + BN <= N);
}

// The 16-bit product on 256 x 256 blocks: four waves of 128 x 128, one per SIMD,
// 256 accumulation registers each.  The MFMAs of a 32-wide k step take 1024
// cycles of a CU.  With eight waves of 128 x 64 its fragment reads (96 KB) and
// stores (32 KB, through registers) took as many cycles of the LDS: 45% MFMA
// busy; here the reads are 64 KB, and the operands go global -> LDS directly.
// A wave has no other one to hide behind, so nothing it waits for is recent:
//   - a step's fragments are read, two per eight MFMAs, during the step before it;
//   - the barrier stands between a stage's two steps: by then the stage's last
//     fragments are in registers, so the second step reads the next stage's first
//     ones and the copies of the stage after next go into the buffer given up.
// A copy of 1 KB is 8 rows of 128 bytes; granule c of row r is kept at c ^ (r % 8),
// so that the 16 rows of a fragment read spread over the banks.  Every element
// takes its products in the order of the 128 x 128 blocks: the same bits.
// Whole calls, before (eight waves) -> after: BF16 NN 8192^3 1122 -> 904 to 925 us,
// TN 1154 -> 935, FP16 1148 -> 947, BF16 4096^3 151 -> 117, 16384 x 4096 x 2048
// 321 -> 266.  An FP8 form (two sets of eight 32-byte fragments) spills: 2349 us
// for 612.
template <int P>
__global__ __launch_bounds__(256) void k_gemm_lowp_big(int64_t M, int64_t N, int64_t K, double alpha, const void* ATv,
                                                       int64_t ldat, const void* Bv, int64_t ldb, double beta,
                                                       void* Cv, int64_t ldc, int cprec) {
  constexpr int BM = LOWP_BIG, TA = 8, WM = 2, NI = BM / 8 / 4;  // NI copies of 8 rows per wave and operand
  constexpr int OP = BM * STAGE;                                 // bytes of an operand's stage
  __shared__ __attribute__((aligned(1024))) uint8_t sm[2][2 * OP];
  int bi, bj;
  lowp_block(bi, bj);
  const int64_t r0 = (int64_t)bi * BM, c0 = (int64_t)bj * BM;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WM, wn = wave / WM;
  const int g16 = lane & 15, q = lane >> 4;

  const int64_t ra = r0 + 64 * wave < M ? r0 + 64 * wave : M - 1, rb = c0 + 64 * wave < N ? c0 + 64 * wave : N - 1;
  const uint8_t* Ap = (const uint8_t*)ATv + ra * ldat * 2;
  const uint8_t* Bp = (const uint8_t*)Bv + rb * ldb * 2;
  uint32_t oa[NI], ob[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int r = 8 * i + (lane >> 3), ch = ((lane & 7) ^ (r & 7)) * 16;
    oa[i] = (uint32_t)((ra + r < M ? r : M - 1 - ra) * ldat * 2) + ch;
    ob[i] = (uint32_t)((rb + r < N ? r : N - 1 - rb) * ldb * 2) + ch;
  }
  const uint32_t lds0 = lds_addr(&sm[0][0]) + wave * NI * 1024;
  auto issue = [&](int64_t t, int buf, int i) {
    const uint32_t l = lds0 + buf * 2 * OP + i * 1024;
    copy16_to_lds(Ap + t * STAGE, oa[i], l);
    copy16_to_lds(Bp + t * STAGE, ob[i], l + OP);
  };

  f4 acc[TA][TA];
#pragma unroll
  for (int a = 0; a < TA; ++a)
#pragma unroll
    for (int b = 0; b < TA; ++b) acc[a][b] = f4{0, 0, 0, 0};
  u16x8 fa0[TA], fb0[TA], fa1[TA], fb1[TA];
  int fo[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) fo[h] = g16 * STAGE + (((4 * h + q) ^ (g16 & 7)) * 16);
  auto frag = [&](int buf, int h, int i, u16x8* fa, u16x8* fb) {
    fb[i] = *(const u16x8*)(&sm[buf][OP + wn * TA * 16 * STAGE + fo[h]] + i * 16 * STAGE);
    fa[i] = *(const u16x8*)(&sm[buf][wm * TA * 16 * STAGE + fo[h]] + i * 16 * STAGE);
  };
  auto mma = [&](int a, const u16x8* fa, const u16x8* fb) {
#pragma unroll
    for (int b = 0; b < TA; ++b) {
      if constexpr (P == BF16)
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fb[b]),
                                                             __builtin_bit_cast(bf16x8, fa[a]), acc[a][b], 0, 0, 0);
      else
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, fb[b]),
                                                            __builtin_bit_cast(f16x8, fa[a]), acc[a][b], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  const int64_t stages = K * 2 / STAGE;
  if (stages > 0) {
#pragma unroll
    for (int i = 0; i < NI; ++i) issue(0, 0, i);
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
#pragma unroll
    for (int i = 0; i < TA; ++i) frag(0, 0, i, fa0, fb0);
    if (stages > 1) {
#pragma unroll
      for (int i = 0; i < NI; ++i) issue(1, 1, i);
    }
    auto stage = [&](int64_t t, int buf, auto more) {
#pragma unroll
      for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TA; ++b) asm volatile("" : "+a"(acc[a][b]));
#pragma unroll
      for (int i = 0; i < TA; ++i) {
        frag(buf, 1, i, fa1, fb1);
        mma(i, fa0, fb0);
      }
      // this stage's last reads are done and the next one's copies are in
      asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
      wait_vmcnt<0>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" : : : "memory");
#pragma unroll
      for (int i = 0; i < TA; ++i) {
        frag(buf ^ 1, 0, i, fa0, fb0);
        if (decltype(more)::value) issue(t + 2, buf, i);
        mma(i, fa1, fb1);
      }
    };
    int64_t t = 0;
    for (; t + 2 < stages; ++t) stage(t, t & 1, std::true_type{});
    for (; t < stages; ++t) stage(t, t & 1, std::false_type{});
  }
  lowp_store<TA, TA>(acc, alpha, beta, Cv, ldc, cprec, r0 + wm * TA * 16 + g16, c0 + wn * TA * 16 + 4 * q, M, N,
                     r0 + BM <= M && c0 + BM <= N);
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

// 256 x 256 blocks (two thirds of the LDS traffic per product of the 128 x 128 ones:
// half the stores, three quarters of the fragment reads; eight waves of 128 x 64) once they fill the chip; a launch that leaves more than a
// fifth of its last round of 256 CUs idle runs 128 x 128 blocks (four waves of 64 x
// 64, two workgroups per CU).
static bool large_blocks(int64_t m, int64_t n) {
  const int64_t blocks = ((m + 255) / 256) * ((n + 255) / 256), rounds = (blocks + 255) / 256;
  return blocks * 5 >= rounds * 256 * 4;
}

// BF16, FP16: a round of 256 blocks of k_gemm_lowp_big takes as long as one of 512
// small blocks (n = 2816, 121 and 484 of them: 76 and 83 us) and brings twice the
// products, so it is taken where the small ones need a second round (n = 3072: 81
// and 128 us; 4100: 219 and 276; 5120: 229 and 383; 5888: 379 and 548; small ones
// 23 and big ones 27 us at 2816 x 2816 x 128).  Its one wave per SIMD starts and
// ends with nothing beside it, which pays from k = 512 (8192 x 8192 x 1024: 152 us,
// eight waves 167; x 512: 110 and 111; x 256: 90 and 81; x 64: 69 and 63).  Long thin
// shapes, whole calls, against the 128 x 128 or whole-block kernels that came before
// it: 65536 x 130 x 1024 157 -> 52 us, 131072 x 64 x 512 91 -> 62, x 4096 645 -> 241, 16
// x 131072 x 1024 156 -> 87, 33000 x 257 x 1024 151 -> 68, 65536 x 256 x 1024 61 -> 52.  Its
// copies hold 63 rows of an operand in a 32-bit offset.
static bool big_blocks(int prec, int64_t m, int64_t n, int64_t k, int64_t ld) {
  return prec != F8 && k % (STAGE / 2) == 0 && ((m + 127) / 128) * ((n + 127) / 128) > 512 && k >= 512 && ld <= (INT64_C(1) << 25);
}

// k per stage of the 16/8-bit product
int gemm_lowp_kstage(int prec) { return STAGE / (prec == F8 ? 1 : 2); }

bool gemm_lowp_whole_stages(int prec, int64_t m, int64_t n, int64_t k) {
  const int64_t st = gemm_lowp_kstage(prec), kp = (k + st - 1) / st * st;
  return big_blocks(prec, m, n, kp, kp);
}

hipError_t launch_gemm_lowp(int prec, int64_t m, int64_t n, int64_t k, double alpha, const void* AT, int64_t ldat,
                            const int8_t* sA, int64_t mbA, int sa_kmajor, const void* B, int64_t ldb,
                            const int8_t* sB, int64_t mbB, int sb_kmajor, double beta, void* C, int64_t ldc, int cprec,
                            hipStream_t s) {
  const int es = prec == F8 ? 1 : 2;
  const bool tail = k % (STAGE / es) != 0;
  if ((ldat * es) % 16 != 0 || (ldb * es) % 16 != 0 || (uintptr_t)AT % 16 != 0 ||
      (uintptr_t)B % 16 != 0)
    return hipErrorInvalidValue;
#define MPCR_LOWP_T(P, WM, WN, TA, TB, PAD, TAIL)                                                                     \
  k_gemm_lowp<P, WM, WN, TA, TB, PAD, TAIL>                                                                           \
      <<<dim3((unsigned)((m + 16 * TA * WM - 1) / (16 * TA * WM)), (unsigned)((n + 16 * TB * WN - 1) / (16 * TB * WN))), \
         64 * WM * WN, 0, s>>>(m, n, k, alpha, AT, ldat, sA, mbA, sa_kmajor, B, ldb, sB, mbB, sb_kmajor, beta, C, ldc, \
                               cprec)
#define MPCR_LOWP(P, WM, WN, TA, TB, PAD)                \
  if (tail) MPCR_LOWP_T(P, WM, WN, TA, TB, PAD, true);   \
  else MPCR_LOWP_T(P, WM, WN, TA, TB, PAD, false)
  if (big_blocks(prec, m, n, k, ldat > ldb ? ldat : ldb)) {
    const dim3 grid((unsigned)((m + LOWP_BIG - 1) / LOWP_BIG), (unsigned)((n + LOWP_BIG - 1) / LOWP_BIG));
    if (prec == BF16) k_gemm_lowp_big<BF16><<<grid, 256, 0, s>>>(m, n, k, alpha, AT, ldat, B, ldb, beta, C, ldc, cprec);
    else k_gemm_lowp_big<F16><<<grid, 256, 0, s>>>(m, n, k, alpha, AT, ldat, B, ldb, beta, C, ldc, cprec);
  } else if (large_blocks(m, n)) {
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
#undef MPCR_LOWP_T
  return hipGetLastError();
}

template <int P, int WM, int WN, int FM, int FN, int BK>
static void run_gemm(int transA, int transB, int64_t m, int64_t n, int64_t k, double alpha, const void* A, int64_t lda,
                     const void* B, int64_t ldb, double beta, void* C, int64_t ldc, int cprec, hipStream_t s) {
  constexpr int BM = 16 * FM * WM, BN = 16 * FN * WN;
  const dim3 grid((unsigned)((m + BM - 1) / BM), (unsigned)((n + BN - 1) / BN));
#define MPCR_GEMM(TA, TB) \
  k_gemm<P, WM, WN, FM, FN, BK, TA, TB><<<grid, 64 * WM * WN, 0, s>>>(m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, cprec)
  if (transA) {
    if (transB) MPCR_GEMM(true, true);
    else MPCR_GEMM(true, false);
  } else {
    if (transB) MPCR_GEMM(false, true);
    else MPCR_GEMM(false, false);
  }
#undef MPCR_GEMM
}

hipError_t launch_gemm(int prec, int transA, int transB, int64_t m, int64_t n, int64_t k, double alpha, const void* A,
                       int64_t lda, const void* B, int64_t ldb, double beta, void* C, int64_t ldc, int cprec,
                       hipStream_t s) {
  // 64 x 64 blocks (four waves of 32 x 32): every size divides well over the 256
  // CUs and several workgroups share one.  FP32 blocks of 128 x 128 (waves of 64 x
  // 64, half the LDS reads per product) run 1.09 times as fast per element once
  // there are two rounds of them (n = 4096: 1056 us, 64-blocks 1154; n = 3000: 653
  // and 537; n = 2048, one round: 179 and 172), so they are taken where what they
  // waste in their last round is less than that.
  auto rounds = [&](int64_t bs) { return (((m + bs - 1) / bs) * ((n + bs - 1) / bs) + 255) / 256; };
  const bool large = rounds(128) >= 2 && rounds(128) * 400 <= rounds(64) * 109;
  switch (prec) {
    case F64: run_gemm<F64, 2, 2, 2, 2, 16>(transA, transB, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, cprec, s); break;
    case F32:
      if (large) run_gemm<F32, 2, 2, 4, 4, 16>(transA, transB, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, cprec, s);
      else run_gemm<F32, 2, 2, 2, 2, 16>(transA, transB, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, cprec, s);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace mpcr
