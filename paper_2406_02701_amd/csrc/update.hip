// Tile updates C(i,j) -= A(i,k) B(j,k)^T of FP64 and FP32 tiles (gfx950), and of
// BF16 tiles from packed panels.
//
// The update runs in the output tile's format; operands in another format are
// converted on load (widening exact, narrowing round-to-nearest-even).
#include <type_traits>

#include "mpcr_internal.h"

namespace mpcr {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

template <int CF> struct CTraits;
template <> struct CTraits<F64> { using T = double; };
template <> struct CTraits<F32> { using T = float; };

constexpr int UBM = 128;

// Four consecutive elements (idx % 4 == 0) of a tile stored in format SF,
// converted to the compute type of CF with one vector load.
template <int CF, int SF>
__device__ __forceinline__ void load4(const void* p, int64_t idx, typename CTraits<CF>::T out[4]) {
  using T = typename CTraits<CF>::T;
  if constexpr (SF == F64) {
    const double4 v = *(const double4*)((const double*)p + idx);
    const double w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r] = (CF == F64) ? (T)w[r] : (T)to_f32(w[r]);
  } else if constexpr (SF == F32) {
    const float4 v = *(const float4*)((const float*)p + idx);
    out[0] = (T)v.x; out[1] = (T)v.y; out[2] = (T)v.z; out[3] = (T)v.w;
  } else if constexpr (SF == F16 || SF == BF16) {
    const ushort4 v = *(const ushort4*)((const uint16_t*)p + idx);
    const uint16_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r] = (T)(SF == F16 ? f16_to_f32(w[r]) : bf16_to_f32(w[r]));
  } else {
    const uchar4 v = *(const uchar4*)((const uint8_t*)p + idx);
    const uint8_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r] = (T)e4m3_to_f32(w[r]);
  }
}

// four elements of an FP32 or BF16 tile, and their update c - acc rounded once
template <int CF> using CElem = typename std::conditional<CF == F32, float, uint16_t>::type;
template <int CF> using CVec = CElem<CF> __attribute__((ext_vector_type(4)));
template <int CF>
__device__ __forceinline__ CVec<CF> sub4(CVec<CF> c, f4 acc) {
  CVec<CF> o;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if constexpr (CF == F32) o[r] = to_f32((double)c[r] - (double)acc[r]);
    else o[r] = to_bf16((double)bf16_to_f32(c[r]) - (double)acc[r]);
  }
  return o;
}

// Operands staged k-major in LDS ([k][m]), double-buffered, one barrier per
// chunk of 16 k; fragments are contiguous across lanes.  The main loop is instantiated per pair of operand
// formats (one branch per workgroup), so each variant holds only its own
// staging registers.  The FP64 MFMA takes the B fragment first: a lane's
// results then lie in one row of C, and the 16 lanes of a group in 16
// consecutive rows of a column (with A first a store touched 16 columns); the
// FP32 one takes A first, which gives a lane four consecutive rows.
//
// FP64 shapes.  Large launches: 128 x 128 blocks, 8 waves of 64 x 32, two
// workgroups per CU (the FP64 MFMA is slow enough that more waves per CU, not
// more work per wave, hides the staging): 65 TF/s on 2016 updates of 512-tiles
// (the library product of 8192^2 reaches 77), where one workgroup of larger
// waves per CU stays at 53.  Launches whose 128-blocks do not go round the chip
// a few times: 64 x 64 blocks, 4 waves of 32 x 32, which split the same work
// four times finer: 6 updates of 512-tiles 78 -> 46 us, 36 updates 204 -> 171 us,
// 210 updates the other way, 922 against 951 us.  Every element of C sums its products in the same order in
// both, so the results are the same bits.
// FP32 (the plain MFMA of mpcr_ctx_set_fp32_split(ctx, 0)): 4 waves of 64 x 64,
// four workgroups per CU.
template <int CF, bool SMALL> struct KMajor {
  using T = typename CTraits<CF>::T;
  static constexpr int NW = (CF == F64 && !SMALL) ? 8 : 4;  // waves per workgroup
  static constexpr int WM = 2;                              // waves along m
  static constexpr int WN = NW / WM;
  static constexpr int BM = SMALL ? 64 : UBM;               // block of C
  static constexpr int TM = BM / WM, TN = BM / WN;          // per-wave block
  static constexpr int FM = TM / 16, FN = TN / 16;          // MFMA tiles per wave
  static constexpr int NT = NW * 64;
  static constexpr int BK = 16;
  static constexpr bool AHEAD = CF == F64;                  // fragments one k step ahead (the large blocks have no registers left)
  // row padding: a fragment read covers 4 consecutive k rows of 16 elements;
  // the padding puts those rows on disjoint LDS banks
  static constexpr int PAD = 16;
  static constexpr int LD = BM * BK / 4 / NT;  // 4-element loads per thread per operand
  using Acc = typename std::conditional<CF == F64, d4, f4>::type;
  using Buf = T[2][BK][BM + PAD];
};

template <int CF, bool SMALL, int FA, int FB>
__device__ __forceinline__ void kmajor_mainloop(const void* Ap, const void* Bp, double ma, double mb, int nb,
                                                int64_t arow0, int64_t brow0, typename KMajor<CF, SMALL>::Buf& As,
                                                typename KMajor<CF, SMALL>::Buf& Bs,
                                                typename KMajor<CF, SMALL>::Acc (&acc)[KMajor<CF, SMALL>::FM]
                                                                                      [KMajor<CF, SMALL>::FN]) {
  using K = KMajor<CF, SMALL>;
  using T = typename K::T;
  constexpr int BK = K::BK, LD = K::LD, NT = K::NT, BM = K::BM;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % K::WM, wn = wave / K::WM;
  T ra[LD][4], rb[LD][4];
  // load e = tid + NT g: rows 4 (e % (BM / 4)) .. +3 of column e / (BM / 4) of the chunk
  auto gload = [&](int kk) {
#pragma unroll
    for (int g = 0; g < LD; ++g) {
      const int e = tid + NT * g, r = (e % (BM / 4)) * 4, k = e / (BM / 4);
      load4<CF, FA>(Ap, (int64_t)(kk + k) * nb + arow0 + r, ra[g]);
      load4<CF, FB>(Bp, (int64_t)(kk + k) * nb + brow0 + r, rb[g]);
      if constexpr (FA == F8) {  // FP8 tiles hold codes of v 2^s: scale back (exact)
#pragma unroll
        for (int u = 0; u < 4; ++u) ra[g][u] = (T)((double)ra[g][u] * ma);
      }
      if constexpr (FB == F8) {
#pragma unroll
        for (int u = 0; u < 4; ++u) rb[g][u] = (T)((double)rb[g][u] * mb);
      }
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int g = 0; g < LD; ++g) {
      const int e = tid + NT * g, r = (e % (BM / 4)) * 4, k = e / (BM / 4);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        As[buf][k][r + u] = ra[g][u];
        Bs[buf][k][r + u] = rb[g][u];
      }
    }
  };
  T av[K::AHEAD ? 2 : 1][K::FM], bv[K::AHEAD ? 2 : 1][K::FN];
  auto frag = [&](int buf, int k4, T (&a)[K::FM], T (&b)[K::FN]) {
#pragma unroll
    for (int x = 0; x < K::FM; ++x) a[x] = As[buf][k4 + (lane >> 4)][wm * K::TM + x * 16 + (lane & 15)];
#pragma unroll
    for (int y = 0; y < K::FN; ++y) b[y] = Bs[buf][k4 + (lane >> 4)][wn * K::TN + y * 16 + (lane & 15)];
  };
  gload(0);
  sstore(0);
  __syncthreads();
  int cur = 0;
  for (int kk = 0; kk < nb; kk += BK) {
    const bool more = kk + BK < nb;
    if (more) gload(kk + BK);
    if (K::AHEAD) frag(cur, 0, av[0], bv[0]);
#pragma unroll
    for (int s = 0; s < BK / 4; ++s) {
      const int c = K::AHEAD ? s & 1 : 0;
      if (!K::AHEAD) frag(cur, 4 * s, av[c], bv[c]);
      else if (s + 1 < BK / 4) frag(cur, 4 * (s + 1), av[c ^ 1], bv[c ^ 1]);
#pragma unroll
      for (int x = 0; x < K::FM; ++x)
#pragma unroll
        for (int y = 0; y < K::FN; ++y) {
          if constexpr (CF == F64)
            acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(bv[c][y], av[c][x], acc[x][y], 0, 0, 0);
          else
            acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[c][x], bv[c][y], acc[x][y], 0, 0, 0);
        }
    }
    if (more) sstore(cur ^ 1);
    __syncthreads();
    cur ^= 1;
  }
}

template <int CF, bool SMALL>
__global__ __launch_bounds__((KMajor<CF, SMALL>::NT)) __attribute__((amdgpu_waves_per_eu(2))) void
k_update_kmajor(TileView tv, int k, const GemmTask* tasks) {
  using K = KMajor<CF, SMALL>;
  __shared__ __attribute__((aligned(16))) typename K::Buf As;
  __shared__ __attribute__((aligned(16))) typename K::Buf Bs;

  const int nb = tv.nb;
  const int sub = nb / K::BM;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int task = lb / (sub * sub);
  const int blk = lb % (sub * sub);
  const int bm = blk % sub, bn = blk / sub;
  const GemmTask t = tasks[task];
  if (t.i == t.j && bn > bm) return;
  if (*tv.info) return;

  const void* Ap = tv.tile(t.i, k);
  const void* Bp = tv.tile(t.j, k);
  const int fa = tv.tfmt(t.i, k), fb = tv.tfmt(t.j, k);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave % K::WM, wn = wave / K::WM;
  const int64_t arow0 = (int64_t)bm * K::BM, brow0 = (int64_t)bn * K::BM;

  typename K::Acc acc[K::FM][K::FN];
#pragma unroll
  for (int a = 0; a < K::FM; ++a)
#pragma unroll
    for (int b = 0; b < K::FN; ++b) acc[a][b] = typename K::Acc{0, 0, 0, 0};

  // operand tiles in any format (codes 0..4; FP8 operands carry their scale)
  const double ma = tv.tmul(t.i, k), mb = tv.tmul(t.j, k);
#define MPCR_PAIR(FA, FB) \
  case FA * 5 + FB: kmajor_mainloop<CF, SMALL, FA, FB>(Ap, Bp, ma, mb, nb, arow0, brow0, As, Bs, acc); break;
#define MPCR_ROW(FA) MPCR_PAIR(FA, F64) MPCR_PAIR(FA, F32) MPCR_PAIR(FA, F16) MPCR_PAIR(FA, BF16) MPCR_PAIR(FA, F8)
  switch (fa * 5 + fb) {
    MPCR_ROW(F64)
    MPCR_ROW(F32)
    MPCR_ROW(F16)
    MPCR_ROW(BF16)
    MPCR_ROW(F8)
    default: break;
  }
#undef MPCR_ROW
#undef MPCR_PAIR

  // the output tile is in format CF; a row of tiles is read before the first of
  // them is written back (one trip to memory for all of it)
  using T = typename K::T;
  T* Cp = (T*)tv.tile(t.i, t.j);
  if constexpr (CF == F64) {
    const bool diag = (t.i == t.j);
#pragma unroll
    for (int a = 0; a < K::FM; ++a) {
      const int64_t R = arow0 + wm * K::TM + 16 * a + (lane & 15), C0 = brow0 + wn * K::TN + (lane >> 4);
      T c[K::FN][4];
#pragma unroll
      for (int b = 0; b < K::FN; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) c[b][r] = Cp[(C0 + 16 * b + 4 * r) * nb + R];
#pragma unroll
      for (int b = 0; b < K::FN; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t C = C0 + 16 * b + 4 * r;
          if (!diag || C <= R) Cp[C * nb + R] = c[b][r] - acc[a][b][r];
        }
    }
  } else {  // (never a diagonal tile: those are FP64)
#pragma unroll
    for (int a = 0; a < K::FM; ++a) {
      const int64_t R = arow0 + wm * K::TM + 16 * a + 4 * (lane >> 4), C0 = brow0 + wn * K::TN + (lane & 15);
      CVec<F32> c[K::FN];
#pragma unroll
      for (int b = 0; b < K::FN; ++b) c[b] = *(const CVec<F32>*)(Cp + (C0 + 16 * b) * nb + R);
#pragma unroll
      for (int b = 0; b < K::FN; ++b) *(CVec<F32>*)(Cp + (C0 + 16 * b) * nb + R) = sub4<F32>(c[b], acc[a][b]);
    }
  }
}

// FP64 updates of a few tiles: one 16 x 16 tile of C per wave (32 x 32 per
// workgroup), operands straight from memory, 32 k per batch with two batches in
// flight.  Such a launch lies on the critical path and cannot fill the chip, so
// what counts is the chain of one wave: nb / 4 dependent MFMAs and few trips to
// memory, no barriers.  Products are added in ascending k as in k_update_kmajor;
// with split_first those of the first task in two halves, as k_syrk_tile does.
// Measured, alone, 64 x 64 blocks -> this: one 256 tile 16.2 -> 7.3 us, eight 16.7
// -> 12.1, sixteen 17.3 -> 20.2; one 512 tile 27.9 -> 11.4, two 28.5 -> 20.2, four
// 30.1 -> 35.0.
// On one stream a step's FP64 tiles go in one launch (n = 1024 591 -> 568 us).
template <int F>
__device__ __forceinline__ void load_batch(const char* p, unsigned own, int64_t step, double (&v)[8]) {
#pragma unroll
  for (int u = 0; u < 8; ++u) v[u] = load_wide(p + u * step + own, F, 0);
}

__global__ __launch_bounds__(256, 4) void k_update_direct(TileView tv, int k, const GemmTask* tasks, int split_first) {
  const int nb = tv.nb, sub = nb / 32, task = blockIdx.x / (sub * sub), blk = blockIdx.x % (sub * sub);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q = lane >> 4, i = lane & 15;
  const GemmTask t = tasks[task];
  const int R0 = blk % sub * 32 + 16 * (wave & 1), C0 = blk / sub * 32 + 16 * (wave >> 1);
  if (t.i == t.j && C0 > R0) return;
  if (*tv.info) return;
  __builtin_amdgcn_s_setprio(2);
  const int fa = __builtin_amdgcn_readfirstlane(tv.tfmt(t.i, k)), fb = __builtin_amdgcn_readfirstlane(tv.tfmt(t.j, k));
  const double ma = tv.tmul(t.i, k), mb = tv.tmul(t.j, k);
  // one operand: its rows' first element, the lane's offset and the way from one k4 step to the next, in bytes
  struct Operand {
    const char* p;
    unsigned own;
    int64_t step;
  };
  auto operand = [&](int ti, int f, int row) {
    const int es = fmt_bytes(f);
    return Operand{(const char*)tv.tile(ti, k) + row * es, (unsigned)((q * nb + i) * es), (int64_t)4 * nb * es};
  };
  Operand a = operand(t.i, fa, R0), b = operand(t.j, fb, C0);
  auto load = [&](Operand& o, int f, double mul, double (&v)[8]) {
    switch (f) {
      case F64: load_batch<F64>(o.p, o.own, o.step, v); break;
      case F32: load_batch<F32>(o.p, o.own, o.step, v); break;
      case F16: load_batch<F16>(o.p, o.own, o.step, v); break;
      case BF16: load_batch<BF16>(o.p, o.own, o.step, v); break;
      default:
        load_batch<F8>(o.p, o.own, o.step, v);
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] *= mul;
    }
    o.p += 8 * o.step;
  };
  double* C = (double*)tv.tile(t.i, t.j) + (int64_t)(C0 + q) * nb + R0 + i;
  double old[4], va[2][8], vb[2][8];
  d4 acc = {0, 0, 0, 0}, half = {0, 0, 0, 0};
  const int mid = split_first && task == 0 ? nb / 2 : nb;
  load(a, fa, ma, va[0]);
  load(b, fb, mb, vb[0]);
  load(a, fa, ma, va[1]);
  load(b, fb, mb, vb[1]);
#pragma unroll
  for (int r = 0; r < 4; ++r) old[r] = C[(int64_t)(4 * r) * nb];
  auto product = [&](int s) {
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(vb[s][u], va[s][u], acc, 0, 0, 0);
  };
  for (int n = 0; n < nb; n += 64) {
    const bool more = n + 64 < nb;
    if (n == mid) {
      half = acc;
      acc = d4{0, 0, 0, 0};
    }
    product(0);
    if (more) {
      load(a, fa, ma, va[0]);
      load(b, fb, mb, vb[0]);
    }
    product(1);
    if (more) {
      load(a, fa, ma, va[1]);
      load(b, fb, mb, vb[1]);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) C[(int64_t)(4 * r) * nb] = old[r] - (mid < nb ? half[r] + acc[r] : acc[r]);
}

// fewer 128 x 128 blocks than this: 64 x 64 ones (three rounds of two
// workgroups per CU; measured on either side, see KMajor)
constexpr int SMALL_UPDATE_MAX = 1536;
// up to this many 32 x 32 blocks (two per CU): one workgroup each (measured on
// either side, see k_update_direct)
constexpr int DIRECT_UPDATE_MAX = 512;

bool direct_update_fits(int nb, int ntasks) {
  return ntasks * (int64_t)(nb / 32) * (nb / 32) <= DIRECT_UPDATE_MAX;
}

hipError_t launch_tile_update_direct(const TileView& tv, int k, const GemmTask* tasks, int ntasks, bool split_first,
                                     hipStream_t s) {
  const int sub = tv.nb / 32;
  k_update_direct<<<(unsigned)(ntasks * sub * sub), 256, 0, s>>>(tv, k, tasks, split_first);
  return hipGetLastError();
}

hipError_t launch_tile_update(const TileView& tv, int k, int cfmt, const GemmTask* tasks, int ntasks, hipStream_t s) {
  if (ntasks == 0) return hipSuccess;
  const int64_t sub = tv.nb / UBM, blocks = ntasks * sub * sub;
  switch (cfmt) {
    case F64:
      if (direct_update_fits(tv.nb, ntasks)) return launch_tile_update_direct(tv, k, tasks, ntasks, false, s);
      if (blocks < SMALL_UPDATE_MAX)
        k_update_kmajor<F64, true><<<(unsigned)(4 * blocks), KMajor<F64, true>::NT, 0, s>>>(tv, k, tasks);
      else
        k_update_kmajor<F64, false><<<(unsigned)blocks, KMajor<F64, false>::NT, 0, s>>>(tv, k, tasks);
      break;
    case F32: k_update_kmajor<F32, false><<<(unsigned)blocks, KMajor<F32, false>::NT, 0, s>>>(tv, k, tasks); break;
    default: return launch_tile_update_16(tv, k, cfmt, tasks, ntasks, s);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// FP32 output tiles through the BF16 MFMA.  gfx950's dense BF16 rate is 16
// times its FP32 rate, so an FP32 product can be formed from BF16 pieces:
// each operand, converted to FP32 as in the FP32 update, is split exactly
// into three BF16 numbers x = h + m + l (h = bf16(x), m = bf16(x - h),
// l = x - h - m; every difference is exact by Sterbenz's lemma and l needs at
// most 8 significant bits), and a b is accumulated as
//   ah bh + ah bm + am bh + ah bl + al bh + am bm
// in FP32 on v_mfma_f32_16x16x32_bf16 (which returns the exact FP32-rounded
// sums).  The three dropped products am bl + al bm + al bl are below
// 2^-23 |a b|, so every update keeps FP32-level accuracy; the output tile is
// rounded to FP32 as in the FP32 update.  One 128 x 128 block of C per
// workgroup, 8 waves of 64 x 32, k chunks of 32; the three planes of both
// operands (61 KB) sit in one LDS buffer so that two workgroups share a CU.
// ---------------------------------------------------------------------------
constexpr int SBK = 32;          // k per chunk
constexpr int SLDK = SBK + 8;    // LDS row (halfwords): 80-byte rows put the 16 rows of a fragment read on disjoint banks

__device__ __forceinline__ void split3_bf16(float x, uint16_t& h, uint16_t& m, uint16_t& l) {
  // finite inputs: round to nearest even by adding half an ulp (ties to even)
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  h = (uint16_t)(u >> 16);
  const float r1 = x - __uint_as_float((uint32_t)h << 16);
  uint32_t v = __float_as_uint(r1);
  v += 0x7fffu + ((v >> 16) & 1u);
  m = (uint16_t)(v >> 16);
  const float r2 = r1 - __uint_as_float((uint32_t)m << 16);
  l = (uint16_t)(__float_as_uint(r2) >> 16);  // r2 has at most 8 significant bits: exact
}

// element idx of a tile (format SF) converted to FP32 (FP8 codes scaled back
// by mul = 2^-s)
template <int SF>
__device__ __forceinline__ float load1_f32(const void* p, int64_t idx, double mul) {
  if constexpr (SF == F64) return to_f32(((const double*)p)[idx]);
  else if constexpr (SF == F32) return ((const float*)p)[idx];
  else if constexpr (SF == F16) return f16_to_f32(((const uint16_t*)p)[idx]);
  else if constexpr (SF == BF16) return bf16_to_f32(((const uint16_t*)p)[idx]);
  else return to_f32((double)e4m3_to_f32(((const uint8_t*)p)[idx]) * mul);
}

// Split panels: after the TRSM of step k, every panel tile (i, k) is converted
// to FP32 and split once into its three BF16 planes, stored for the update
// kernel in chunks of 32 k: plane p of panel tile q = i - k - 1 at
//   out3[(q * 3 + p) * nb^2 + (c * nb + row) * 32 + kk]   (k = 32 c + kk),
// so a 128-row block of one chunk is 8 contiguous KB.  The FP32 updates of the
// step then copy planes instead of splitting every operand in every block.
// outb (when not NULL) receives, in the same layout, each element rounded once
// to BF16 from its stored format: the operands of the step's BF16 updates.
template <int SF>
__device__ __forceinline__ uint16_t load1_bf16(const void* p, int64_t idx, double mul) {
  if constexpr (SF == BF16) return ((const uint16_t*)p)[idx];
  else if constexpr (SF == F32) return f32_to_bf16_rne(((const float*)p)[idx]);
  else if constexpr (SF == F64) return to_bf16(((const double*)p)[idx]);
  else if constexpr (SF == F16) return to_bf16((double)f16_to_f32(((const uint16_t*)p)[idx]));
  else return to_bf16((double)e4m3_to_f32(((const uint8_t*)p)[idx]) * mul);
}

__global__ __launch_bounds__(512) void k_pack_split(TileView tv, int k, uint16_t* out3, uint16_t* outb) {
  const int nb = tv.nb, nch = nb / SBK, nrb = nb / UBM;
  const int b = blockIdx.x;
  const int q = b / (nch * nrb), c = (b / nrb) % nch, rb = b % nrb;
  const int i = k + 1 + q;
  const void* P = tv.tile(i, k);
  const int f = tv.tfmt(i, k);
  const double mul = tv.tmul(i, k);
  const int mr = threadIdx.x & (UBM - 1), k0 = 8 * (threadIdx.x / UBM);
  const int64_t row = (int64_t)rb * UBM + mr;
  const int64_t nb2 = (int64_t)nb * nb;
  const int64_t at = ((int64_t)c * nb + row) * SBK + k0;
  float v[8];
  u16x8 bv;
  auto load = [&](auto tag) {
    constexpr int SF = decltype(tag)::value;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t idx = (int64_t)(SBK * c + k0 + e) * nb + row;
      if (out3) v[e] = load1_f32<SF>(P, idx, mul);
      if (outb) bv[e] = load1_bf16<SF>(P, idx, mul);
    }
  };
  switch (f) {
    case F64: load(std::integral_constant<int, F64>{}); break;
    case F32: load(std::integral_constant<int, F32>{}); break;
    case F16: load(std::integral_constant<int, F16>{}); break;
    case BF16: load(std::integral_constant<int, BF16>{}); break;
    default: load(std::integral_constant<int, F8>{}); break;
  }
  if (outb) *(u16x8*)(outb + (int64_t)q * nb2 + at) = bv;
  if (out3) {
    u16x8 h, m, l;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      uint16_t a, bb, cc;
      split3_bf16(v[e], a, bb, cc);
      h[e] = a;
      m[e] = bb;
      l[e] = cc;
    }
    uint16_t* o = out3 + (int64_t)q * 3 * nb2 + at;
    *(u16x8*)o = h;
    *(u16x8*)(o + nb2) = m;
    *(u16x8*)(o + 2 * nb2) = l;
  }
}

hipError_t launch_pack_split(const TileView& tv, int k, uint16_t* out3, uint16_t* outb, hipStream_t s) {
  const int cnt = tv.nt - k - 1;
  if (cnt <= 0 || (!out3 && !outb)) return hipSuccess;
  k_pack_split<<<cnt * (tv.nb / SBK) * (tv.nb / UBM), 512, 0, s>>>(tv, k, out3, outb);
  return hipGetLastError();
}

// Updates from the packed panels of step k (see k_pack_split), planes copied
// with 16-byte loads (four per row of a chunk).  NPL = 3: FP32 output tiles,
// the six split products; NPL = 1: BF16 output tiles, one BF16 product per
// fragment pair on operands rounded once to BF16 (the same k order of MFMAs as
// k_update_mmajor<BF16>, so the same results).  128 x 128 blocks of 8 waves of 64 x
// 32: the three planes (6 bytes per operand element) make the operand stream, not
// the LDS or the MFMA, the limit, which is why large FP32 launches take
// k_update_split_big.
constexpr int SPLIT_WAVES = 8;

template <int NW, int NPL>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW == 8 ? 4 : 2))) void
k_update_packed(TileView tv, int k, const GemmTask* tasks, const uint16_t* split) {
  constexpr int NT = 64 * NW;
  constexpr int WN = NW / 2;             // waves along n (2 along m)
  constexpr int FY = (UBM / WN) / 16;    // 16-column MFMA tiles per wave along n
  constexpr int G = NPL * UBM * 4 / NT;  // 16-byte vectors per thread per operand and chunk
  constexpr int CF = NPL == 3 ? F32 : BF16;
  __shared__ __attribute__((aligned(16))) uint16_t As[NPL][UBM][SLDK];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[NPL][UBM][SLDK];

  const int nb = tv.nb;
  const int sub = nb / UBM;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int task = lb / (sub * sub);
  const int blk = lb % (sub * sub);
  const int bm = blk % sub, bn = blk / sub;
  const GemmTask t = tasks[task];
  if (t.i == t.j && bn > bm) return;
  if (*tv.info) return;

  const int64_t nb2 = (int64_t)nb * nb;
  const uint16_t* Ap = split + (int64_t)(t.i - k - 1) * NPL * nb2;
  const uint16_t* Bp = split + (int64_t)(t.j - k - 1) * NPL * nb2;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const int64_t arow0 = (int64_t)bm * UBM, brow0 = (int64_t)bn * UBM;

  f4 acc[4][FY];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < FY; ++y) acc[x][y] = f4{0, 0, 0, 0};

  // vector v = tid + NT g: plane v / 512, row (v % 512) / 4, k offset 8 (v % 4)
  u16x8 ra[G], rb[G];
  auto gload = [&](int kk) {
    const int64_t c = kk / SBK;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int v = tid + NT * g, p = v / (UBM * 4), r = (v % (UBM * 4)) >> 2, k0 = 8 * (v & 3);
      ra[g] = *(const u16x8*)(Ap + p * nb2 + (c * nb + arow0 + r) * SBK + k0);
      rb[g] = *(const u16x8*)(Bp + p * nb2 + (c * nb + brow0 + r) * SBK + k0);
    }
  };
  auto sstore = [&]() {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int v = tid + NT * g, p = v / (UBM * 4), r = (v % (UBM * 4)) >> 2, k0 = 8 * (v & 3);
      *(u16x8*)&As[p][r][k0] = ra[g];
      *(u16x8*)&Bs[p][r][k0] = rb[g];
    }
  };
  gload(0);
  sstore();
  __syncthreads();
  const int kq8 = 8 * (lane >> 4);
  for (int kk = 0; kk < nb; kk += SBK) {
    const bool more = kk + SBK < nb;
    if (more) gload(kk + SBK);
    u16x8 a[NPL][4], b[NPL][FY];
#pragma unroll
    for (int p = 0; p < NPL; ++p) {
#pragma unroll
      for (int x = 0; x < 4; ++x) a[p][x] = *(const u16x8*)&As[p][wm * 64 + x * 16 + (lane & 15)][kq8];
#pragma unroll
      for (int y = 0; y < FY; ++y) b[p][y] = *(const u16x8*)&Bs[p][wn * (16 * FY) + y * 16 + (lane & 15)][kq8];
    }
#define MPCR_MF(PA, PB)                                                                                   \
  acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[PA][x]),              \
                                                      __builtin_bit_cast(bf16x8, b[PB][y]), acc[x][y], 0, 0, 0)
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int y = 0; y < FY; ++y) {
        if constexpr (NPL == 3) {
          MPCR_MF(1, 1);
          MPCR_MF(0, 2);
          MPCR_MF(2, 0);
          MPCR_MF(0, 1);
          MPCR_MF(1, 0);
        }
        MPCR_MF(0, 0);
      }
#undef MPCR_MF
    if (more) {
      __syncthreads();
      sstore();
      __syncthreads();
    }
  }

  // a lane's four results of a tile are four consecutive rows of one column
  void* Cp = tv.tile(t.i, t.j);  // never a diagonal tile (those are FP64)
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    CVec<CF> c[FY];
    const int64_t R = arow0 + wm * 64 + x * 16 + 4 * (lane >> 4);
    auto at = [&](int y) { return (brow0 + wn * (16 * FY) + y * 16 + (lane & 15)) * nb + R; };
#pragma unroll
    for (int y = 0; y < FY; ++y) c[y] = *(const CVec<CF>*)((const CElem<CF>*)Cp + at(y));
#pragma unroll
    for (int y = 0; y < FY; ++y) *(CVec<CF>*)((CElem<CF>*)Cp + at(y)) = sub4<CF>(c[y], acc[x][y]);
  }
}

// The FP32 update (three planes) on 256 x 128 blocks of C, eight waves of
// 64 x 64, one workgroup per CU.  The 128 x 128 kernel above reads 193 KB of
// LDS per 1536 cycles of MFMA (the LDS rate); here a chunk's 3072 cycles of
// MFMA come with 192 KB of fragment reads and 72 KB of copies, two thirds of
// that rate.  The planes go global -> LDS directly (no registers, no LDS
// stores): two stages of 72 KB, the next chunk's copies in flight during this
// chunk's products, one barrier per chunk.  A copy of 1 KB is 16 rows of 64
// bytes; its 16-byte granules are permuted within each row (lane l fetches
// granule (l % 4) ^ (l / 16) of row l / 4), so that the 16 rows of a fragment
// read hit disjoint banks.  Every element of C takes its products in the order
// of the 128 x 128 kernel: the same bits.
constexpr int BSM = 256, BSN = 128;                   // block of C
constexpr int BS_STAGE = 3 * (BSM + BSN) * SBK * 2;   // bytes of a stage

__global__ __launch_bounds__(512) void k_update_split_big(TileView tv, int k, const GemmTask* tasks,
                                                          const uint16_t* split) {
  __shared__ __attribute__((aligned(1024))) uint8_t sm[2][BS_STAGE];
  const int nb = tv.nb;
  const int subm = nb / BSM, subn = nb / BSN;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int task = lb / (subm * subn);
  const int blk = lb % (subm * subn);
  const int bm = blk % subm, bn = blk / subm;
  const GemmTask t = tasks[task];
  if (*tv.info) return;

  const int64_t pl = (int64_t)nb * nb * 2;  // bytes of a plane
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 3, wn = wave >> 2;
  const int lr = lane >> 4, lc = lane & 15;
  const int64_t arow0 = (int64_t)bm * BSM, brow0 = (int64_t)bn * BSN;
  // copies of 1 KB: wave w takes rows 16 w .. (and 128 + 16 w ..) of every plane of A, 16 w .. of B
  const uint8_t* Ap = (const uint8_t*)split + (int64_t)(t.i - k - 1) * 3 * pl + (arow0 + 16 * wave) * 64;
  const uint8_t* Bp = (const uint8_t*)split + (int64_t)(t.j - k - 1) * 3 * pl + (brow0 + 16 * wave) * 64;
  const uint32_t loff = (lane >> 2) * 64 + (((lane & 3) ^ (lane >> 4)) * 16);
  const uint32_t lds0 = lds_addr(&sm[0][0]) + wave * 1024;
  auto issue = [&](int c, int buf) {
    const int64_t ck = (int64_t)c * nb * 64;
    const uint32_t l = lds0 + buf * BS_STAGE;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      copy16_to_lds(Ap + p * pl + ck, loff, l + p * (BSM * 64));
      copy16_to_lds(Ap + p * pl + ck + 128 * 64, loff, l + p * (BSM * 64) + 8 * 1024);
      copy16_to_lds(Bp + p * pl + ck, loff, l + 3 * BSM * 64 + p * (BSN * 64));
    }
  };

  f4 acc[4][4];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) acc[x][y] = f4{0, 0, 0, 0};

  const int nch = nb / SBK;
  const int foff = (lc * 4 + (lr ^ (lc >> 2))) * 16;  // this lane's granule of a 16-row fragment
  issue(0, 0);
  for (int c = 0; c < nch; ++c) {
    const int buf = c & 1;
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
    if (c + 1 < nch) issue(c + 1, buf ^ 1);
    const uint8_t* As = &sm[buf][wm * 4 * 1024 + foff];
    const uint8_t* Bs = &sm[buf][3 * BSM * 64 + wn * 4 * 1024 + foff];
    u16x8 b[3][4];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int y = 0; y < 4; ++y) b[p][y] = *(const u16x8*)(Bs + p * (BSN * 64) + y * 1024);
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      u16x8 a[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) a[p] = *(const u16x8*)(As + p * (BSM * 64) + x * 1024);
#define MPCR_MF(PA, PB)                                                                                        \
  _Pragma("unroll") for (int y = 0; y < 4; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(           \
      __builtin_bit_cast(bf16x8, a[PA]), __builtin_bit_cast(bf16x8, b[PB][y]), acc[x][y], 0, 0, 0)
      MPCR_MF(1, 1);
      MPCR_MF(0, 2);
      MPCR_MF(2, 0);
      MPCR_MF(0, 1);
      MPCR_MF(1, 0);
      MPCR_MF(0, 0);
#undef MPCR_MF
    }
  }

  float* Cp = (float*)tv.tile(t.i, t.j);
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    CVec<F32> c[4];
    const int64_t R = arow0 + wm * 64 + x * 16 + 4 * lr;
    auto at = [&](int y) { return (brow0 + wn * 64 + y * 16 + lc) * nb + R; };
#pragma unroll
    for (int y = 0; y < 4; ++y) c[y] = *(const CVec<F32>*)(Cp + at(y));
#pragma unroll
    for (int y = 0; y < 4; ++y) *(CVec<F32>*)(Cp + at(y)) = sub4<F32>(c[y], acc[x][y]);
  }
}

// 128 x 128 blocks from which the 256 x 128 kernel is used.  A round of either is 512
// such blocks (two workgroups per CU of the small kernel, one of the big).  Launches
// alone, small -> big, 512-tiles: up to 256 blocks the small one, whose workgroups
// then have a CU each (128: 29 -> 38 us, 256: 33 -> 44); 272 to 512 the big one (320:
// 51 -> 47, 448: 49 -> 45); in the second round first the small one (576: 70 -> 78,
// 720: 72 -> 80), then the big one (880: 91 -> 83), and so on with less and less
// between them (1056: 112 -> 118, 1456: 139 -> 130, 2176: 213 -> 209, 2448: 239 ->
// 225, 3696: 374 -> 361; 256- and 1024-tiles alike).  No one line fits: at 512 the
// wrong one costs about a tenth of a launch below 0.1 ms, and the long launches get
// the big one.
constexpr int SPLIT_BIG_MIN = 512;

hipError_t launch_tile_update_packed(const TileView& tv, int k, int cfmt, const GemmTask* tasks, int ntasks,
                                     const uint16_t* planes, hipStream_t s) {
  if (ntasks == 0) return hipSuccess;
  const int sub = tv.nb / UBM;
  if (cfmt == F32 && tv.nb % BSM == 0 && ntasks * sub * sub >= SPLIT_BIG_MIN)
    k_update_split_big<<<ntasks * (tv.nb / BSM) * (tv.nb / BSN), 512, 0, s>>>(tv, k, tasks, planes);
  else if (cfmt == F32)
    k_update_packed<SPLIT_WAVES, 3><<<ntasks * sub * sub, 64 * SPLIT_WAVES, 0, s>>>(tv, k, tasks, planes);
  else if (cfmt == BF16)
    k_update_packed<8, 1><<<ntasks * sub * sub, 512, 0, s>>>(tv, k, tasks, planes);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mpcr
