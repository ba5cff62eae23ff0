// Tile Cholesky kernels (gfx950).
//
// Right-looking tile Cholesky over nb x nb tiles held in per-tile formats
// (the tiled multi-precision algorithm named in the paper's "Discussion and
// Future Work" section; the factor feeds the log-determinant and the solves
// of the MLE section):
//   POTRF  L_kk = chol(A_kk)                          FP64, one workgroup
//   TRSM   L_ik = A_ik L_kk^{-T}                      FP64 compute, rounded once to p(i,k)
//   SYRK   A_jj -= L_jk L_jk^T                        FP64 MFMA
//   GEMM   A_ij -= L_ik L_jk^T (i > j)                MFMA in the format of tile (i,j)
// Every kernel first checks the device info word and does nothing once a
// pivot has failed, so a whole factorisation can be queued without host syncs.
#include <type_traits>

#include "mpcr_internal.h"

namespace mpcr {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

// MFMA 16x16 lane layouts on gfx950 (checked with an in-bounds probe):
//   operands (f64 16x16x4, f32 16x16x4): lane l holds A[l%16][l/16], B[l/16][l%16]
//   operands (bf16/f16 16x16x32): lane l holds A[l%16][8(l/16) .. 8(l/16)+7], B likewise
//   result f32: lane l, register r -> D[4(l/16) + r][l%16]
//   result f64: lane l, register r -> D[l/16 + 4r][l%16]

// ---------------------------------------------------------------------------
// batched tile update  C(i,j) -= A(i,k) B(j,k)^T of 16-bit and FP8 tiles (FP64
// and FP32: update.hip), one 128 x 128 block of C per workgroup (4 waves,
// 2 x 2, each 64 x 64 = 4 x 4 MFMA tiles of 16 x 16)
// ---------------------------------------------------------------------------
constexpr int UBM = 128;

// C[idx] <- round_f(C[idx] - acc) for the epilogue, with a static format.
template <int F>
__device__ __forceinline__ void rmw_sub(void* Cp, int64_t idx, double acc) {
  if constexpr (F == F64) { double* c = (double*)Cp; c[idx] = c[idx] - acc; }
  else if constexpr (F == F32) { float* c = (float*)Cp; c[idx] = to_f32((double)c[idx] - acc); }
  else if constexpr (F == F16) { uint16_t* c = (uint16_t*)Cp; c[idx] = to_f16((double)f16_to_f32(c[idx]) - acc); }
  else if constexpr (F == BF16) { uint16_t* c = (uint16_t*)Cp; c[idx] = to_bf16((double)bf16_to_f32(c[idx]) - acc); }
  else { uint8_t* c = (uint8_t*)Cp; c[idx] = to_e4m3((double)e4m3_to_f32(c[idx]) - acc); }
}

// BF16 / FP16: operands staged m-major in LDS ([m][k]) so that each lane reads
// its 8 consecutive k values with one 16-byte load.  The column-major tiles
// are read 8 rows at a time (one vector load per column), converted to the
// compute format and scattered into 8 LDS rows; LDS is double-buffered and
// the main loop is instantiated per pair of operand formats.
template <int CF, int SF>
__device__ __forceinline__ void load8_16(const void* p, int64_t idx, uint16_t out[8], double mul) {
  auto cvt = [](double x) -> uint16_t { return CF == BF16 ? to_bf16(x) : to_f16(x); };
  if constexpr (SF == CF) {
    const u16x8 v = *(const u16x8*)((const uint16_t*)p + idx);
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = v[e];
  } else if constexpr (SF == F64) {
    const double4 v0 = *(const double4*)((const double*)p + idx), v1 = *(const double4*)((const double*)p + idx + 4);
    const double w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = cvt(w[e]);
  } else if constexpr (SF == F32) {
    const float4 v0 = *(const float4*)((const float*)p + idx), v1 = *(const float4*)((const float*)p + idx + 4);
    const float w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = CF == BF16 ? f32_to_bf16_rne(w[e]) : __builtin_bit_cast(uint16_t, (_Float16)w[e]);
  } else if constexpr (SF == F8) {  // codes of v 2^s: widen, scale back (mul = 2^-s), round once
    const uint2 v = *(const uint2*)((const uint8_t*)p + idx);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint8_t c = (uint8_t)(((e < 4 ? v.x : v.y) >> (8 * (e & 3))) & 0xffu);
      out[e] = cvt((double)e4m3_to_f32(c) * mul);
    }
  } else {  // the other 16-bit format: widen exactly, round once
    const u16x8 v = *(const u16x8*)((const uint16_t*)p + idx);
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = cvt((double)(SF == F16 ? f16_to_f32(v[e]) : bf16_to_f32(v[e])));
  }
}

constexpr int MBK = 64;        // k per chunk
constexpr int MLDK = MBK + 8;  // LDS row (halfwords)

template <int CF, int FA, int FB>
__device__ __forceinline__ void mmajor_mainloop(const void* Ap, const void* Bp, double ma, double mb, int nb,
                                                int64_t arow0, int64_t brow0,
                                                uint16_t (&As)[2][UBM][MLDK], uint16_t (&Bs)[2][UBM][MLDK],
                                                f4 (&acc)[4][4]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const int rg = tid & 15;  // rows 8 rg .. 8 rg + 7
  const int kq = tid >> 4;  // k = kq + 16 g
  uint16_t ra[4][8], rb[4][8];
  auto gload = [&](int kk) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int64_t col = kk + kq + 16 * g;
      load8_16<CF, FA>(Ap, col * nb + arow0 + 8 * rg, ra[g], ma);
      load8_16<CF, FB>(Bp, col * nb + brow0 + 8 * rg, rb[g], mb);
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        As[buf][8 * rg + e][kq + 16 * g] = ra[g][e];
        Bs[buf][8 * rg + e][kq + 16 * g] = rb[g][e];
      }
  };
  gload(0);
  sstore(0);
  __syncthreads();
  int cur = 0;
  for (int kk = 0; kk < nb; kk += MBK) {
    const bool more = kk + MBK < nb;
    if (more) gload(kk + MBK);
#pragma unroll
    for (int k32 = 0; k32 < MBK; k32 += 32) {
      u16x8 av[4], bv[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) av[a] = *(const u16x8*)&As[cur][wm * 64 + a * 16 + (lane & 15)][k32 + 8 * (lane >> 4)];
#pragma unroll
      for (int b = 0; b < 4; ++b) bv[b] = *(const u16x8*)&Bs[cur][wn * 64 + b * 16 + (lane & 15)][k32 + 8 * (lane >> 4)];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          if constexpr (CF == BF16)
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[a]),
                                                                 __builtin_bit_cast(bf16x8, bv[b]), acc[a][b], 0, 0, 0);
          else
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, av[a]),
                                                                __builtin_bit_cast(f16x8, bv[b]), acc[a][b], 0, 0, 0);
        }
    }
    if (more) sstore(cur ^ 1);
    __syncthreads();
    cur ^= 1;
  }
}

template <int CF>
__global__ __launch_bounds__(256) void k_update_mmajor(TileView tv, int k, const GemmTask* tasks) {
  __shared__ __attribute__((aligned(16))) uint16_t As[2][UBM][MLDK];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][UBM][MLDK];

  const int nb = tv.nb;
  const int sub = nb / UBM;
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
  const int wm = wave & 1, wn = wave >> 1;
  const int64_t arow0 = (int64_t)bm * UBM, brow0 = (int64_t)bn * UBM;

  f4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f4{0, 0, 0, 0};

  const double ma = tv.tmul(t.i, k), mb = tv.tmul(t.j, k);
#define MPCR_PAIR(FA, FB) \
  case FA * 5 + FB: mmajor_mainloop<CF, FA, FB>(Ap, Bp, ma, mb, nb, arow0, brow0, As, Bs, acc); break;
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

  void* Cp = tv.tile(t.i, t.j);  // in format CF (the update runs in the output tile's format)
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int64_t R = arow0 + wm * 64 + a * 16 + 4 * (lane >> 4) + r;
        int64_t C = brow0 + wn * 64 + b * 16 + (lane & 15);
        rmw_sub<CF>(Cp, C * nb + R, (double)acc[a][b][r]);
      }
}

// ---------------------------------------------------------------------------
// Updates of FP8 output tiles (the update runs in the output tile's format):
// both operands are converted to FP8 on load with the scale of their own tile
// (a stored FP8 tile keeps its codes; any other operand tile (i, k) is
// quantised with the scale that its largest magnitude pamax[i] gives), the
// products accumulate in FP32 through v_mfma_f32_16x16x32_fp8_fp8, and the new
// tile C - 2^-(sA+sB) acc is formed in FP64 and staged in FP32 by round-to-odd
// with its largest magnitude; k_requant_f8 then rounds it once to FP8 with the
// scale of that maximum (the two roundings equal one: FP32 keeps two more bits
// than E4M3 needs).
// ---------------------------------------------------------------------------
constexpr int FBK = 128;           // k per chunk
constexpr int FLDK = FBK + 16;     // LDS row (bytes)

template <int SF>
__device__ __forceinline__ void load8_f8(const void* p, int64_t idx, uint8_t out[8], double qs) {
  if constexpr (SF == F8) {
    const uint2 v = *(const uint2*)((const uint8_t*)p + idx);
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = (uint8_t)(((e < 4 ? v.x : v.y) >> (8 * (e & 3))) & 0xffu);
  } else if constexpr (SF == F64) {
    const double4 v0 = *(const double4*)((const double*)p + idx), v1 = *(const double4*)((const double*)p + idx + 4);
    const double w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = to_e4m3(w[e] * qs);
  } else if constexpr (SF == F32) {
    const float4 v0 = *(const float4*)((const float*)p + idx), v1 = *(const float4*)((const float*)p + idx + 4);
    const float w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = to_e4m3((double)w[e] * qs);
  } else {
    const u16x8 v = *(const u16x8*)((const uint16_t*)p + idx);
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = to_e4m3((double)(SF == F16 ? f16_to_f32(v[e]) : bf16_to_f32(v[e])) * qs);
  }
}

template <int FA, int FB>
__device__ __forceinline__ void f8_mainloop(const void* Ap, const void* Bp, double qa, double qb, int nb, int64_t arow0,
                                            int64_t brow0, uint8_t (&As)[2][UBM][FLDK], uint8_t (&Bs)[2][UBM][FLDK],
                                            f4 (&acc)[4][4]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const int rg = tid & 15;  // rows 8 rg .. 8 rg + 7
  const int kq = tid >> 4;  // k = kq + 16 g, g = 0 .. 7
  uint8_t ra[8][8], rb[8][8];
  auto gload = [&](int kk) {
#pragma unroll
    for (int g = 0; g < FBK / 16; ++g) {
      const int64_t col = kk + kq + 16 * g;
      load8_f8<FA>(Ap, col * nb + arow0 + 8 * rg, ra[g], qa);
      load8_f8<FB>(Bp, col * nb + brow0 + 8 * rg, rb[g], qb);
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int g = 0; g < FBK / 16; ++g)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        As[buf][8 * rg + e][kq + 16 * g] = ra[g][e];
        Bs[buf][8 * rg + e][kq + 16 * g] = rb[g][e];
      }
  };
  gload(0);
  sstore(0);
  __syncthreads();
  int cur = 0;
  for (int kk = 0; kk < nb; kk += FBK) {
    const bool more = kk + FBK < nb;
    if (more) gload(kk + FBK);
#pragma unroll
    for (int k32 = 0; k32 < FBK; k32 += 32) {
      long av[4], bv[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) av[a] = *(const long*)&As[cur][wm * 64 + a * 16 + (lane & 15)][k32 + 8 * (lane >> 4)];
#pragma unroll
      for (int b = 0; b < 4; ++b) bv[b] = *(const long*)&Bs[cur][wn * 64 + b * 16 + (lane & 15)][k32 + 8 * (lane >> 4)];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
    if (more) sstore(cur ^ 1);
    __syncthreads();
    cur ^= 1;
  }
}

// scale exponent of operand tile (i, k) as an FP8 operand
__device__ __forceinline__ int operand_f8_scale(const TileView& tv, int i, int k, const double* pamax) {
  return tv.tfmt(i, k) == F8 ? tv.tscale(i, k) : fp8_scale_exp(pamax[i]);
}

__global__ __launch_bounds__(256) void k_update_f8(TileView tv, int k, const GemmTask* tasks, const double* pamax,
                                                   float* ws32, unsigned* amax32) {
  __shared__ __attribute__((aligned(16))) uint8_t As[2][UBM][FLDK];
  __shared__ __attribute__((aligned(16))) uint8_t Bs[2][UBM][FLDK];
  __shared__ float red[256];
  const int nb = tv.nb;
  const int sub = nb / UBM;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int task = lb / (sub * sub);
  const int blk = lb % (sub * sub);
  const int bm = blk % sub, bn = blk / sub;
  const GemmTask t = tasks[task];
  if (*tv.info) return;

  const void* Ap = tv.tile(t.i, k);
  const void* Bp = tv.tile(t.j, k);
  const int fa = tv.tfmt(t.i, k), fb = tv.tfmt(t.j, k);
  const int sa = operand_f8_scale(tv, t.i, k, pamax), sb = operand_f8_scale(tv, t.j, k, pamax);
  const double qa = ldexp(1.0, sa), qb = ldexp(1.0, sb);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const int64_t arow0 = (int64_t)bm * UBM, brow0 = (int64_t)bn * UBM;

  f4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f4{0, 0, 0, 0};
#define MPCR_PAIR(FA, FB) \
  case FA * 5 + FB: f8_mainloop<FA, FB>(Ap, Bp, qa, qb, nb, arow0, brow0, As, Bs, acc); break;
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

  const uint8_t* Cp = (const uint8_t*)tv.tile(t.i, t.j);
  const double mc = ldexp(1.0, -tv.tscale(t.i, t.j)), mp = ldexp(1.0, -(sa + sb));
  float* W = ws32 + (int64_t)task * nb * nb;
  float m = 0.0f;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t R = arow0 + wm * 64 + a * 16 + 4 * (lane >> 4) + r;
        const int64_t C = brow0 + wn * 64 + b * 16 + (lane & 15);
        const int64_t idx = C * nb + R;
        const float v = round_odd_f32((double)e4m3_to_f32(Cp[idx]) * mc - (double)acc[a][b][r] * mp);
        W[idx] = v;
        m = fmaxf(m, fabsf(v));
      }
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicMax(&amax32[task], __float_as_uint(red[0]));  // non-negative floats order as integers
}

// one workgroup per (FP8 task, 16-column slab): round the staged tile once to FP8
__global__ __launch_bounds__(256) void k_requant_f8(TileView tv, const GemmTask* tasks, const float* ws32,
                                                    const unsigned* amax32) {
  if (*tv.info) return;
  const int nb = tv.nb, slabs = nb / 16;
  const int task = blockIdx.x / slabs, c0 = (blockIdx.x % slabs) * 16;
  const GemmTask t = tasks[task];
  const int s = fp8_scale_exp((double)__uint_as_float(amax32[task]));
  uint8_t* Cp = (uint8_t*)tv.tile(t.i, t.j);
  const float* W = ws32 + (int64_t)task * nb * nb;
  for (int e = threadIdx.x; e < 16 * nb; e += 256) {
    const int64_t idx = (int64_t)(c0 + e / nb) * nb + e % nb;
    Cp[idx] = to_e4m3(ldexp((double)W[idx], s));
  }
  if (blockIdx.x % slabs == 0 && threadIdx.x == 0) tv.sc[tri_index(t.i, t.j)] = (int8_t)s;
}

__global__ void k_zero_u32(unsigned* p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

hipError_t launch_tile_update_fp8(const TileView& tv, int k, const GemmTask* tasks, int ntasks, const double* pamax,
                                  float* ws32, unsigned* amax32, hipStream_t s) {
  if (ntasks == 0) return hipSuccess;
  const int sub = tv.nb / UBM;
  k_zero_u32<<<(ntasks + 255) / 256, 256, 0, s>>>(amax32, ntasks);
  k_update_f8<<<ntasks * sub * sub, 256, 0, s>>>(tv, k, tasks, pamax, ws32, amax32);
  k_requant_f8<<<ntasks * (tv.nb / 16), 256, 0, s>>>(tv, tasks, ws32, amax32);
  return hipGetLastError();
}

// 16-bit output tiles
hipError_t launch_tile_update_16(const TileView& tv, int k, int cfmt, const GemmTask* tasks, int ntasks, hipStream_t s) {
  const int sub = tv.nb / UBM;
  if (cfmt == BF16) k_update_mmajor<BF16><<<ntasks * sub * sub, 256, 0, s>>>(tv, k, tasks);
  else if (cfmt == F16) k_update_mmajor<F16><<<ntasks * sub * sub, 256, 0, s>>>(tv, k, tasks);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// largest magnitude of each panel tile (i, k), i > k (widened values)
__global__ __launch_bounds__(256) void k_panel_amax(TileView tv, int k, double* pamax) {
  const int i = k + 1 + blockIdx.x;
  const int nb = tv.nb;
  const void* P = tv.tile(i, k);
  const int f = tv.tfmt(i, k);
  __shared__ double red[256];
  double m = 0.0;
  for (int64_t e = threadIdx.x; e < (int64_t)nb * nb; e += 256) m = fmax(m, fabs(load_wide(P, f, e)));
  red[threadIdx.x] = m * tv.tmul(i, k);
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) pamax[i] = red[0];
}

hipError_t launch_panel_amax(const TileView& tv, int k, double* pamax, hipStream_t s) {
  const int cnt = tv.nt - k - 1;
  if (cnt <= 0) return hipSuccess;
  k_panel_amax<<<cnt, 256, 0, s>>>(tv, k, pamax);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Shared pieces of the diagonal-tile POTRF and the panel TRSM.
// ---------------------------------------------------------------------------
constexpr int PW = 32;

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
//   (b) k_potrf_panel  the rows below solve X D_jj^T = A, one wave per 16
//                      rows (trsm_rows16_inv),
//   (c) k_potrf_syrk   the lower trailing part loses L_{:,j} L_{:,j}^T
//                      (64 x 64 output blocks, FP64 MFMA).
// ---------------------------------------------------------------------------
constexpr int SB = 128;

// acc[h] += A[R0 .. R0+15, K0:K1] * B[C0 + 16h .. C0 + 16h + 15, K0:K1]^T, h < 4,
// straight from column-major FP64 storage (leading dimension ld), 16 k per
// batch with the next batch's loads in flight.  K1 - K0 is a multiple of 16.
__device__ __forceinline__ void mfma_rows16x64(const double* A, const double* B, int64_t ld, int R0, int C0, int K0,
                                               int K1, int lane, d4 (&acc)[4]) {
  const int r = lane & 15, q = lane >> 4;
  auto ld20 = [&](int kk, double* a, double (*b)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t col = kk + 4 * u + q;
      a[u] = A[col * ld + R0 + r];
#pragma unroll
      for (int h = 0; h < 4; ++h) b[h][u] = B[col * ld + C0 + 16 * h + r];
    }
  };
  double a[4], b[4][4];
  ld20(K0, a, b);
  for (int kk = K0; kk < K1; kk += 16) {
    double na[4], nbv[4][4];
    const bool more = kk + 16 < K1;
    if (more) ld20(kk + 16, na, nbv);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int h = 0; h < 4; ++h) acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[h][u], acc[h], 0, 0, 0);
    if (more) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        a[u] = na[u];
#pragma unroll
        for (int h = 0; h < 4; ++h) b[h][u] = nbv[h][u];
      }
    }
  }
}

// rows c1 .. nb of block column j: X D_jj^T = A in place, one wave per 16 rows
__global__ __launch_bounds__(64) void k_potrf_panel(TileView tv, int k, int j, const double* dinv) {
  if (*tv.info) return;
  const int nb = tv.nb, c0 = j * SB, c1 = c0 + SB;
  double* A = (double*)tv.tile(k, k);
  __shared__ double Ts[16][PW + 1];
  trsm_rows16_inv(A, A, nb, dinv, c0, c1, c1 + blockIdx.x * 16, Ts, threadIdx.x, [&](int64_t i) { return A[i]; },
                  [&](int64_t i, double v) { A[i] = v; });
}

// A[R, C] -= L[R, c0:c1] L[C, c0:c1]^T for c1 <= C <= R < nb; one workgroup per
// lower 64 x 64 block (bi >= bj), eight waves: wave w takes rows 16 (w % 4) ..
// of the block over one half of the 128 columns, and the second half's partial
// products are added to the first's through LDS (half the chain of dependent
// loads and MFMAs per wave on this critical-path step)
__global__ __launch_bounds__(512) void k_potrf_syrk(TileView tv, int k, int j) {
  if (*tv.info) return;
  const int nb = tv.nb, c0 = j * SB, c1 = c0 + SB;
  double* A = (double*)tv.tile(k, k);
  int bi = 0, rem = blockIdx.x;
  while (rem > bi) { rem -= bi + 1; ++bi; }
  const int bj = rem;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rg = wave & 3, kh = wave >> 2, kw = SB / 2;
  const int R0 = c1 + bi * 64 + rg * 16, C0 = c1 + bj * 64;
  __shared__ double red[4][16][65];
  d4 acc[4];
#pragma unroll
  for (int h = 0; h < 4; ++h) acc[h] = d4{0, 0, 0, 0};
  mfma_rows16x64(A, A, nb, R0, C0, c0 + kh * kw, c0 + (kh + 1) * kw, lane, acc);
  if (kh == 1) {
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[rg][(lane >> 4) + 4 * r][16 * h + (lane & 15)] = acc[h][r];
  }
  __syncthreads();
  if (kh == 0) {
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int R = R0 + (lane >> 4) + 4 * r, C = C0 + 16 * h + (lane & 15);
        if (R >= C) A[(int64_t)C * nb + R] -= acc[h][r] + red[rg][(lane >> 4) + 4 * r][16 * h + (lane & 15)];
      }
  }
}

// A_jj -= L_jk L_jk^T for one diagonal tile with an FP64 panel tile (the SYRK
// on the factorisation's critical path): one workgroup per lower 64 x 64 block,
// eight waves: wave w takes rows 16 (w % 4) .. of the block over one half of
// the contraction (FP64 MFMA straight from the tiles); the second half's
// partial products are added to the first's through LDS.  Halving each wave's
// chain of dependent MFMAs halves the kernel's latency, which is what counts
// here: the 36 workgroups of a 512-tile occupy few CUs.
__global__ __launch_bounds__(512) void k_syrk_tile(TileView tv, int k, int j) {
  if (*tv.info) return;
  const int nb = tv.nb;
  int bi = 0, rem = blockIdx.x;
  while (rem > bi) { rem -= bi + 1; ++bi; }
  const int bj = rem;
  const double* L = (const double*)tv.tile(j, k);
  double* A = (double*)tv.tile(j, j);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rg = wave & 3, kh = wave >> 2, kw = nb / 2;
  const int R0 = bi * 64 + rg * 16, C0 = bj * 64;
  __shared__ double red[4][16][65];
  d4 acc[4];
#pragma unroll
  for (int h = 0; h < 4; ++h) acc[h] = d4{0, 0, 0, 0};
  mfma_rows16x64(L, L, nb, R0, C0, kh * kw, (kh + 1) * kw, lane, acc);
  if (kh == 1) {
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[rg][(lane >> 4) + 4 * r][16 * h + (lane & 15)] = acc[h][r];
  }
  __syncthreads();
  if (kh == 0) {
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int R = R0 + (lane >> 4) + 4 * r, C = C0 + 16 * h + (lane & 15);
        if (R >= C) A[(int64_t)C * nb + R] -= acc[h][r] + red[rg][(lane >> 4) + 4 * r][16 * h + (lane & 15)];
      }
  }
}

hipError_t launch_syrk_tile(const TileView& tv, int k, int j, hipStream_t s) {
  const int nbk = tv.nb / 64;
  k_syrk_tile<<<nbk * (nbk + 1) / 2, 512, 0, s>>>(tv, k, j);
  return hipGetLastError();
}

hipError_t launch_potrf_tile(const TileView& tv, int k, double* dinv, hipStream_t s) {
  const int nsb = tv.nb / SB;
  for (int j = 0; j < nsb; ++j) {
    if (const hipError_t e = launch_potrf_block(tv, k, j, dinv, s); e != hipSuccess) return e;
    const int rest = (tv.nb - (j + 1) * SB) / 64;  // 64-row blocks below block j
    if (rest > 0) {
      k_potrf_panel<<<rest * 4, 64, 0, s>>>(tv, k, j, dinv);
      k_potrf_syrk<<<rest * (rest + 1) / 2, 512, 0, s>>>(tv, k, j);
    }
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Panel TRSM: for i > k, X = A_ik L_kk^{-T} in FP64, rounded once to p(i,k).
// One wave per 16 rows of a panel tile (trsm_rows16_inv with the inverted
// diagonal blocks of L_kk from its POTRF); the FP64 X goes to the workspace ws
// ((nt-k-1) tiles of nb x nb) and the tile receives one rounding of it.
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

hipError_t launch_trsm_panel(const TileView& tv, int k, double* ws, const double* dinv, bool fp8_panel,
                             hipStream_t s) {
  int ntile = tv.nt - k - 1;
  if (ntile <= 0) return hipSuccess;
  if (ntile <= TRSM_SPLIT_MAX)
    k_trsm4<<<ntile * (tv.nb / 16), 256, 0, s>>>(tv, k, ws, dinv);
  else
    k_trsm<<<ntile * (tv.nb / 16), 64, 0, s>>>(tv, k, ws, dinv);
  if (fp8_panel) k_quant_panel_f8<<<ntile, 256, 0, s>>>(tv, k, ws);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// log|Sigma| = 2 sum_i log L_ii over the first n diagonal entries; fixed
// summation order (strided per thread, then a fixed tree).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_logdet(TileView tv, double* out) {
  __shared__ double red[256];
  const int nb = tv.nb;
  double s = 0.0;
  if (*tv.info == 0) {
    for (int g = threadIdx.x; g < tv.n; g += 256) {
      int t = g / nb, l = g % nb;
      s += log(((const double*)tv.tile(t, t))[(int64_t)l * nb + l]);
    }
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = 2.0 * red[0];
}

hipError_t launch_logdet(const TileView& tv, double* out, hipStream_t s) {
  k_logdet<<<1, 256, 0, s>>>(tv, out);
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

hipError_t launch_trtri_diag(const TileView& tv, double* Linv, const double* dinv, hipStream_t s) {
  k_trtri<<<tv.nt * (tv.nb / 16), 64, 0, s>>>(tv, Linv, dinv);
  return hipGetLastError();
}

}  // namespace mpcr
