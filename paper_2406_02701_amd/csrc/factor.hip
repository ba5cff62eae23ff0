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

}  // namespace mpcr
