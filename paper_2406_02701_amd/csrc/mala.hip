// Kernels of the Metropolis-adjusted Langevin sampler (the paper's
// "Metropolis-Hastings Algorithm in High Dimensions" section) that the tile
// solves and covariance products do not already cover: the product of the
// lower tile factor with a vector (the proposal noise L eps) and the
// element-wise combinations of the proposal.
#include "mpcr_internal.h"

namespace mpcr {

// y = L x over the lower tiles (L widened to FP64; x has tv.n entries).  One
// workgroup per 16 rows: 64 groups of 16 threads (a column's rows are read 128
// bytes at a time) take every 64th column, eight of a tile's in flight; the groups'
// sums are added through LDS in a fixed order.  Bound by the latency of those
// batches; many small workgroups instead of one per 64 rows with four groups:
// n = 1024 (64 workgroups for 16) 52 -> 7 us.
constexpr int TRMV_GROUPS = 64;

template <int F>
__device__ __forceinline__ double trmv_tile(const void* t, int nb, int r, int g, int cend, const double* x, double mul) {
  double a = 0.0;
  int c = g;
  auto elem = [&](int cc) { return load_wide(t, F, (int64_t)cc * nb + r); };
  for (; c + 7 * TRMV_GROUPS < cend; c += 8 * TRMV_GROUPS) {
    double v[8], w[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      v[u] = elem(c + u * TRMV_GROUPS);
      w[u] = x[c + u * TRMV_GROUPS];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) a += v[u] * w[u];
  }
  double v[8], w[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int cc = c + u * TRMV_GROUPS;
    v[u] = cc < cend ? elem(cc) : 0.0;
    w[u] = cc < cend ? x[cc] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < 8; ++u) a += v[u] * w[u];
  return a * mul;
}

__global__ __launch_bounds__(16 * TRMV_GROUPS) void k_trmv_lower(TileView tv, const double* x, double* y) {
  __shared__ double part[TRMV_GROUPS][17];
  const int i = blockIdx.x, nb = tv.nb, lr = threadIdx.x & 15, g = threadIdx.x >> 4;
  const int r = blockIdx.y * 16 + lr;
  double acc = 0.0;
  for (int j = 0; j <= i; ++j) {
    const void* t = tv.tile(i, j);
    const double mul = tv.tmul(i, j);
    const double* xj = x + (int64_t)j * nb;
    int cend = j == i ? r + 1 : nb;
    if (j * nb + cend > tv.n) cend = tv.n - j * nb;
    switch (tv.tfmt(i, j)) {
      case F64: acc += trmv_tile<F64>(t, nb, r, g, cend, xj, mul); break;
      case F32: acc += trmv_tile<F32>(t, nb, r, g, cend, xj, mul); break;
      case F16: acc += trmv_tile<F16>(t, nb, r, g, cend, xj, mul); break;
      case BF16: acc += trmv_tile<BF16>(t, nb, r, g, cend, xj, mul); break;
      default: acc += trmv_tile<F8>(t, nb, r, g, cend, xj, mul);
    }
  }
  part[g][lr] = acc;
  __syncthreads();
  if (g < 8) {
#pragma unroll
    for (int u = 1; u < 8; ++u) acc += part[g + 8 * u][lr];
    part[g][lr] = acc;
  }
  __syncthreads();
  if (g == 0) {
#pragma unroll
    for (int u = 1; u < 8; ++u) acc += part[u][lr];
    y[(int64_t)i * nb + r] = acc;
  }
}

hipError_t launch_trmv_lower(const TileView& tv, const double* x, double* y, hipStream_t s) {
  k_trmv_lower<<<dim3((unsigned)tv.nt, (unsigned)(tv.nb / 16)), 16 * TRMV_GROUPS, 0, s>>>(tv, x, y);
  return hipGetLastError();
}

// out = a + alpha * b (element-wise, n entries)
__global__ void k_axpby(int n, const double* a, double alpha, const double* b, double* out) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) out[i] = a[i] + alpha * b[i];
}

hipError_t launch_axpby(int n, const double* a, double alpha, const double* b, double* out, hipStream_t s) {
  int g = (n + 255) / 256;
  k_axpby<<<g < 1024 ? (g > 0 ? g : 1) : 1024, 256, 0, s>>>(n, a, alpha, b, out);
  return hipGetLastError();
}

}  // namespace mpcr
