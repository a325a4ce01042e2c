// Objective of the pattern search (Appendix A, Algorithm 4): per head and
// token class, the sum of squared differences between two attention
// outputs, bound by reading both once. 16 lanes read one row (256 contiguous
// bytes), a workgroup takes a run of rows of one head; the sums run in fp64
// in a fixed order (a thread's rows ascending, lane shuffles, waves in order,
// then the runs in order), so the result is bitwise reproducible. The search
// gives scratch for SQ_CHUNKS runs per head; the public call has none and
// takes one run per head. 24K tokens x 28 heads (352 MB): one workgroup per
// head with a whole row per thread took 715 us.
#include "device.hpp"
#include "internal.hpp"

namespace mmi {

constexpr int SQ_THREADS = 512;
constexpr int SQ_ROWS = SQ_THREADS / 16;     // rows read at once by a workgroup
constexpr int SQ_UNROLL = 4;

__global__ __launch_bounds__(SQ_THREADS) void k_sqerr(const uint16_t* a, const uint16_t* b, int64_t ss, int64_t sh,
                                                      const uint8_t* cls, int n_class, int S, int rows, double* out) {
  const int h = blockIdx.x, chunk = blockIdx.y;
  const int64_t x0 = (int64_t)chunk * rows;
  const int x1 = (int)min((int64_t)S, x0 + rows);
  const int sub = threadIdx.x >> 4, d = (threadIdx.x & 15) * 8;
  double acc[MMI_MAX_MODALITIES];
#pragma unroll
  for (int c = 0; c < MMI_MAX_MODALITIES; ++c) acc[c] = 0.0;
  for (int64_t xb = x0 + sub; xb < x1; xb += SQ_ROWS * SQ_UNROLL) {
    bf16x8 va[SQ_UNROLL], vb[SQ_UNROLL];
    int c[SQ_UNROLL];
#pragma unroll
    for (int u = 0; u < SQ_UNROLL; ++u) {
      const int64_t x = xb + u * SQ_ROWS;
      c[u] = x < x1 ? cls[x] : MMI_MAX_MODALITIES;
      const int64_t at = min(x, (int64_t)x1 - 1) * ss + (int64_t)h * sh + d;
      va[u] = load16(a + at);
      vb[u] = load16(b + at);
    }
#pragma unroll
    for (int u = 0; u < SQ_UNROLL; ++u) {
      double part = 0.0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float diff = (float)va[u][e] - (float)vb[u][e];
        part += (double)diff * (double)diff;
      }
      // a row past the run or of no class adds to none (its values may be infinite)
#pragma unroll
      for (int k = 0; k < MMI_MAX_MODALITIES; ++k) acc[k] += k == c[u] ? part : 0.0;
    }
  }
  __shared__ double part[SQ_THREADS / 64][MMI_MAX_MODALITIES];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < MMI_MAX_MODALITIES; ++k) {
    double v = acc[k];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if (lane == 0) part[wave][k] = v;
  }
  __syncthreads();
  if ((int)threadIdx.x < n_class) {
    double s = 0.0;
    for (int w = 0; w < SQ_THREADS / 64; ++w) s += part[w][threadIdx.x];
    out[((int64_t)chunk * gridDim.x + h) * n_class + threadIdx.x] = s;
  }
}

// out[i] = sum of the runs' sums part[c][i], c ascending
__global__ void k_sqerr_sum(const double* part, int n, int chunks, double* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = 0.0;
  for (int c = 0; c < chunks; ++c) s += part[(int64_t)c * n + i];
  out[i] = s;
}

hipError_t launch_sqerr(const void* a, const void* b, int64_t ss, int64_t sh, const uint8_t* cls, int n_class,
                        int S, int H, double* out, double* part, hipStream_t st) {
  if (H <= 0) return hipSuccess;
  const int chunks = part ? SQ_CHUNKS : 1, rows = (S + chunks - 1) / chunks;
  hipLaunchKernelGGL(k_sqerr, dim3(H, chunks), dim3(SQ_THREADS), 0, st, reinterpret_cast<const uint16_t*>(a),
                     reinterpret_cast<const uint16_t*>(b), ss, sh, cls, n_class, S, rows, part ? part : out);
  if (part)
    hipLaunchKernelGGL(k_sqerr_sum, dim3((H * n_class + 63) / 64), dim3(64), 0, st, part, H * n_class, chunks, out);
  return hipGetLastError();
}

}  // namespace mmi
