// Explicit row permutation: the permute(Q), permute(K), permute(V) steps of
// Algorithms 1-3 done as a separate HBM pass (the attention kernel performs
// the same gathers inline; this pass exists for the identity tests and to
// measure what an explicit permutation costs). 16-byte vector copies,
// neighbouring lanes on neighbouring vectors of a row; perm = -1 writes a zero
// row. Bound by HBM: rows of a power-of-two number of vectors (every head
// dimension of 16-byte multiples in use) take a variant whose index arithmetic
// is shifts, with PU independent rows in flight per thread and stores that do
// not displace what is still to be read: 64 copies of 131072 256-byte rows
// (4.3 GB) 993 -> 891 us, 4.8 TB/s.
#include "device.hpp"
#include "internal.hpp"

namespace mmi {

__global__ __launch_bounds__(256) void k_permute(const uint8_t* src, int64_t ss, uint8_t* dst, int64_t ds,
                                                 const int32_t* perm, int64_t n, int64_t row_bytes,
                                                 int inverse) {
  const int64_t vec_per_row = row_bytes / 16;
  const int64_t total = n * vec_per_row;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t x = idx / vec_per_row, c = idx % vec_per_row;
    const int p = perm[x];
    if (!inverse) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (p >= 0) v = *reinterpret_cast<const uint4*>(src + p * ss + c * 16);
      *reinterpret_cast<uint4*>(dst + x * ds + c * 16) = v;
    } else if (p >= 0) {
      *reinterpret_cast<uint4*>(dst + p * ds + c * 16) = *reinterpret_cast<const uint4*>(src + x * ss + c * 16);
    }
  }
}

constexpr int PU = 4;              // rows in flight per thread

// The same for rows of 2^shift vectors, fewer than 2^31 of them: thread t of
// a workgroup copies vector t mod 2^shift of rows t >> shift, then on by the
// rows of a workgroup.
template <bool INVERSE>
__global__ __launch_bounds__(256) void k_permute_pow2(const uint8_t* src, int64_t ss, uint8_t* dst, int64_t ds,
                                                      const int32_t* perm, int n, int shift) {
  typedef __attribute__((__vector_size__(16))) unsigned int v4;
  const int rows = 256 >> shift;   // rows of one step of the workgroup (shift <= 8)
  const int c = ((int)threadIdx.x & ((1 << shift) - 1)) * 16, r = (int)threadIdx.x >> shift;
  const int64_t x0 = (int64_t)blockIdx.x * rows * PU + r;
  int p[PU];
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int64_t x = x0 + u * rows;
    p[u] = x < n ? perm[x] : -1;
  }
  v4 v[PU];
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int64_t x = x0 + u * rows;
    const v4 zero = {};
    v[u] = p[u] >= 0 ? *reinterpret_cast<const v4*>(src + (INVERSE ? x : (int64_t)p[u]) * ss + c) : zero;
  }
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int64_t x = x0 + u * rows;
    if (INVERSE ? p[u] >= 0 : x < n)
      __builtin_nontemporal_store(v[u], reinterpret_cast<v4*>(dst + (INVERSE ? (int64_t)p[u] : x) * ds + c));
  }
}

hipError_t launch_permute(const void* src, int64_t ss, void* dst, int64_t ds, const int32_t* perm, int64_t n,
                          int64_t row_bytes, int inverse, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const uint8_t* s = reinterpret_cast<const uint8_t*>(src);
  uint8_t* d = reinterpret_cast<uint8_t*>(dst);
  const int64_t vecs = row_bytes / 16;
  // n is an int there, and a launch holds fewer than 2^32 threads (a quarter of the vectors)
  if (vecs <= 256 && (vecs & (vecs - 1)) == 0 && n <= 0x7fffffff && n <= ((int64_t)1 << 33) / vecs) {
    int shift = 0;
    while ((1 << shift) < vecs) ++shift;
    const int64_t per = (int64_t)(256 >> shift) * PU;
    const dim3 grid((unsigned)((n + per - 1) / per));
    if (inverse) hipLaunchKernelGGL(k_permute_pow2<true>, grid, dim3(256), 0, st, s, ss, d, ds, perm, (int)n, shift);
    else hipLaunchKernelGGL(k_permute_pow2<false>, grid, dim3(256), 0, st, s, ss, d, ds, perm, (int)n, shift);
    return hipGetLastError();
  }
  const int64_t total = n * vecs;
  const int64_t blocks = (total + 255) / 256;
  const unsigned grid = (unsigned)(blocks < 65536 * 4 ? blocks : 65536 * 4);
  hipLaunchKernelGGL(k_permute, dim3(grid), dim3(256), 0, st, s, ss, d, ds, perm, n, row_bytes, inverse);
  return hipGetLastError();
}

}  // namespace mmi
