// Discrete choices taken from the estimate.
//
// Grid stride/phase search (Algorithm 1, "Online search grid stride and
// phase"): for each candidate stride s the column scores v are folded with
// period s, c_s[p] = mean_{t: t s + p < L_c} v[t s + p]; score_s = max_p c_s[p]
// with the smallest maximising phase. k_grid_fold computes one stride per
// workgroup (each thread sums its phases in ascending t: fixed order);
// k_grid_pick scans the strides in ascending order and keeps a later stride
// only if its score exceeds best * 1.02 (fp32 product), then publishes
// {sigma, phase} (sigma 0 = no stride with two visible periods: dense).
//
// Vertical-Slash top-k (Appendix C.3): the n largest scores of [0, L),
// ties to the smaller index, as an ascending index list. Radix select on the
// fp32 bit patterns (scores are non-negative, so bits order like values):
// three digit passes with LDS histograms find the n-th largest value T; then
// one ordered pass (wave prefix sums, consecutive elements per thread) keeps
// every score > T and the first (n - #greater) indices equal to T. All counts are integers, so the result does not depend on thread
// timing.
#include <algorithm>

#include "device.hpp"
#include "internal.hpp"

namespace mmi {

__global__ __launch_bounds__(256) void k_grid_fold(const GridJob* jobs) {
  const GridJob jb = jobs[blockIdx.x];
  const int y = blockIdx.y;
  const int s = jb.lo + y;
  if (jb.hi < jb.lo || s > jb.hi) return;
  __shared__ float bv[256];
  __shared__ int bp[256];
  float best = -1.0f;
  int bestp = 0x7fffffff;
  constexpr int U = 16;   // loads in flight per thread; the sum keeps ascending t order
  for (int p = threadIdx.x; p < s; p += 256) {
    float acc = 0.0f;
    int n = 0;
    int x = p;
    for (; x + (U - 1) * s < jb.L_c; x += U * s) {
      float t[U];
#pragma unroll
      for (int u = 0; u < U; ++u) t[u] = jb.v[x + u * s];
#pragma unroll
      for (int u = 0; u < U; ++u) acc += t[u];
      n += U;
    }
    for (; x < jb.L_c; x += s) {
      acc += jb.v[x];
      ++n;
    }
    const float c = acc / (float)n;
    jb.fold[(int64_t)y * FOLD_W + p] = c;
    if (c > best) { best = c; bestp = p; }     // p ascending per thread: keeps the smallest
  }
  bv[threadIdx.x] = best;
  bp[threadIdx.x] = bestp;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      const float ov = bv[threadIdx.x + w];
      const int op = bp[threadIdx.x + w];
      if (ov > bv[threadIdx.x] || (ov == bv[threadIdx.x] && op < bp[threadIdx.x])) {
        bv[threadIdx.x] = ov;
        bp[threadIdx.x] = op;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    jb.score[y] = bv[0];
    jb.pick[y] = bp[0];
  }
}

__global__ void k_grid_pick(const GridJob* jobs, int njobs) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= njobs) return;
  const GridJob jb = jobs[j];
  float b = 0.0f;
  int sig = 0, ph = 0;
  const float one_eps = 1.02f;
  for (int s = jb.lo; s <= jb.hi; ++s) {
    const float sc = jb.score[s - jb.lo];
    const float thr = b * one_eps;
    if (sc > thr) {
      b = sc;
      sig = s;
      ph = jb.pick[s - jb.lo];
    }
  }
  jb.params[0] = sig;
  jb.params[1] = ph;
  jb.params[2] = jb.L_c;
  jb.params[3] = jb.nrows;
}

// Top-n of a score array: a radix select of the n-th largest fp32 bit
// pattern T (scores are >= 0, so the bit patterns order like the values),
// 11, 11 and 10 bits per pass from the top, then an order-preserving
// selection: every element above T and the first `remaining` copies of T by
// index, written in ascending index order. Counts are integers, so the
// result does not depend on the order of the additions.
//
// Both variants are bound by latency, not by bytes (28 heads x 32K scores are
// 3.7 MB): what counts is how few dependent steps lie between the scores and
// the list. The digit of a pass is found by a scan of the bins over the
// whole workgroup; one thread walking 256 bins by dependent loads took 50-75
// us of every pass (28 heads, 3K to 128K scores: 207-313 us per plan in the
// histogram passes alone; a whole layer of 3,001 tokens went 838 -> 536 us
// and one of 32K tokens 4263 -> 4001 us with these two variants).
//   k_topk_one: one workgroup per job, scores in registers, one launch.
//     Scores up to TK_ONE_MAX.
//   k_topk_init / hist / count / write: longer arrays, a job spread over
//     TK_CHUNKS workgroups per pass; the last workgroup to finish (a counter)
//     picks the digit for the next pass. Per-job scratch (int32, TK_SCR):
//     prefix, mask, remaining, then a histogram and a finish counter per
//     pass, then the chunks' counts of elements above T and equal to T.
constexpr int TK_WG = 256;
constexpr int TK_WAVES = TK_WG / 64;
constexpr int TK_CHUNKS = 16;
constexpr int TK_PER = 8;          // consecutive elements per thread in the selection pass
constexpr int TK_PASSES = 3;
constexpr int TK_BINS = 2048;      // bins of one pass (the last uses half of them)
constexpr int TK_HIST = 4;
constexpr int TK_DONE = TK_HIST + TK_PASSES * TK_BINS;
constexpr int TK_CNT = TK_DONE + 4;
constexpr int TK_SCR = TK_CNT + 2 * TK_CHUNKS;
constexpr int TK1_WG = 1024;       // threads of the one-workgroup variant
constexpr int TK1_PER_MAX = 32;    // scores per thread held in registers
constexpr int TK_ONE_MAX = TK1_WG * TK1_PER_MAX;

__device__ __forceinline__ int tk_shift(int pass) { return pass == 0 ? 21 : pass == 1 ? 10 : 0; }
__device__ __forceinline__ uint32_t tk_digit_mask(int pass) { return pass == 2 ? 1023u : 2047u; }

__device__ __forceinline__ bool topk_trivial(const TopkJob& jb) { return jb.n <= 0 || jb.n >= jb.L; }

__device__ __forceinline__ void chunk_range(const TopkJob& jb, int c, int& lo, int& hi) {
  const int ch = (jb.L + TK_CHUNKS - 1) / TK_CHUNKS;
  lo = min(jb.L, c * ch);
  hi = min(jb.L, lo + ch);
}

// The digit that holds the `remaining`-th element from the top of a
// TK_BINS-bin histogram, and the elements above it (to out[0], out[1]): the
// NT threads of the workgroup take TK_BINS / NT consecutive bins each from
// the top, scan their sums, and the one whose bins reach `remaining` walks
// its own. load(bin) reads a bin; wsum: NT / 64 ints of LDS. Ends with a
// barrier.
template <int NT, typename F>
__device__ __forceinline__ void pick_digit(F load, int remaining, int* wsum, int* out) {
  constexpr int PER = TK_BINS / NT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int h[PER];
  int sum = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    h[e] = load(TK_BINS - 1 - (tid * PER + e));
    sum += h[e];
  }
  int s = sum;
  for (int off = 1; off < 64; off <<= 1) {
    const int t = __shfl_up(s, off, 64);
    if (lane >= off) s += t;
  }
  if (lane == 63) wsum[wave] = s;
  __syncthreads();
  int above = s - sum;
  for (int w = 0; w < NT / 64; ++w) above += w < wave ? wsum[w] : 0;
  if (above < remaining && above + sum >= remaining) {
    int found = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      if (!found && above + h[e] >= remaining) {
        out[0] = TK_BINS - 1 - (tid * PER + e);
        out[1] = above;
        found = 1;
      }
      if (!found) above += h[e];
    }
  }
  __syncthreads();
}

// One workgroup per job: thread t holds scores [t PER, t PER + PER).
template <int PER>
__global__ __launch_bounds__(TK1_WG) void k_topk_one(const TopkJob* jobs) {
  const TopkJob jb = jobs[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (jb.n <= 0) return;
  if (jb.n >= jb.L) {
    for (int i = tid; i < jb.L; i += TK1_WG) jb.out[i] = i;
    return;
  }
  constexpr int NW = TK1_WG / 64;
  __shared__ int hist[4][TK_BINS];   // four copies: neighbouring lanes mostly hold the same digit
  __shared__ int wg[NW], we[NW], dig[2];
  const uint32_t* bits = reinterpret_cast<const uint32_t*>(jb.x);
  const int i0 = tid * PER;
  uint32_t x[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) x[e] = i0 + e < jb.L ? bits[i0 + e] : 0u;
  uint32_t prefix = 0, mask = 0;
  int remaining = jb.n;
  for (int pass = 0; pass < TK_PASSES; ++pass) {
    const int shift = tk_shift(pass);
    const uint32_t dm = tk_digit_mask(pass);
    for (int b = tid; b < 4 * TK_BINS; b += TK1_WG) (&hist[0][0])[b] = 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (i0 + e < jb.L && (x[e] & mask) == prefix) atomicAdd(&hist[lane & 3][(x[e] >> shift) & dm], 1);
    __syncthreads();
    pick_digit<TK1_WG>([&](int b) { return hist[0][b] + hist[1][b] + hist[2][b] + hist[3][b]; }, remaining, wg, dig);
    prefix |= (uint32_t)dig[0] << shift;
    mask |= dm << shift;
    remaining -= dig[1];
    __syncthreads();               // dig and the bins are rewritten by the next pass
  }
  const uint32_t T = prefix;
  int cg = 0, ce = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    cg += (i0 + e < jb.L && x[e] > T) ? 1 : 0;
    ce += (i0 + e < jb.L && x[e] == T) ? 1 : 0;
  }
  int sg = cg, se = ce;
  for (int off = 1; off < 64; off <<= 1) {
    const int a = __shfl_up(sg, off, 64), b2 = __shfl_up(se, off, 64);
    if (lane >= off) { sg += a; se += b2; }
  }
  if (lane == 63) { wg[wave] = sg; we[wave] = se; }
  __syncthreads();
  int g_before = sg - cg, e_before = se - ce;
  for (int w = 0; w < NW; ++w)
    if (w < wave) { g_before += wg[w]; e_before += we[w]; }
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    if (i0 + e >= jb.L) continue;
    const bool gt = x[e] > T, eq = x[e] == T;
    if (gt || (eq && e_before < remaining)) jb.out[g_before + min(e_before, remaining)] = i0 + e;
    g_before += gt ? 1 : 0;
    e_before += eq ? 1 : 0;
  }
}

__global__ __launch_bounds__(256) void k_topk_init(const TopkJob* jobs, int njobs, int32_t* scr) {
  const int j = blockIdx.x;
  if (j >= njobs) return;
  int32_t* sj = scr + (int64_t)j * TK_SCR;
  for (int x = threadIdx.x; x < TK_SCR; x += blockDim.x) sj[x] = x == 2 ? jobs[j].n : 0;
}

__global__ __launch_bounds__(TK_WG) void k_topk_hist(const TopkJob* jobs, int32_t* scr, int pass) {
  const TopkJob jb = jobs[blockIdx.x];
  if (topk_trivial(jb)) return;
  int32_t* sj = scr + (int64_t)blockIdx.x * TK_SCR;
  __shared__ int hist[TK_WAVES][TK_BINS];
  __shared__ int sh_last, wsum[TK_WAVES], dig[2];
  const int tid = threadIdx.x, wave = tid >> 6;
  const int shift = tk_shift(pass);
  const uint32_t dm = tk_digit_mask(pass);
  const uint32_t prefix = (uint32_t)sj[0], mask = (uint32_t)sj[1];
  for (int b = tid; b < TK_WAVES * TK_BINS; b += TK_WG) (&hist[0][0])[b] = 0;
  __syncthreads();
  int lo, hi;
  chunk_range(jb, blockIdx.y, lo, hi);
  const uint32_t* bits = reinterpret_cast<const uint32_t*>(jb.x);
  constexpr int HU = 8;            // loads in flight per thread
  for (int i0 = lo + tid; i0 < hi; i0 += TK_WG * HU) {
    uint32_t xs[HU];
#pragma unroll
    for (int u = 0; u < HU; ++u) xs[u] = i0 + u * TK_WG < hi ? bits[i0 + u * TK_WG] : 0u;
#pragma unroll
    for (int u = 0; u < HU; ++u)
      if (i0 + u * TK_WG < hi && (xs[u] & mask) == prefix) atomicAdd(&hist[wave][(xs[u] >> shift) & dm], 1);
  }
  __syncthreads();
  int32_t* gh = sj + TK_HIST + pass * TK_BINS;
  for (int b = tid; b < TK_BINS; b += TK_WG) {
    int c = 0;
    for (int w = 0; w < TK_WAVES; ++w) c += hist[w][b];
    if (c) atomicAdd(&gh[b], c);
  }
  __threadfence();
  __syncthreads();
  if (tid == 0) sh_last = atomicAdd(&sj[TK_DONE + pass], 1) == TK_CHUNKS - 1;
  __syncthreads();
  if (!sh_last) return;
  __threadfence();
  // the digit of the n-th largest among the candidates
  const int remaining = sj[2];
  pick_digit<TK_WG>([&](int b) { return __atomic_load_n(&gh[b], __ATOMIC_RELAXED); }, remaining, wsum, dig);
  if (tid == 0) {
    sj[0] = (int32_t)(prefix | ((uint32_t)dig[0] << shift));
    sj[1] = (int32_t)(mask | (dm << shift));
    sj[2] = remaining - dig[1];
  }
}

// Elements above T and equal to T in each chunk.
__global__ __launch_bounds__(TK_WG) void k_topk_count(const TopkJob* jobs, int32_t* scr) {
  const TopkJob jb = jobs[blockIdx.x];
  if (topk_trivial(jb)) return;
  int32_t* sj = scr + (int64_t)blockIdx.x * TK_SCR;
  __shared__ int wg[TK_WAVES], we[TK_WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t T = (uint32_t)sj[0];
  int lo, hi;
  chunk_range(jb, blockIdx.y, lo, hi);
  const uint32_t* bits = reinterpret_cast<const uint32_t*>(jb.x);
  int g = 0, e = 0;
  for (int i = lo + tid; i < hi; i += TK_WG) {
    const uint32_t x = bits[i];
    g += x > T ? 1 : 0;
    e += x == T ? 1 : 0;
  }
  for (int off = 32; off > 0; off >>= 1) { g += __shfl_xor(g, off, 64); e += __shfl_xor(e, off, 64); }
  if (lane == 0) { wg[wave] = g; we[wave] = e; }
  __syncthreads();
  if (tid == 0) {
    int tg = 0, te = 0;
    for (int w = 0; w < TK_WAVES; ++w) { tg += wg[w]; te += we[w]; }
    sj[TK_CNT + blockIdx.y] = tg;
    sj[TK_CNT + TK_CHUNKS + blockIdx.y] = te;
  }
}

// Output slot of a selected element i = (elements above T before i) +
// min(copies of T before i, remaining): ascending indices.
__global__ __launch_bounds__(TK_WG) void k_topk_write(const TopkJob* jobs, const int32_t* scr) {
  const TopkJob jb = jobs[blockIdx.x];
  int lo, hi;
  chunk_range(jb, blockIdx.y, lo, hi);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (jb.n <= 0) return;
  if (jb.n >= jb.L) {
    for (int i = lo + tid; i < hi; i += TK_WG) jb.out[i] = i;
    return;
  }
  const int32_t* sj = scr + (int64_t)blockIdx.x * TK_SCR;
  __shared__ int wgt[TK_WAVES], weq[TK_WAVES];
  const uint32_t T = (uint32_t)sj[0];
  const int remaining = sj[2];
  int gt_base = 0, eq_base = 0;    // counts of the chunks before this one
  for (int c = 0; c < (int)blockIdx.y; ++c) {
    gt_base += sj[TK_CNT + c];
    eq_base += sj[TK_CNT + TK_CHUNKS + c];
  }
  const uint32_t* bits = reinterpret_cast<const uint32_t*>(jb.x);
  for (int start = lo; start < hi; start += TK_WG * TK_PER) {
    const int i0 = start + tid * TK_PER;
    uint32_t xs[TK_PER];
    int cg = 0, ce = 0;
#pragma unroll
    for (int e = 0; e < TK_PER; ++e) {
      xs[e] = i0 + e < hi ? bits[i0 + e] : 0u;
      cg += (i0 + e < hi && xs[e] > T) ? 1 : 0;
      ce += (i0 + e < hi && xs[e] == T) ? 1 : 0;
    }
    int sg = cg, se = ce;          // inclusive scan over the wave's lanes
    for (int off = 1; off < 64; off <<= 1) {
      const int a = __shfl_up(sg, off, 64), b2 = __shfl_up(se, off, 64);
      if (lane >= off) { sg += a; se += b2; }
    }
    if (lane == 63) { wgt[wave] = sg; weq[wave] = se; }
    __syncthreads();
    int pg = 0, pe = 0, tg = 0, te = 0;
    for (int w = 0; w < TK_WAVES; ++w) {
      if (w < wave) { pg += wgt[w]; pe += weq[w]; }
      tg += wgt[w];
      te += weq[w];
    }
    __syncthreads();               // wgt/weq are rewritten by the next stretch
    int g_before = gt_base + pg + sg - cg, e_before = eq_base + pe + se - ce;
#pragma unroll
    for (int e = 0; e < TK_PER; ++e) {
      if (i0 + e < hi) {
        const bool gt = xs[e] > T, eq = xs[e] == T;
        if (gt || (eq && e_before < remaining)) {
          const int pos = g_before + min(e_before, remaining);
          if (pos < jb.n) jb.out[pos] = i0 + e;
        }
        g_before += gt ? 1 : 0;
        e_before += eq ? 1 : 0;
      }
    }
    gt_base += tg;
    eq_base += te;
  }
}

hipError_t launch_grid_search(const GridJob* jobs, int njobs, int max_cands, hipStream_t st) {
  if (njobs <= 0) return hipSuccess;
  if (max_cands > 0) hipLaunchKernelGGL(k_grid_fold, dim3(njobs, max_cands), dim3(256), 0, st, jobs);
  hipLaunchKernelGGL(k_grid_pick, dim3((njobs + 63) / 64), dim3(64), 0, st, jobs, njobs);
  return hipGetLastError();
}

size_t topk_scratch_ints(int njobs, int max_L) { return max_L > TK_ONE_MAX ? (size_t)std::max(njobs, 1) * TK_SCR : 0; }

hipError_t launch_topk(const TopkJob* jobs, int njobs, int max_L, int32_t* scr, hipStream_t st) {
  if (njobs <= 0) return hipSuccess;
  // one launch while a workgroup's registers hold the longest array of the plan
  if (max_L <= TK1_WG * 8) {
    hipLaunchKernelGGL(k_topk_one<8>, dim3(njobs), dim3(TK1_WG), 0, st, jobs);
    return hipGetLastError();
  }
  if (max_L <= TK_ONE_MAX) {
    hipLaunchKernelGGL(k_topk_one<TK1_PER_MAX>, dim3(njobs), dim3(TK1_WG), 0, st, jobs);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_topk_init, dim3(njobs), dim3(256), 0, st, jobs, njobs, scr);
  for (int pass = 0; pass < TK_PASSES; ++pass)
    hipLaunchKernelGGL(k_topk_hist, dim3(njobs, TK_CHUNKS), dim3(TK_WG), 0, st, jobs, scr, pass);
  hipLaunchKernelGGL(k_topk_count, dim3(njobs, TK_CHUNKS), dim3(TK_WG), 0, st, jobs, scr);
  hipLaunchKernelGGL(k_topk_write, dim3(njobs, TK_CHUNKS), dim3(TK_WG), 0, st, jobs, scr);
  return hipGetLastError();
}

}  // namespace mmi
