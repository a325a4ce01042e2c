// Work statistics of a plan (not on the prefill path).
//
// k_head_stats: chosen strides and phases, row-group stride and the selected
// blocks by (query modality, key modality) of every head, one launch per
// plan: the pattern search reads them for each of its plans, and copying a
// head's permutations and columns to count them on the host took most of the
// host's 2.9 of the 6.6 ms that a 24K-token, 28-head candidate cost (the
// whole search 421 -> 193 ms with this and the faster output difference).
// k_pair_count: the query-key pairs inside one head's selected blocks that
// the attention uses. Every pair of a
// selected block is computed (block semantics, "sparse loading, dense
// computation"); live query rows times live key rows with k <= q in original
// positions (all live pairs for a bidirectional head) are the useful part.
#include "device.hpp"
#include "internal.hpp"

namespace mmi {

// One workgroup per row group, one wave per member (lane = query row). A
// union entry without the member's mask bit holds 64 live keys at or below
// every query of the member; with it, the key positions are compared.
__global__ __launch_bounds__(256) void k_pair_count(const HeadDev* heads, int head, int R,
                                                    unsigned long long* out) {
  const HeadDev hd = heads[head];
  const int g = blockIdx.x;
  if (g >= hd.gp[1]) return;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (wave >= R) return;
  const int qb = group_row(g, wave, R, hd.gp[0]);
  if (qb >= hd.nbq) return;
  const int qslot = qb * B + lane;
  const int qpos = hd.qperm ? hd.qperm[qslot] : (qslot < hd.S ? qslot : -1);
  unsigned long long acc = 0;
  for (int e = hd.growptr[g]; e < hd.growptr[g + 1]; ++e) {
    const uint32_t en = (uint32_t)hd.gcol[e];
    if (!((en >> (16 + wave)) & 1u)) continue;
    const int kslot = (int)(en & 0xffffu) * B + lane;
    const int kpos = hd.kperm ? hd.kperm[kslot] : (kslot < hd.S ? kslot : -1);
    if (!((en >> (24 + wave)) & 1u)) {
      acc += qpos >= 0 ? B : 0;
      continue;
    }
    int c = 0;
    for (int x = 0; x < B; ++x) {
      const int k = __shfl(kpos, x, 64);
      c += (qpos >= 0 && k >= 0 && (!hd.causal || k <= qpos)) ? 1 : 0;
    }
    acc += c;
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane == 0 && acc) atomicAdd(out, acc);
}

// Modality of the first live slot of block j, -1 if it has none.
__device__ __forceinline__ int block_modality(const int32_t* perm, const uint8_t* mod, int j, int S) {
  for (int x = 0; x < B; ++x) {
    const int slot = j * B + x;
    const int p = perm ? perm[slot] : (slot < S ? slot : -1);
    if (p >= 0) return mod[p];
  }
  return -1;
}

// Workgroup = (head, STAT_ROWS query blocks). The modalities of the head's
// key blocks go to LDS first; each wave then walks the bitmap of a query block
// at a time, a counter per key modality.
constexpr int STAT_ROWS = 64;

__global__ __launch_bounds__(256) void k_head_stats(const HeadDev* heads, const OpDev* ops, const int32_t* op_slot,
                                                    const int32_t* nops, const uint8_t* mod, HeadStatDev* out) {
  const HeadDev hd = heads[blockIdx.x];
  HeadStatDev* o = out + blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.y == 0 && tid == 0) {
    o->group_stride = hd.gp[0];
    for (int i = 0; i < nops[blockIdx.x]; ++i) {
      const OpDev& op = ops[hd.op0 + i];
      const int slot = op_slot[hd.op0 + i];
      if (op.params && slot < MMI_MAX_MODALITIES) {
        o->sigma[slot] = op.params[0];
        o->phase[slot] = op.params[1];
      }
    }
  }
  const int q0 = blockIdx.y * STAT_ROWS;
  if (q0 >= hd.nbq) return;
  __shared__ int8_t kmod[MMI_MAX_SEQ / B + MMI_MAX_MODALITIES];   // + one block per padded group
  __shared__ unsigned long long cnt[MMI_MAX_MODALITIES * MMI_MAX_MODALITIES];
  for (int j = tid; j < hd.nbk; j += 256) kmod[j] = (int8_t)block_modality(hd.kperm, mod, j, hd.S);
  if (tid < MMI_MAX_MODALITIES * MMI_MAX_MODALITIES) cnt[tid] = 0;
  __syncthreads();
  for (int qb = q0 + wave; qb < min(q0 + STAT_ROWS, hd.nbq); qb += 4) {
    const int mq = block_modality(hd.qperm, mod, qb, hd.S);
    if (mq < 0) continue;
    int c[MMI_MAX_MODALITIES] = {};
    for (int w = lane; w < hd.nwords; w += 64)
      for (uint32_t v = hd.bitmap[(int64_t)qb * hd.nwords + w]; v; v &= v - 1) {
        const int mk = kmod[w * 32 + __ffs(v) - 1];
#pragma unroll
        for (int m = 0; m < MMI_MAX_MODALITIES; ++m) c[m] += mk == m ? 1 : 0;
      }
#pragma unroll
    for (int m = 0; m < MMI_MAX_MODALITIES; ++m) {
      for (int off = 32; off > 0; off >>= 1) c[m] += __shfl_xor(c[m], off, 64);
      if (lane == 0 && c[m]) atomicAdd(&cnt[mq * MMI_MAX_MODALITIES + m], (unsigned long long)c[m]);
    }
  }
  __syncthreads();
  if (tid < MMI_MAX_MODALITIES * MMI_MAX_MODALITIES && cnt[tid]) atomicAdd(&o->blocks[tid], cnt[tid]);
}

hipError_t launch_head_stats(const HeadDev* heads, int nheads, const OpDev* ops, const int32_t* op_slot,
                             const int32_t* nops, const uint8_t* mod, int max_nbq, HeadStatDev* out, hipStream_t st) {
  if (nheads <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_head_stats, dim3(nheads, (max_nbq + STAT_ROWS - 1) / STAT_ROWS), dim3(256), 0, st, heads, ops,
                     op_slot, nops, mod, out);
  return hipGetLastError();
}

hipError_t launch_pair_count(const HeadDev* heads, int head, int R, int ngroups, unsigned long long* out,
                             hipStream_t st) {
  if (ngroups <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pair_count, dim3(ngroups), dim3(256), 0, st, heads, head, R, out);
  return hipGetLastError();
}

}  // namespace mmi
