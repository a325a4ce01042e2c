// Online estimate of the attention map from the final queries (Algorithm 1,
// first step; Appendix C.3): A_hat[r, k] = exp(tau q_r.k_k - LSE_r) for
// k <= pos(r), each row normalised over all causal keys of the sequence.
//
// Pass 1 (k_est_lse): per query set and key chunk, running (max, sum) of
//   2^(tau log2e q.k) per row -> partials; k_est_merge folds the chunks in
//   a fixed order into log2-domain LSE.
// Pass 2 (k_est_scores): per query set and run of 64-key tiles of the key
//   coordinate system, A_hat tile through MFMA, the column sums (v, written
//   directly: each tile owns its keys) from registers and, where the job asks
//   for diagonals, the 127 diagonal partial sums of the tile in LDS;
//   k_est_udiag adds the (at most two) tiles that
//   touch each diagonal offset. Every reduction has a fixed order, so the
//   scores are bitwise reproducible.
// The query rows are contiguous positions [row0, row0+nrows), nrows <= 64,
// and contiguous in the key coordinate system too (coordinate coord0 + r).
// The query sets that read the same keys (pass 1: one KV head; pass 2 also
// one key coordinate system) form a group, and the work of a group over one
// key range runs back to back on one XCD. Pass 1 takes up to four sets of a
// group per workgroup (two waves each, 32 rows per wave, the query rows in
// registers as the MFMA B operand): each 64-key tile is loaded once by all
// 512 threads into LDS (the next tile's rows load while the current one is
// multiplied) and read as the A operand by every set. Pass 2 takes one job
// per workgroup and reads its K rows straight from HBM into MFMA operands,
// each row by one wave (wave w multiplies keys 32 w .. 32 w + 31 of every
// tile by all 64 rows; two tiles of rows in registers: tile t + 2 loads
// while t and t + 1 are multiplied and reduced); the jobs of a group over
// one range find it in that XCD's L2.
#include <algorithm>

#include "device.hpp"
#include "internal.hpp"

namespace mmi {

namespace {

constexpr float SC = 0.08838834764831845f * LOG2E;   // sqrt(1/128) * log2(e)
constexpr int EKP = 136;          // bf16 per staged K row (272 B: conflict-free operand reads)
constexpr int EMEM = 4;           // query sets (LSE pass) or score jobs per workgroup, 2 waves each

// Logical work index of physical workgroup b when runs of `run` consecutive
// logical items go to one XCD (workgroups are dispatched to the 8 XCDs in
// turn) and the runs to XCDs in turn.
__device__ __forceinline__ int64_t run_item(int64_t b, int run) {
  const int64_t xcd = b & 7, k = b >> 3;
  return (k / run) * (8 * (int64_t)run) + xcd * run + (k % run);
}

struct __align__(16) EstStage {
  uint16_t k[B * EKP];
};

__device__ __forceinline__ void load_q_operand(bf16x8 (&qr)[8], const Tensor& q, int head, int pos,
                                               int h) {
  const uint16_t* row = reinterpret_cast<const uint16_t*>(q.p) + (int64_t)head * q.sh +
                        (int64_t)max(pos, 0) * q.ss + h * 64;
#pragma unroll
  for (int s = 0; s < 8; ++s) qr[s] = pos >= 0 ? load16(row + 8 * s) : zero8();
}

// This thread's 32 bytes of key row kpos (zeros for kpos < 0): thread
// (key, part) of the 512 stages dims [16 part, 16 part + 16) of one key.
__device__ __forceinline__ void fetch_key(bf16x8 (&r)[2], const Tensor& k, int kvh, int kpos, int part) {
  const uint16_t* row = reinterpret_cast<const uint16_t*>(k.p) + (int64_t)kvh * k.sh +
                        (int64_t)max(kpos, 0) * k.ss + part * 16;
  r[0] = kpos >= 0 ? load16(row) : zero8();
  r[1] = kpos >= 0 ? load16(row + 8) : zero8();
}

__device__ __forceinline__ void stage_key(EstStage& st, const bf16x8 (&r)[2], int key, int part) {
  *reinterpret_cast<bf16x8*>(&st.k[key * EKP + part * 16]) = r[0];
  *reinterpret_cast<bf16x8*>(&st.k[key * EKP + part * 16 + 8]) = r[1];
}

// S^T of the 64 staged keys x this wave's 32 queries: s[kt] holds keys
// 32 kt + 8i + 4h + j for query c in element 4i + j.
__device__ __forceinline__ void staged_product(const EstStage& st, const bf16x8 (&qr)[8], int c, int h,
                                               f32x16 (&s)[2]) {
  const f32x16 zero = {};
#pragma unroll
  for (int st8 = 0; st8 < 8; ++st8) {
    const bf16x8 k0 = *reinterpret_cast<const bf16x8*>(&st.k[c * EKP + h * 64 + st8 * 8]);
    const bf16x8 k1 = *reinterpret_cast<const bf16x8*>(&st.k[(32 + c) * EKP + h * 64 + st8 * 8]);
    s[0] = mfma32(k0, qr[st8], st8 == 0 ? zero : s[0]);
    s[1] = mfma32(k1, qr[st8], st8 == 0 ? zero : s[1]);
  }
}


// This lane's half of key row kpos (zeros for kpos < 0): the K operand of
// one 32-key tile.
__device__ __forceinline__ void load_key(bf16x8 (&ka)[8], const Tensor& k, int kvh, int kpos, int h) {
  const uint16_t* row = reinterpret_cast<const uint16_t*>(k.p) + (int64_t)kvh * k.sh +
                        (int64_t)max(kpos, 0) * k.ss + h * 64;
#pragma unroll
  for (int s = 0; s < 8; ++s) ka[s] = kpos >= 0 ? load16(row + 8 * s) : zero8();
}

// S tile of 32 queries x 32 keys; lane (c, h) holds queries 8i + 4h + j for key c.
__device__ __forceinline__ f32x16 key_product(const bf16x8 (&qr)[8], const bf16x8 (&ka)[8]) {
  f32x16 acc;
#pragma unroll
  for (int x = 0; x < 16; ++x) acc[x] = 0.0f;
#pragma unroll
  for (int s = 0; s < 8; ++s) acc = mfma32(qr[s], ka[s], acc);
  return acc;
}

}  // namespace

// Pass 1. Logical item = (group, key chunk, batch of EMEM members):
// order[group * nr + member] is a row-set index (-1 = none); the row sets
// of a group share one KV head, so every 64-key tile of the chunk is staged
// once in LDS and multiplied by all members' query rows. Waves w and w + 4
// hold rows 0-31 and 32-63 of member w. Per row: running (max, sum) of
// 2^(tau log2e q.k) over its causal keys of the chunk, the fixed order of
// the tiles, then the two key halves of each tile.
__global__ __launch_bounds__(512) void k_est_lse(const RowSet* sets, const int32_t* order, int ngrp, int nr,
                                                 int nbat, int nch, Tensor q, Tensor k, int chunk_keys) {
  __shared__ EstStage stg[2];
  const int64_t lg = run_item(blockIdx.x, nbat);
  const int bat = (int)(lg % nbat);
  const int64_t pair = lg / nbat;
  const int grp = (int)(pair / nch), ch = (int)(pair % nch);
  if (grp >= ngrp) return;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, c = lane & 31, h = lane >> 5;
  int kend = 0;                        // keys [0, kend) are visible to some member
  for (int m = 0; m < EMEM; ++m) {
    const int mi = bat * EMEM + m;
    const int si = mi < nr ? order[grp * nr + mi] : -1;
    if (si >= 0) kend = max(kend, sets[si].row0 + sets[si].nrows);
  }
  const int k0 = ch * chunk_keys;
  if (k0 >= kend) return;
  const int k1 = min(k0 + chunk_keys, kend);
  const int kvh = sets[order[grp * nr]].kvh;
  const int mem = wave & (EMEM - 1), half = wave >> 2;
  const int mi = bat * EMEM + mem;
  const int si = mi < nr ? order[grp * nr + mi] : -1;
  RowSet rs{};
  if (si >= 0) rs = sets[si];
  const bool active = si >= 0 && ch < rs.nchunks;
  const int r = half * 32 + c;
  const int qpos = active && r < rs.nrows ? rs.row0 + r : -1;
  bf16x8 qr[8];
  load_q_operand(qr, q, rs.head, qpos, h);
  const int key = tid >> 3, part = tid & 7;
  const int ntile = (k1 - k0 + B - 1) / B;
  bf16x8 rg[2];
  fetch_key(rg, k, kvh, k0 + key < k1 ? k0 + key : -1, part);
  stage_key(stg[0], rg, key, part);
  if (ntile > 1) fetch_key(rg, k, kvh, k0 + B + key < k1 ? k0 + B + key : -1, part);
  __syncthreads();
  float m = NEG_BIG, l = 0.0f;
  for (int t = 0; t < ntile; ++t) {
    const int kb = k0 + t * B;
    if (active) {
      f32x16 s[2];
      staged_product(stg[t & 1], qr, c, h, s);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        float mx = NEG_BIG;
        float x[16];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int kk = kb + kt * 32 + 8 * i + 4 * h + j;
            const float v = s[kt][4 * i + j] * SC;
            x[4 * i + j] = (kk < k1 && kk <= qpos) ? v : -INFINITY;
            mx = fmaxf(mx, x[4 * i + j]);
          }
        const float mn = fmaxf(m, mx);
        float acc = 0.0f;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc += fast_exp2(x[e] - mn);
        l = l * fast_exp2(m - mn) + acc;
        m = mn;
      }
    }
    // tile t+1 was loaded during tile t-1; its stage was last read in tile t-1
    if (t + 1 < ntile) {
      stage_key(stg[(t + 1) & 1], rg, key, part);
      const int nk = k0 + (t + 2) * B + key;
      if (t + 2 < ntile) fetch_key(rg, k, kvh, nk < k1 ? nk : -1, part);
    }
    __syncthreads();
  }
  if (!active) return;
  const float m2 = __shfl_xor(m, 32), l2 = __shfl_xor(l, 32);
  const float mt = fmaxf(m, m2);
  const float lt = h == 0 ? l * fast_exp2(m - mt) + l2 * fast_exp2(m2 - mt)
                          : l2 * fast_exp2(m2 - mt) + l * fast_exp2(m - mt);
  if (h == 0 && r < rs.nrows) {
    float* p = rs.part + ((int64_t)ch * LASTQ + r) * 2;
    p[0] = mt;
    p[1] = lt;
  }
}

// The chunks' (max, sum) pairs of every row folded in a fixed order: one lane
// per row, wave w takes chunks w, w + MERGE_W, ... (running maximum, so each
// partial is read once), then wave 0 folds the waves. One wave walking 256
// chunks twice took 129 us at 1M tokens: the latency of one dependent step after
// another.
constexpr int MERGE_W = 16;

__device__ __forceinline__ void fold_part(float& M, float& L, float m, float l) {
  const float mn = fmaxf(M, m);
  L = L * fast_exp2(M - mn) + l * fast_exp2(m - mn);
  M = mn;
}

__global__ __launch_bounds__(64 * MERGE_W) void k_est_merge(const RowSet* sets) {
  const RowSet rs = sets[blockIdx.x];
  __shared__ float2 sh[MERGE_W][LASTQ];
  const int r = threadIdx.x & 63, w = threadIdx.x >> 6;
  float M = NEG_BIG, L = 0.0f;
  if (r < rs.nrows) {
    const float2* part = reinterpret_cast<const float2*>(rs.part);
#pragma unroll 4
    for (int ch = w; ch < rs.nchunks; ch += MERGE_W) {
      const float2 p = part[(int64_t)ch * LASTQ + r];
      fold_part(M, L, p.x, p.y);
    }
  }
  sh[w][r] = make_float2(M, L);
  __syncthreads();
  if (w > 0 || r >= rs.nrows) return;
  for (int v = 1; v < MERGE_W; ++v) fold_part(M, L, sh[v][r].x, sh[v][r].y);
  rs.lse2[r] = M + fast_log2(L);
}

constexpr int APITCH = 65;   // floats per key row of A_hat in LDS: odd, so that a row's lanes and a
                             // diagonal's rows fall in different banks
constexpr int EST_TPW_MAX = 8;  // most 64-key tiles per workgroup of the score pass

// Each workgroup takes tpw consecutive tiles of one job: the query rows are
// loaded once, and the key positions and K rows of the tile after next load
// while the current tile is reduced. A tile comes out of the MFMAs with one
// key per lane and the query rows in its registers, so a column sum is a sum
// over registers and one lane swap: jobs without diagonals (Grid, VERT) need
// neither LDS nor barriers, the others put the tile in LDS for the diagonal
// sums only. (With the queries over the lanes both sums went through LDS,
// three barriers a tile: 66K Grid jobs 105.6 -> 87.5 us, 128K 290 -> 240, 256K
// 356 -> 312.)
// Logical item = (group, run of tpw tiles, member): order[group * nr +
// member] is a job index (-1 = none), nrun runs per group.
__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(2))) void k_est_scores(const EstJob* jobs, const int32_t* order, int ngrp, int nr,
                                                    int nrun, int tpw, const RowSet* sets, Tensor q, Tensor k) {
  __shared__ __align__(16) float ahat[B * APITCH];
  const int64_t lg = run_item(blockIdx.x, nr);
  const int64_t pair = lg / nr;
  const int grp = (int)(pair / nrun), tr = (int)(pair % nrun);
  if (grp >= ngrp) return;
  const int ji = order[grp * nr + (int)(lg % nr)];
  if (ji < 0) return;
  const EstJob jb = jobs[ji];
  const int ta = tr * tpw;
  if (ta >= jb.ntiles) return;
  const int tb = min(ta + tpw, jb.ntiles);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, c = lane & 31, h = lane >> 5;
  // wave w multiplies all 64 rows by keys 32 w .. 32 w + 31 of each tile (each
  // K row is loaded once per workgroup); lane (c, h) holds rows c and 32 + c as
  // A operands and, of the product, key c and rows 32 hf + 8 i + 4 h + j
  float lse2[2][16];
  bf16x8 qr[2][8];
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
    const int r = hf * 32 + c;
    load_q_operand(qr[hf], q, jb.head, r < jb.nrows ? jb.row0 + r : -1, h);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int x = hf * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
      lse2[hf][e] = x < jb.nrows ? sets[jb.rowset].lse2[x] : 0.0f;
    }
  }
  auto key_pos = [&](int kap) { return kap < jb.L_c ? (jb.keymap ? jb.keymap[kap] : kap) : -1; };
  // two tiles of K rows in registers: tile t + 2 loads while tiles t and t + 1 are used
  int kp[2];
  bf16x8 ka[2][8];
  auto fetch = [&](int buf, int t) {
    kp[buf] = key_pos(t * B + wave * 32 + c);
    load_key(ka[buf], k, jb.kvh, kp[buf], h);
  };
  auto tile = [&](int buf, int t) {
    f32x16 s[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) s[hf] = key_product(qr[hf], ka[buf]);
    // rows from `first` on see the lane's key (none if it is past L_c)
    const int first = kp[buf] >= 0 ? kp[buf] - jb.row0 : INT_BIG;
    if (t + 2 < tb) fetch(buf, t + 2);
    float sum = 0.0f;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int r = hf * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
        const float a = first <= r && r < jb.nrows ? fast_exp2(s[hf][e] * SC - lse2[hf][e]) : 0.0f;
        s[hf][e] = a;
        sum += a;
      }
    const float other = __shfl_xor(sum, 32);
    const int kap = t * B + wave * 32 + c;
    if (h == 0 && kap < jb.L_c) jb.v[kap] = sum + other;
    if (!jb.dpart) return;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int e = 0; e < 16; ++e) ahat[(wave * 32 + c) * APITCH + hf * 32 + 8 * (e >> 2) + 4 * h + (e & 3)] = s[hf][e];
    __syncthreads();
    // diagonals d = r - kk + 63 in [0, 127): d and d + 64 together hold one key
    // of every row (rows up to d the first, the others the second), so a pair
    // of lanes takes both, 32 rows each, the rows ascending
    {
      const int d = wave * 32 + c;
      float lo = 0.0f, hi = 0.0f;
#pragma unroll 16
      for (int i = 0; i < 32; ++i) {
        const int r = h * 32 + i;
        const float x = ahat[((r + 63 - d) & 63) * APITCH + r];
        lo += r <= d ? x : 0.0f;
        hi += r <= d ? 0.0f : x;
      }
      const float lo2 = __shfl_xor(lo, 32), hi2 = __shfl_xor(hi, 32);
      float* dp = jb.dpart + (int64_t)t * 128 + d;
      if (h == 0) dp[0] = lo + lo2;
      else dp[64] = hi2 + hi;
    }
    __syncthreads();    // ahat is rewritten by the next tile
  };
  fetch(0, ta);
  if (ta + 1 < tb) fetch(1, ta + 1);
  for (int t = ta; t < tb; t += 2) {
    tile(0, t);
    if (t + 1 < tb) tile(1, t + 1);
  }
}

__device__ __forceinline__ int floordiv(int a, int b) {
  int q = a / b;
  return (a % b != 0 && ((a < 0) != (b < 0))) ? q - 1 : q;
}

// u[o] = sum over tiles t (ascending) of dpart[t][o - coord0 + 64 t + 63].
__global__ __launch_bounds__(256) void k_est_udiag(const EstJob* jobs) {
  const EstJob jb = jobs[blockIdx.x];
  if (!jb.u) return;
  const int o = blockIdx.y * 256 + threadIdx.x;
  if (o >= jb.L_c) return;
  const int base = jb.coord0 - o;
  const int tlo = max(0, -floordiv(-(base - 63), 64));   // ceil((base - 63) / 64)
  const int thi = min(jb.ntiles - 1, floordiv(base + 63, 64));
  float acc = 0.0f;
  for (int t = tlo; t <= thi; ++t) {
    const int d = o - jb.coord0 + 64 * t + 63;
    if (d >= 0 && d < 127) acc += jb.dpart[(int64_t)t * 128 + d];
  }
  jb.u[o] = acc;
}

// Workgroups for ngrp groups x nper items x nr members, rounded up to whole
// runs of nr on each of the 8 XCDs.
static unsigned grouped_grid(int ngrp, int nper, int nr) {
  const int64_t items = (int64_t)ngrp * nper * nr, run = 8 * (int64_t)nr;
  return (unsigned)((items + run - 1) / run * run);
}

// Keys per workgroup of the LSE pass: the pass is a serial chain of 64-key
// tiles (about 1.6 us each) per workgroup, so short inputs are cut until
// some EST_FILL workgroups run (four fit a CU); long ones keep 4096 keys, where a
// chunk's partials and query loads cost nothing beside its tiles. 4096 keys
// always: 105 us at 4K tokens and 2 heads, 83 us at 3K and 28 heads (a whole
// layer 448 -> 338 and 536 -> 446 us with this and the score pass's rule).
constexpr int EST_FILL = 1024, EST_CHUNK_MAX = 4096, EST_CHUNK_MIN = 128;

int est_chunk_keys(int ngrp, int nr, int max_keys) {
  const int64_t tiles = (int64_t)std::max(ngrp, 1) * ((std::max(nr, 1) + EMEM - 1) / EMEM) * ((max_keys + B - 1) / B);
  const int64_t keys = (tiles + EST_FILL - 1) / EST_FILL * B;
  return (int)std::min<int64_t>(EST_CHUNK_MAX, std::max<int64_t>(EST_CHUNK_MIN, keys));
}

hipError_t launch_est_lse(const RowSet* rs, int nrs, const int32_t* order, int ngrp, int nr, int max_chunks,
                          Tensor q, Tensor k, int chunk_keys, hipStream_t st) {
  if (nrs <= 0) return hipSuccess;
  const int nbat = (nr + EMEM - 1) / EMEM;
  hipLaunchKernelGGL(k_est_lse, dim3(grouped_grid(ngrp, max_chunks, nbat)), dim3(512), 0, st, rs, order, ngrp, nr,
                     nbat, max_chunks, q, k, chunk_keys);
  hipLaunchKernelGGL(k_est_merge, dim3(nrs), dim3(64 * MERGE_W), 0, st, rs);
  return hipGetLastError();
}

hipError_t launch_est_scores(const EstJob* jobs, int njobs, const int32_t* order, int ngrp, int nr, int max_tiles,
                             const RowSet* rs, Tensor q, Tensor k, hipStream_t st) {
  if (njobs <= 0) return hipSuccess;
  // eight workgroups of two waves fit a CU: fewer tiles each until 2048 run
  const int64_t tiles = (int64_t)njobs * max_tiles;
  const int tpw = (int)std::min<int64_t>(EST_TPW_MAX, std::max<int64_t>(1, tiles / 2048));
  const int nrun = (max_tiles + tpw - 1) / tpw;
  hipLaunchKernelGGL(k_est_scores, dim3(grouped_grid(ngrp, nrun, nr)), dim3(128), 0, st, jobs, order, ngrp, nr,
                     nrun, tpw, rs, q, k);
  return hipGetLastError();
}

hipError_t launch_est_udiag(const EstJob* jobs, int njobs, int max_L, hipStream_t st) {
  if (njobs <= 0 || max_L <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_est_udiag, dim3(njobs, (max_L + 255) / 256), dim3(256), 0, st, jobs);
  return hipGetLastError();
}

}  // namespace mmi
