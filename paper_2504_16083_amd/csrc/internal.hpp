// Internal device-side descriptors and launch entry points of libmmi.
// Host C++ (runtime.hip) fills these records; the kernels in k_*.hip read
// them. Nothing here is part of the public C-ABI (include/mmi.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <stdexcept>
#include <string>

#include "../../include/mmi.h"

namespace mmi {

// Error of a host call: the C entry points turn it into their status code
// and the thread's last-error text.
struct Error : std::runtime_error {
  int code;
  Error(int c, const std::string& m) : std::runtime_error(m), code(c) {}
};

constexpr int B = 64;            // block size (rows and keys)
constexpr int D = 128;           // head dim
constexpr int LASTQ = 64;        // estimation rows
constexpr int FOLD_W = 1024;     // fold row width (max stride)
constexpr int INT_BIG = 0x7fffffff;

// Tensor view: element strides, head dim contiguous.
struct Tensor {
  const void* p;
  int64_t ss, sh;
};

// ---------------------------------------------------------------- layout
struct Segment {      // maximal run of one modality
  int32_t pos;        // first position
  int32_t len;
  int32_t loc;        // index of `pos` inside its modality's position list
  int32_t mod;
};

// ---------------------------------------------------------------- estimation
struct RowSet {       // estimation query rows: positions [row0, row0 + nrows)
  int32_t head, kvh, row0, nrows;
  int32_t nchunks;    // key chunks of pass 1
  float* part;        // [nchunks][64][2] (max, sum) in log2 domain
  float* lse2;        // [64] log2-domain LSE
};

struct EstJob {       // one query set x one key coordinate system
  int32_t head, kvh, row0, nrows, rowset;
  int32_t coord0;     // coordinate of row0 in the key system (u only)
  const int32_t* keymap;  // coordinate -> position, nullptr = identity
  int32_t L_c, ntiles;
  float* v;           // [L_c]
  float* u;           // [L_c] or nullptr
  float* dpart;       // [ntiles][128] or nullptr
};

struct GridJob {      // stride search over one job's v
  const float* v;
  int32_t L_c, lo, hi;   // candidate strides after the 2*s <= L_c cut (hi < lo: none)
  float* fold;        // [hi-lo+1][1024]
  float* score;       // [hi-lo+1]
  int32_t* pick;      // [hi-lo+1] phase of the max
  int32_t* params;    // [4] out: sigma (0 = dense), phase, L_c, nrows
  int32_t nrows;
};

struct TopkJob {
  const float* x;
  int32_t L, n;       // n <= L
  int32_t* out;       // [n] ascending
};

// ---------------------------------------------------------------- plan
struct OpDev {
  int32_t kind;               // MMI_OP_* (GRID may fall back to dense via params)
  int32_t sink, local;
  int32_t use_h, use_v, use_s;
  int32_t stride, bottom;     // SF_FIXED / SF_STRIDED stride; TRISHAPE final queries
  int32_t L;                  // extent of the op's coordinate system
  int32_t kbase, nkblk;       // first key block / number of key blocks of the key group
  const int32_t* params;      // GRID: {sigma, phase}
  const int32_t* vsel; int32_t nv;
  const int32_t* ssel; int32_t ns;
  int2* selpb;                // [nv] position and key block (from kbase) of each selected vertical
  const int32_t* keymap;      // coordinate -> position for VSLASH/VERT (nullptr = identity)
  int32_t kgrid;              // key group is Grid-ordered (VERT into a Grid group)
  const int32_t* kparams;     // that group's {sigma, phase}
  int32_t koff;               // key group slot offset
  int32_t grid[3], win[3], tile[3];   // NATTEN token grid, window, permutation tile
};

struct HeadDev {
  int32_t kind, kvh;
  int32_t causal;             // 0: bidirectional (NATTEN), only padding keys are masked
  int32_t nbq, nbk;           // permuted query / key blocks
  int32_t S;
  int32_t* qperm;             // [nbq*64] or nullptr (identity)
  int32_t* kperm;             // [nbk*64] or nullptr (identity)
  int32_t* kminpos;           // [nbk] smallest key position per key block
  int32_t* kmaxpos;           // [nbk] largest key position per key block (INT_BIG if it holds padding)
  int32_t* counts;            // [nbq]
  int32_t* rowptr;            // [nbq+1]
  uint32_t* bitmap;           // [nbq][nwords]
  int32_t nwords;
  int32_t op0;                // first OpDev of this head
  // Row groups: R query blocks processed by one work item over the union of
  // their key lists (entries: key block | flags << 16, bit r of the flags =
  // member r selects that key block). Member r of group g is query block
  // (g / rho) * R * rho + g % rho + r * rho; rho is chosen per head.
  int32_t gcap;               // capacity of the per-group arrays (>= groups for any stride)
  int32_t rho_alt[2];         // extra row-stride candidates besides 1, 2, 4, 8 (0 = none)
  int32_t* gp;                // [2] chosen row stride rho, number of groups
  int32_t* growptr;           // [ngroups+1]
  int32_t* gcol;              // [gnnz] union entries: key block, select flags << 16, mask flags << 24
  int32_t* chunks;            // [ngroups] work items per group
  int32_t* itembase;          // [ngroups] exclusive prefix of chunks
  int32_t* splitoff;          // [ngroups] exclusive prefix of (chunks > 1)
  int32_t* partoff;           // [ngroups] exclusive prefix of chunks over split groups
};

// group table (modalities present, ascending); identical for every boundary head
struct Groups {
  int32_t n;
  int32_t mod[MMI_MAX_MODALITIES];
  int32_t off[MMI_MAX_MODALITIES];    // slot offset (multiple of 64)
  int32_t len[MMI_MAX_MODALITIES];    // |T_m|
  int32_t toff[MMI_MAX_MODALITIES];   // offset of T_m inside the position pool
};

struct QbOrderJob {   // phase order of one Q-Boundary Grid modality's queries
  const int32_t* params;      // the op's {sigma, phase} (sigma <= 1: position order stays)
  int32_t* qperm;             // the head's qperm at the modality group's slot offset
  int32_t mod;                // modality id
  int32_t* cnt;               // [qb_order_chunks(S)] scratch: counts, then offsets
};

struct WorkItem {
  int32_t head, group, e0, e1;   // union entries [e0, e1) of row group `group`
  int32_t part;       // -1: write O directly; else partial slot
  int32_t lead;       // > 0: start beside the items of the run; at most this many steps' worth of waiting
  int32_t pad[2];
};

struct SplitRow {     // a row group whose union list is split over several items
  int32_t head, group, part0, nparts;
};

// ---------------------------------------------------------------- launches
// k_layout.hip
// modpos (nullable): [S] modality id of every position
hipError_t launch_positions(const Segment* segs, int nseg, const int32_t* toff_by_mod, int32_t* tpos,
                            uint8_t* modpos, int S, hipStream_t st);
// max_slots >= every head's nbq*64 and nbk*64
hipError_t launch_perms(const HeadDev* heads, int nheads, const OpDev* ops, Groups g,
                        const int32_t* tpos, int S, int max_slots, hipStream_t st);
// after launch_perms: Q-Boundary Grid modalities' queries in phase order
hipError_t launch_qb_order(const QbOrderJob* jobs, int njobs, const uint8_t* modpos, int S, hipStream_t st);
int qb_order_chunks(int S);
// k_estimate.hip
// order: [ngrp][nr] member indices (-1 = none) of the groups that read the
// same keys (row sets of one KV head; jobs of one KV head and key map).
// est_chunk_keys: keys per chunk of the LSE pass for ngrp groups of nr row
// sets over max_keys keys (a multiple of 64).
int est_chunk_keys(int ngrp, int nr, int max_keys);
hipError_t launch_est_lse(const RowSet* rs, int nrs, const int32_t* order, int ngrp, int nr, int max_chunks,
                          Tensor q, Tensor k, int chunk_keys, hipStream_t st);
hipError_t launch_est_scores(const EstJob* jobs, int njobs, const int32_t* order, int ngrp, int nr, int max_tiles,
                             const RowSet* rs, Tensor q, Tensor k, hipStream_t st);
hipError_t launch_est_udiag(const EstJob* jobs, int njobs, int max_L, hipStream_t st);
// k_select.hip
hipError_t launch_grid_search(const GridJob* jobs, int njobs, int max_cands, hipStream_t st);
// max_L: longest score array of the jobs; scr: int32 scratch of
// topk_scratch_ints(njobs, max_L) entries (initialised by the launch)
size_t topk_scratch_ints(int njobs, int max_L);
hipError_t launch_topk(const TopkJob* jobs, int njobs, int max_L, int32_t* scr, hipStream_t st);
// k_blocks.hip
hipError_t launch_key_summaries(const HeadDev* heads, int nheads, OpDev* ops, int nops,
                                Groups g, int max_nbk, int max_sel, hipStream_t st);
// cand: int64 [nheads][NRHO], cleared by this launch for launch_group_stride
constexpr int NRHO = 6;
hipError_t launch_blocks_count(const HeadDev* heads, int nheads, const OpDev* ops, Groups g, int max_nbq,
                               int64_t* cand, hipStream_t st);
// Union sizes of every row group for each head's candidate row strides 1, 2,
// 4, 8 and its rho_alt (gcnt [nheads][NRHO][max_groups]) and their totals
// (cand); extra: some head has rho_alt candidates.
hipError_t launch_group_stride(const HeadDev* heads, int nheads, int R, int max_groups, int max_nbq, bool extra,
                               int64_t* cand, int32_t* gcnt, hipStream_t st);
// Each head's stride (smallest total union, ties to the earlier candidate)
// and offsets; totals[head] = {nnz, gnnz, nitems, nsplit, nparts}. A union is
// split into work items beyond max(min_chunk, staged blocks of the layer /
// items) entries; min_chunk 0: from the average union of the all_groups groups.
constexpr int NTOT = 5;
hipError_t launch_blocks_scan(const HeadDev* heads, int nheads, int R, const int64_t* cand, const int32_t* gcnt,
                              int max_groups, int min_chunk, int items, int all_groups, int64_t* totals, hipStream_t st);
hipError_t launch_group_fill(const HeadDev* heads, int nheads, int R, int max_groups, int max_nbk, hipStream_t st);
// Runs of consecutive work items and their slots in the item map ([8][cap *
// run], -1 = none): 32 items per run, fewer for small layers so that every XCD
// gets some, more where there would be over MAP_RUNS runs; at most a quarter
// more runs on an XCD than the average.
constexpr int MAP_RUNS = 4096, MAP_CAP = MAP_RUNS / 8 + MAP_RUNS / 32 + 2;
struct MapShape {
  int32_t run, nruns, cap;
};
inline MapShape map_shape(int64_t n) {
  int64_t run = n / 64 < 1 ? 1 : n / 64 < 32 ? n / 64 : 32;
  if (n > run * MAP_RUNS) run = (n + MAP_RUNS - 1) / MAP_RUNS;
  const int64_t nruns = (n + run - 1) / run, avg = (nruns + 7) / 8;
  return {(int32_t)run, (int32_t)nruns, (int32_t)(avg + (avg / 4 > 1 ? avg / 4 : 1))};
}
// Items whose workgroups start side by side (WorkItem::lead): long walks over
// the K and V of a head with many keys (32 KB per 64 of them, once: the key
// layouts of a Q-Boundary head hold the same keys), which miss the 256 MB
// last-level cache when they are read apart. Attention without | with waiting,
// 28/4 heads unless said:
//   from RUN_KEYS key blocks (as much as the cache), walks of RUN_STEPS steps:
//     mixed heads 512K 303 | 283 ms, 768K 505 | 459, 1M 655 | 588;
//   from RUN_KEYS_LONG, walks of RUN_STEPS_LONG steps, which lose each other
//     over fewer keys: two mixed layers, 384K 202.2 | 200.3 and 251.4 | 245.1,
//     340K 174.7 | 172.0 and 219.2 | 213.1, 300K 144.8 | 145.7 and 181.1 |
//     178.9; below it the waiting loses: 256K 112.2 | 115.8 and 138.6 | 142.1;
//   from RUN_KEYS_DENSE, such walks over unions that every member of the row
//     group selects (all but the blocks past a member's last query), so that
//     the walks of a run read the same blocks: dense 256K 489 | 453. (With
//     three of four members as the line some walks of the mixed 256K layers
//     wait and some do not: 115.9 and 142.9.)
constexpr int RUN_KEYS = 8192, RUN_STEPS = 256;
constexpr int RUN_KEYS_LONG = 4608, RUN_STEPS_LONG = 1024;
constexpr int RUN_KEYS_DENSE = 4096;
// WorkItem::lead of an item of `steps` of the `staged` union entries of a row
// group of R members that computes `computed` blocks over them.
__host__ __device__ inline int lead_steps(int S, int R, int steps, int staged, int computed) {
  const int keys = (S + B - 1) / B;
  const bool dense = 40 * (int64_t)computed >= 39 * (int64_t)R * staged;
  const bool side = keys >= RUN_KEYS ? steps >= RUN_STEPS
                                     : steps >= RUN_STEPS_LONG && keys >= (dense ? RUN_KEYS_DENSE : RUN_KEYS_LONG);
  return side ? steps : 0;
}
// Entries of an XCD's list that start side by side: a run, or all (nobody
// waits) where a run would leave more than an eighth of the XCD's workgroups
// asleep, as it does in layers of under 1800 items (one head of 256K to 450K
// tokens). Dense, one head, attention with a run waiting | nobody waiting:
// 256K (run 16) 18.6 | 16.7 ms, 300K (18) 25.6 | 23.3, 350K (21) 33.9 | 31.5,
// 400K (24) 42.9 | 41.1, 450K (27) 52.9 | 51.5, 500K (30) 62.7 | 63.5, 512K
// (32) 65.1 | 67.5. (As many whole runs as give each workgroup an item, 256K
// to 450K: 17.2, 23.1, 32.8, 41.6, 52.1.)
inline int32_t side_by_side(int32_t run, int32_t cus) { return run < cus * 7 / 64 ? INT_BIG : run; }
// Entries of the list that are finished before entry k starts, if it waits.
constexpr int LEAD_SLACK = 2;            // items of the run before that may still be running
__host__ __device__ inline int lead_need(int k, int side) { return k / side * side - LEAD_SLACK; }
hipError_t launch_work_fill(const HeadDev* heads, int nheads, int R, const int64_t* item_base,
                            const int64_t* part_base, const int64_t* split_base, int max_groups,
                            WorkItem* items, float* cost, SplitRow* splits, hipStream_t st);
// also clears queues[nqueues]
hipError_t launch_item_map(const float* cost, int64_t n, int32_t* map, int32_t* queues, int nqueues, hipStream_t st);
// k_attention.hip
struct AttnArgs {
  Tensor q, k, v;
  void* o; int64_t o_ss, o_sh;
  float* lse;                 // [Hq][S] or nullptr
  int32_t S;
  const HeadDev* heads;
  const WorkItem* items;
  int64_t nitems;
  const int32_t* item_map;    // [8][map_len]: work items of each XCD in order, -1 = none
  int64_t map_len;
  int32_t side;               // entries of a list that start side by side
  float* part_o;              // [nparts][R*64][128], each row normalised by its bf16-P sum
  float* part_ml;             // [nparts][R*64][4]: running max m, bf16-P sum lo, fp32-P sum l, unused
  int32_t R;                  // query blocks per row group (1, 2 or 4)
  int32_t* queue;             // QUEUE_INTS zeroed counters of one launch at a time (left zeroed), or
                              // nullptr: one workgroup per item
  int32_t cus;                // persistent workgroups (a multiple of 8)
};
constexpr int QUEUE_LINE = 32;              // one counter per 128 bytes
constexpr int QUEUE_INTS = 17 * QUEUE_LINE; // entries taken of 8 lists, entries finished, workgroups through
hipError_t launch_attention(const AttnArgs& a, hipStream_t st);
hipError_t launch_combine(const AttnArgs& a, const SplitRow* splits, int64_t nsplit, hipStream_t st);
// k_search.hip: out[h * n_class + c] = sum over x with cls[x] == c of |a[x,h] - b[x,h]|^2
// (bf16 outputs of S x H rows); part: scratch of H * n_class * SQ_CHUNKS doubles, or nullptr (fewer workgroups)
constexpr int SQ_CHUNKS = 64;
hipError_t launch_sqerr(const void* a, const void* b, int64_t ss, int64_t sh, const uint8_t* cls, int n_class,
                        int S, int H, double* out, double* part, hipStream_t st);
// k_permute.hip
hipError_t launch_permute(const void* src, int64_t ss, void* dst, int64_t ds, const int32_t* perm,
                          int64_t n, int64_t row_bytes, int inverse, hipStream_t st);

// k_stats.hip: what mmi_plan_stats reports from the device, for every head
// (out zeroed by the caller; op_slot: export slot of every op, nops: ops of
// every head, mod: modality of every position)
struct HeadStatDev {
  unsigned long long blocks[MMI_MAX_MODALITIES * MMI_MAX_MODALITIES];
  int32_t sigma[MMI_MAX_MODALITIES], phase[MMI_MAX_MODALITIES];
  int32_t group_stride, pad;
};
hipError_t launch_head_stats(const HeadDev* heads, int nheads, const OpDev* ops, const int32_t* op_slot,
                             const int32_t* nops, const uint8_t* mod, int max_nbq, HeadStatDev* out, hipStream_t st);
// useful query-key pairs of one head's selected blocks, added to *out
hipError_t launch_pair_count(const HeadDev* heads, int head, int R, int ngroups, unsigned long long* out,
                             hipStream_t st);

// ---------------------------------------------------------------- check.hip
// Host consistency checks of a plan's tables: empty, or the first violation.
std::string check_index(const mmi_index_view& v);
std::string check_work(const mmi_work_view& w);

// The pattern search of Algorithm 4 (search.hip) over plans of this library;
// the problem is already validated, out has prob.Hq entries.
void search_layer(mmi_ctx* ctx, const mmi_problem& prob, const void* q, const void* k, const void* v,
                  const mmi_op* cands, int nc, const mmi_op* xc, int nx, const mmi_op& target, hipStream_t st,
                  mmi_head_cfg* out, mmi_search_report* rep);

}  // namespace mmi
