// lg_prune.hip -- Stage 2 of LoopGuard: the retained index set and in-place cache compaction
// (Sec. 5.3, Eq. (10) and Eq. (11)), plus the per-step commit of the appended row and budget
// upkeep.
//
// keepset_kernel (one workgroup per sequence): commit the append, decide whether the sequence is
// pruned (trigger, or cache at its budget), and write the kept slots to keep_idx:
//   kept(j) = anchor(j) or (middle(j) and rank_mid(j) is one of the S evenly spaced ranks) or
//             (clean recent(j) and it is among the last R >> l clean recent slots)
// Positions ascend over the slots, so these regions are ranges whose ends are found by search and
// every kept slot has a closed form; pos is gathered in place.
//
// With the baseline policies (H2O, StreamingLLM; Sec. 6.1) only a cache at its budget is pruned and
// the kept set is the policy's: h2o_score_kernel first sums every slot's acc over the layers and KV
// heads into keep_idx (float bits, used as scratch), and keepset_kernel finds the H2O threshold
// key by an 8-bit radix select over (score, slot) keys and stream-compacts the slots at or above it
// with block-wide prefix sums.
//
// compact_kernel (a workgroup at a time per 128-byte column of a (sequence, layer, kv head)'s K or V
// rows): moves K, V and acc rows r <- keep_idx[r] in place. keep_idx is ascending with keep_idx[r] >= r,
// so walking the rows in chunks, reading a whole chunk before writing it, never overwrites a row a later
// chunk reads; the next chunk's loads are issued before the current chunk's stores.
#include <algorithm>

#include "lg_keepset.h"

namespace lg {

constexpr int kMaxLayersPerLaunch = 64;

struct ScoreArgs {
  const float* acc[kMaxLayersPerLaunch];
  int32_t n_layers, first;  // layers in this launch; the first launch writes, later ones add
  int32_t B, Hkv, cap;
  const int32_t* len;
  const int32_t* budget;
  const int32_t* t_append;
  float* score;             // keep_idx viewed as float [B][cap]
};

// Live slots after the commit of the append, as keepset_kernel computes them.
__device__ __forceinline__ int committed_len(const int32_t* len, const int32_t* t_append, int b,
                                             int cap) {
  int L = len[b];
  L = L < 0 ? 0 : (L > cap ? cap : L);
  if (t_append != nullptr && L < cap) L += 1;
  return L;
}

// H2O score of every live slot of a sequence at its budget: acc summed over this launch's layers
// (ascending) and KV heads (ascending) in float32, added to the previous launches' partial sum.
__global__ __launch_bounds__(256) void h2o_score_kernel(ScoreArgs a) {
  const int b = blockIdx.y;
  const int L = committed_len(a.len, a.t_append, b, a.cap);
  if (L < min(a.budget[b], a.cap)) return;  // not pruned at this step
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= L) return;
  float* sc = a.score + (size_t)b * a.cap;
  float s = a.first ? 0.f : sc[j];
  // Terms i = l * Hkv + h in ascending order; each chunk of kChunk terms is loaded before it is
  // added, so the loads are in flight together while the additions keep their order.
  constexpr int kChunk = 16;
  const int total = a.n_layers * a.Hkv;
  const size_t row = (size_t)b * a.Hkv * a.cap + j;
  for (int i0 = 0; i0 < total; i0 += kChunk) {
    float v[kChunk];
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
      const int i = i0 + k;
      if (i < total) {
        const int l = i / a.Hkv, h = i - l * a.Hkv;
        v[k] = a.acc[l][row + (size_t)h * a.cap];
      }
    }
#pragma unroll
    for (int k = 0; k < kChunk; ++k)
      if (i0 + k < total) s = s + v[k];
  }
  sc[j] = s;
}

struct CompactLayer {
  void* k;
  void* v;
  float* acc;
};

struct CompactArgs {
  CompactLayer layer[kMaxLayersPerLaunch];
  const int32_t* keep_idx;
  const int32_t* new_len;
  int32_t B, Hkv, cap, row_bytes;
  int32_t n_layers;               // layers of this launch
  int32_t n_col;                  // 128-byte columns of a K row and a V row together
  int32_t per_seq;                // items of a sequence: n_layers x Hkv x n_col
  int32_t step_rank, step_rest;   // the grid as whole sequences and items
};

__global__ __launch_bounds__(kKeepThreads) void keepset_kernel(KeepArgs a) {
  const int b = blockIdx.x;
  const KeepInputs in = load_keep_inputs(a, b);
  bool trig = false;
  int span = -1, level = 0;
  if (a.policy == LG_POLICY_LOOPGUARD && a.decision != nullptr) {
    trig = a.decision[b].trigger != 0;
    span = a.decision[b].span_lo;
    level = a.decision[b].level;
  }
  keep_set_block<kKeepThreads>(a, in, trig, span, level);
}

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// A compaction workgroup moves one 128-byte column of one layer's K or V for one KV head: a row's
// columns are independent, so a sequence's rows spread over row_bytes / 64 times as many workgroups
// as there are (layer, kv head) pairs. With whole K and V rows per workgroup, one flagged sequence
// (the usual event) of the 7B shape was 112 workgroups, each a chain of ten dependent passes:
// 52.8 us for the 1261 rows in 28 layers on MI355X, 33 us now; all 32 sequences at once 0.89 ms (5.5
// GB, read and written), 0.91 ms before. Threads x rows in flight per thread, for one sequence (the
// whole call) / for all: 256 x 8 44.1 / 915 us, 512 x 8 44.8 / 861, 512 x 4 41.8 / 888, 1024 x 4
// 48.0 / 831, 1024 x 8 (spills) 95 / 869.
constexpr int kCompactThreads = 512;
constexpr int kCompactUnroll = 4;                        // rows in flight per thread
constexpr int kColBytes = 128;
constexpr int kColLanes = kColBytes / 16;                // lanes of a row
constexpr int kPassRows = kCompactThreads / kColLanes;   // rows of one load instruction
constexpr int kRowsPerPass = kPassRows * kCompactUnroll;
constexpr int kCompactWorkgroups = 1024;
static_assert(kRowsPerPass <= kCompactThreads, "at most one score per thread and pass");

// Rows of a compaction pass, held in registers between its loads and its stores.
struct MovePass {
  u32x4_t x[kCompactUnroll];
  int src[kCompactUnroll];
  float acc;     // column 0 of K only: the score of row r0 + tid
  int acc_src;
};

__device__ __forceinline__ void compact_load(MovePass& m, int r0, int rsub, int nl,
                                             const int32_t* kidx, const char* col, int row_bytes,
                                             const float* acc) {
#pragma unroll
  for (int u = 0; u < kCompactUnroll; ++u) {  // all source indices first: one wait before the loads
    const int r = r0 + u * kPassRows + rsub;
    m.src[u] = r < nl ? kidx[r] : r;
  }
  const int ra = r0 + (int)threadIdx.x;
  m.acc_src = acc != nullptr && (int)threadIdx.x < kRowsPerPass && ra < nl ? kidx[ra] : ra;
#pragma unroll
  for (int u = 0; u < kCompactUnroll; ++u) {
    const int r = r0 + u * kPassRows + rsub;
    if (m.src[u] != r)  // rows are read once: non-temporal
      m.x[u] = __builtin_nontemporal_load((const u32x4_t*)(col + (size_t)m.src[u] * row_bytes));
  }
  if (m.acc_src != ra) m.acc = acc[m.acc_src];
}

__device__ __forceinline__ void compact_store(const MovePass& m, int r0, int rsub, char* col,
                                              int row_bytes, float* acc) {
#pragma unroll
  for (int u = 0; u < kCompactUnroll; ++u) {
    const int r = r0 + u * kPassRows + rsub;
    if (m.src[u] != r)  // non-temporal: the rows are next read by a streaming attention sweep
      __builtin_nontemporal_store(m.x[u], (u32x4_t*)(col + (size_t)r * row_bytes));
  }
  const int ra = r0 + (int)threadIdx.x;
  if (m.acc_src != ra) acc[ra] = m.acc;
}

// Passes of kRowsPerPass rows in ascending order. Pass p writes rows [r0, r0 + kRowsPerPass) and may
// read them as sources, so its loads must all complete before any of its stores (one barrier per
// pass); its sources are >= its rows, and the next pass's sources are >= the next pass's rows,
// which lie above every row pass p writes, so the next pass's loads are issued before pass p's
// stores.
__device__ __forceinline__ void compact_column(const CompactArgs& a, int l, int hkv, int col, int b,
                                               int nl) {
  const int tid = threadIdx.x;
  const int rsub = tid / kColLanes, piece = tid % kColLanes;
  const int ncol = a.row_bytes / kColBytes;
  const size_t bk = (size_t)b * a.Hkv + hkv;
  char* rows = (char*)(col < ncol ? a.layer[l].k : a.layer[l].v) + bk * a.cap * (size_t)a.row_bytes +
               (col % ncol) * kColBytes + 16 * piece;
  float* acc = col == 0 ? a.layer[l].acc + bk * a.cap : nullptr;
  const int32_t* kidx = a.keep_idx + (size_t)b * a.cap;
  MovePass cur, nxt;
  compact_load(cur, 0, rsub, nl, kidx, rows, a.row_bytes, acc);
  for (int r0 = 0; r0 < nl; r0 += kRowsPerPass) {
    __syncthreads();  // every thread holds this pass's rows
    const bool more = r0 + kRowsPerPass < nl;
    if (more) compact_load(nxt, r0 + kRowsPerPass, rsub, nl, kidx, rows, a.row_bytes, acc);
    compact_store(cur, r0, rsub, rows, a.row_bytes, acc);
    if (more) cur = nxt;
  }
}

// A fixed grid walks the (flagged sequence, kv head, column, layer) items, the layer fastest: the
// dispatcher deals consecutive workgroups round-robin to the 8 XCDs, so the rows of one flagged sequence
// spread over all of them. Most steps move nothing, and then the launch costs what its workgroups cost
// to start: 1024 (four a CU, as many as are resident) 1.9 us at 28 layers of the 7B shape, where a grid
// with the sequences in z, 4032 workgroups, took 6.0; one of 32 sequences flagged 34.7 us and 34.5, all
// 32 1.07 ms with both.
__global__ __launch_bounds__(kCompactThreads) void compact_kernel(CompactArgs a) {
  const int lane = threadIdx.x & 63;
  int b0 = 0, seen = 0;  // the chunk of 64 sequences at hand, flagged sequences before the bits of m
  int mine = lane < a.B ? a.new_len[lane] : 0;
  unsigned long long m = __ballot(mine > 0);
  if (m == 0 && a.B <= 64) return;  // before the division
  int rank = blockIdx.x / a.per_seq, rest = blockIdx.x % a.per_seq;  // the item: flagged sequence, and within
  for (;;) {
    while (m == 0 || seen < rank) {
      const int c = __popcll(m);
      if (m != 0 && seen + c > rank) {
        m &= m - 1;
        ++seen;
        continue;
      }
      seen += c;
      b0 += 64;
      if (b0 >= a.B) return;
      mine = b0 + lane < a.B ? a.new_len[b0 + lane] : 0;
      m = __ballot(mine > 0);
    }
    const int k = __builtin_ctzll(m);
    const int t = rest / a.n_layers;
    compact_column(a, rest % a.n_layers, t / a.n_col, t % a.n_col, b0 + k, __builtin_amdgcn_readlane(mine, k));
    __syncthreads();
    rank += a.step_rank;
    rest += a.step_rest;
    if (rest >= a.per_seq) {
      rest -= a.per_seq;
      ++rank;
    }
  }
}

hipError_t launch_h2o_scores(const KeepArgs& ka, int n_layers, const lg_layer_cache* layers,
                             hipStream_t st) {
  // H2O scores into keep_idx (as float bits), 64 layers per launch, added in layer order.
  for (int l0 = 0; l0 < n_layers; l0 += kMaxLayersPerLaunch) {
    ScoreArgs sa;
    sa.n_layers = min(kMaxLayersPerLaunch, n_layers - l0);
    for (int i = 0; i < sa.n_layers; ++i) sa.acc[i] = layers[l0 + i].acc;
    sa.first = l0 == 0;
    sa.B = ka.B;
    sa.Hkv = layers[0].n_kv_heads;
    sa.cap = ka.cap;
    sa.len = ka.len;
    sa.budget = ka.budget;
    sa.t_append = ka.t_append;
    sa.score = (float*)ka.keep_idx;
    hipLaunchKernelGGL(h2o_score_kernel, dim3((ka.cap + 255) / 256, ka.B), dim3(256), 0, st, sa);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_compact(const KeepArgs& ka, int n_layers, const lg_layer_cache* layers,
                          hipStream_t st) {
  if (n_layers == 0) return hipSuccess;
  const int Hkv = layers[0].n_kv_heads;
  const int row_bytes = layers[0].head_dim * (layers[0].dtype == LG_BF16 ? 2 : 4);
  for (int l0 = 0; l0 < n_layers; l0 += kMaxLayersPerLaunch) {
    const int nl = min(kMaxLayersPerLaunch, n_layers - l0);
    CompactArgs ca;
    for (int i = 0; i < nl; ++i) {
      ca.layer[i].k = layers[l0 + i].k;
      ca.layer[i].v = layers[l0 + i].v;
      ca.layer[i].acc = layers[l0 + i].acc;
    }
    ca.keep_idx = ka.keep_idx;
    ca.new_len = ka.new_len;
    ca.B = ka.B;
    ca.Hkv = Hkv;
    ca.cap = ka.cap;
    ca.row_bytes = row_bytes;
    ca.n_layers = nl;
    ca.n_col = 2 * row_bytes / kColBytes;
    ca.per_seq = nl * Hkv * ca.n_col;  // at most 64 x 65535 x 8
    const int grid = (int)std::min((long)ca.per_seq * ka.B, (long)kCompactWorkgroups);
    ca.step_rank = grid / ca.per_seq;
    ca.step_rest = grid % ca.per_seq;
    hipLaunchKernelGGL(compact_kernel, dim3(grid), dim3(kCompactThreads), 0, st, ca);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_prune(const lg_guard_params* p, int batch, int cap, int n_layers,
                        const lg_layer_cache* layers, int32_t* pos, int32_t* len,
                        const int32_t* budget, const int32_t* t_append,
                        const lg_decision* decision, int32_t* keep_idx, int32_t* new_len,
                        hipStream_t st) {
  const KeepArgs ka = keep_args(p, batch, cap, n_layers, pos, len, budget, t_append, decision,
                                keep_idx, new_len);
  hipError_t e = ka.have_scores ? launch_h2o_scores(ka, n_layers, layers, st) : hipSuccess;
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(keepset_kernel, dim3(batch), dim3(kKeepThreads), 0, st, ka);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_compact(ka, n_layers, layers, st);
}

}  // namespace lg
