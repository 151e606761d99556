// lg_keepset.h -- the keep set of Stage 2 (Sec. 5.3, Eq. (10) and Eq. (11)) as a workgroup-level
// device routine, shared by the prune launch (keepset_kernel) and the fused detector launch
// (lg_detect.hip). See the file comment of lg_prune.hip for the algorithm.
#pragma once

#include "lg_internal.h"

namespace lg {

constexpr int kKeepThreads = 512;    // keepset_kernel

struct KeepArgs {
  int32_t n_anchor, recent_div, sparse_div, policy, have_scores;
  int32_t B, cap;
  int32_t* pos;
  int32_t* len;
  const int32_t* budget;
  const int32_t* t_append;
  const lg_decision* decision;
  int32_t* keep_idx;
  int32_t* new_len;
};

inline KeepArgs keep_args(const lg_guard_params* p, int batch, int cap, int n_layers,
                          int32_t* pos, int32_t* len, const int32_t* budget,
                          const int32_t* t_append, const lg_decision* decision,
                          int32_t* keep_idx, int32_t* new_len) {
  KeepArgs ka;
  ka.n_anchor = p->n_anchor;
  ka.recent_div = p->recent_div;
  ka.sparse_div = p->sparse_div;
  ka.policy = p->policy;
  ka.have_scores = (p->policy == LG_POLICY_H2O && n_layers > 0) ? 1 : 0;
  ka.B = batch;
  ka.cap = cap;
  ka.pos = pos;
  ka.len = len;
  ka.budget = budget;
  ka.t_append = t_append;
  ka.decision = decision;
  ka.keep_idx = keep_idx;
  ka.new_len = new_len;
  return ka;
}

// Exclusive prefix sum over the TPB lanes of the workgroup; *total gets the sum.
template <int TPB>
__device__ __forceinline__ int block_exclusive_scan(int x, int* total, int* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  __syncthreads();
  if (lane == 63) red[wave] = inc;
  __syncthreads();
  int before = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < TPB / 64; ++w) {
    if (w < wave) before += red[w];
    tot += red[w];
  }
  *total = tot;
  return before + inc - x;
}

// Elements of the ascending array x[0, n) below thr, found by one wave: 64 probes a round, each at
// the end of one of 64 equal segments, so 65536 positions take three dependent loads where a scan of
// them by the workgroup took 256 rounds. An array that is not ascending gives some value in [0, n].
__device__ __forceinline__ int wave_lower_bound(const int32_t* x, int n, int thr) {
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = n;
  while (lo < hi) {
    const int step = (hi - lo + 63) >> 6;
    const long long first = (long long)lo + (long long)lane * step;  // the lane's segment
    const bool below = first < hi && x[min((int)first + step - 1, hi - 1)] < thr;
    const int cnt = __popcll(__ballot(below));
    const int seg = (int)min((long long)lo + (long long)cnt * step, (long long)hi);
    hi = step == 1 ? seg : (int)min((long long)seg + step, (long long)hi);
    lo = seg;
    if (step == 1) break;
  }
  return lo;
}

// Keys of the H2O order: the score as an order-preserving unsigned integer (float order, -0 below
// +0) above the slot index, so equal scores rank the later slot (higher position) first.
__device__ __forceinline__ unsigned long long h2o_key(const int32_t* scores, int j, bool have) {
  uint32_t u = have ? (uint32_t)scores[j] : 0u;
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((unsigned long long)u << 32) | (uint32_t)j;
}

// What the keep set of a sequence needs from memory, requested before anything waits for it (the
// fused launch does so before the detector's work).
struct KeepInputs {
  int len, budget, t_append, appended;  // len: live slots before the commit, clamped into the cache
};
__device__ __forceinline__ KeepInputs load_keep_inputs(const KeepArgs& a, int b) {
  KeepInputs x;
  x.len = a.len[b];
  x.budget = min(a.budget[b], a.cap);  // a budget above the cache's capacity acts as the capacity
  x.t_append = a.t_append != nullptr ? a.t_append[b] : 0;
  x.len = x.len < 0 ? 0 : (x.len > a.cap ? a.cap : x.len);
  x.appended = a.t_append != nullptr && x.len < a.cap;
  return x;
}

// The need-th largest key among slots [0, n) (1 <= need <= n): 8-bit digits from the top, one
// histogram pass per digit over the keys that match the digits found so far; the digit holding
// the need-th largest is found with a block scan over the bins from the top.
template <int TPB>
__device__ unsigned long long radix_select_desc(const int32_t* scores, bool have, int n, int need,
                                                unsigned int* hist, unsigned long long* s_prefix,
                                                int* s_need, int* red) {
  static_assert(TPB >= 256, "one thread per 8-bit bin");
  const int tid = threadIdx.x;
  unsigned long long prefix = 0;
  for (int shift = 56; shift >= 0; shift -= 8) {
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    for (int j = tid; j < n; j += TPB) {
      const unsigned long long key = h2o_key(scores, j, have);
      if (shift == 56 || (key >> (shift + 8)) == (prefix >> (shift + 8)))
        atomicAdd(&hist[(key >> shift) & 255u], 1u);
    }
    __syncthreads();
    const int d = 255 - tid;  // thread tid < 256 looks at digit d, larger digits first
    const int cnt = tid < 256 ? (int)hist[d] : 0;
    int tot;
    const int above = block_exclusive_scan<TPB>(cnt, &tot, red);  // keys with a larger digit
    if (tid < 256 && above < need && above + cnt >= need) {
      *s_need = need - above;
      *s_prefix = prefix | ((unsigned long long)d << shift);
    }
    __syncthreads();
    prefix = *s_prefix;
    need = *s_need;
    __syncthreads();
  }
  return prefix;
}

// The keep set of sequence blockIdx.x (see the file comment of lg_prune.hip), by the TPB
// threads of the workgroup. trig, span and level are the sequence's decision (uniform).
//
// Positions ascend over the slots, so the anchors, the middle and the recent window are ranges of
// slots, and LoopGuard's and StreamingLLM's keep sets are known once the ranges' ends are: kept
// entry r is a slot in closed form. Three waves find the ends (wave_lower_bound), and every entry is
// then written independently. Before, the workgroup classified and scanned the slots 256 at a time:
// 64 contexts of up to 65536 tokens 416 us, a 2048-slot cache 15.7 us (MI355X).
template <int TPB>
__device__ void keep_set_block(const KeepArgs& a, const KeepInputs& in, bool trig, int span,
                               int level) {
  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  __shared__ int red[TPB / 64];
  int32_t* pos = a.pos + (size_t)b * a.cap;
  int32_t* kidx = a.keep_idx + (size_t)b * a.cap;
  const int Ls = in.len, L = Ls + in.appended;  // stored slots; live slots after the commit
  const int budget = in.budget;
  const bool flag = trig || L >= budget;
  if (tid == 0) {
    if (in.appended) pos[Ls] = in.t_append;
    if (!flag) {
      if (a.t_append != nullptr) a.len[b] = L;
      a.new_len[b] = -1;
    }
  }
  if (!flag) return;
  if (!trig) span = -1;
  level = trig ? min(max(level, 0), 30) : 0;
  const int t = in.appended ? in.t_append : (L > 0 ? pos[L - 1] : 0);
  const int R = budget / a.recent_div;
  const int thrR = sat_sub(sat_sub(t, R), -1);  // t - R + 1
  // The kept set leaves room for the next append: at most budget - 1 slots (LoopGuard: claimed by
  // the anchors first, then the recent window, then the sparse history; the baselines: their keep
  // size capped). With the paper's constants nothing is cut.
  const int cap_k = max(0, budget - 1);
  const int Ktot = min(budget / a.sparse_div + budget / a.recent_div, cap_k);  // baselines
  int kept;
  if (a.policy == LG_POLICY_H2O) {
    // Slots [0, older) are ranked by score, the later ones kept.
    const bool have = a.have_scores != 0;
    const int Rp = max(0, min(min(R, L), Ktot));
    const int older = L - Rp;
    const int heavy = max(0, Ktot - Rp);
    const bool keep_all_older = older <= heavy;
    __shared__ unsigned int hist[256];
    __shared__ unsigned long long s_prefix;
    __shared__ int s_need;
    unsigned long long thr_key = ~0ull;  // keeps none of the older slots
    // Without scores the order is the slots': the latest heavy ones stay.
    if (!keep_all_older && heavy > 0)
      thr_key = have ? radix_select_desc<TPB>(kidx, have, older, heavy, hist, &s_prefix, &s_need, red)
                     : h2o_key(kidx, older - heavy, have);
    kept = 0;
    for (int j0 = 0; j0 < L; j0 += TPB) {
      const int j = j0 + tid;
      const bool keep = j < L && (j >= older || keep_all_older || h2o_key(kidx, j, have) >= thr_key);
      int ktot;
      const int slot = kept + block_exclusive_scan<TPB>(keep ? 1 : 0, &ktot, red);
      if (keep) kidx[slot] = j;
      kept += ktot;
    }
    __syncthreads();
    // Gather pos in place (ascending chunks, read all before writing).
    for (int r0 = 0; r0 < kept; r0 += TPB) {
      const int r = r0 + tid;
      int v = 0;
      if (r < kept) {
        const int j = kidx[r];
        v = in.appended && j == Ls ? in.t_append : pos[j];
      }
      __syncthreads();
      if (r < kept) pos[r] = v;
    }
  } else {
    // Ends of the ranges among the stored slots, then with the appended one.
    __shared__ int s_end[3];
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave < 3) {
      const int thr = wave == 0 ? a.n_anchor : wave == 1 ? thrR : span;
      const int e = wave_lower_bound(pos, Ls, thr) + (in.appended && in.t_append < thr ? 1 : 0);
      if ((tid & 63) == 0) s_end[wave] = e;
    }
    __syncthreads();
    const int NA = s_end[0];
    // Kept: slots [0, n_a), n_s of the M slots from NA, and n_r slots from r_lo.
    int n_a, n_s = 0, M = 0, S = 0, n_r, r_lo;
    if (a.policy == LG_POLICY_STREAMING) {
      n_a = min(NA, max(Ktot, 0));
      r_lo = max(n_a, L - max(0, Ktot - n_a));
      n_r = L - r_lo;
    } else {
      const int jR = max(NA, s_end[1]);                    // middle: [NA, jR)
      const int jB = span >= 0 ? max(jR, s_end[2]) : L;    // clean recent window: [jR, jB)
      M = jR - NA;
      n_a = min(NA, cap_k);
      const int Br = min(R >> level, cap_k - n_a);
      S = max(0, min(budget / a.sparse_div - a.n_anchor, cap_k - n_a - Br));
      n_s = min(M, S);
      n_r = max(0, min(Br, jB - jR));
      r_lo = jB - n_r;
    }
    kept = n_a + n_s + n_r;
    // Entry r of the keep list, and pos gathered in place: entries ascend and slot(r) >= r, so a
    // chunk's writes lie below every slot a later chunk reads; a chunk is read before it is written.
    constexpr int U = 8;
    for (int r0 = 0; r0 < kept; r0 += TPB * U) {
      int j[U], v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = r0 + u * TPB + tid;
        const int k = r - n_a;
        int x = r;
        if (k >= 0 && k < n_s && M > n_s)
          x = NA + (((long long)k * M) >> 32 ? (int)((long long)k * M / S)
                                             : (int)((unsigned)k * (unsigned)M / (unsigned)S));
        else if (k >= 0 && k < n_s) x = NA + k;
        else if (k >= n_s) x = r_lo + (k - n_s);
        j[u] = x;
        v[u] = 0;
        if (r < kept) v[u] = in.appended && x == Ls ? in.t_append : pos[x];
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = r0 + u * TPB + tid;
        if (r < kept) {
          kidx[r] = j[u];
          pos[r] = v[u];
        }
      }
    }
  }
  if (tid == 0) {
    a.new_len[b] = kept;
    a.len[b] = kept;
  }
}

// Host side of a prune, around the keep set (lg_prune.hip): the H2O scores it ranks (baseline
// policy H2O) and the compaction of every layer's rows by the kept list.
hipError_t launch_h2o_scores(const KeepArgs& ka, int n_layers, const lg_layer_cache* layers,
                             hipStream_t st);
hipError_t launch_compact(const KeepArgs& ka, int n_layers, const lg_layer_cache* layers,
                          hipStream_t st);

}  // namespace lg
