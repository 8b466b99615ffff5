// Dynamic draft tree: top-k log-probabilities over the vocabulary, best-first level expansion,
// final selection.  Everything after the lm_head GEMM is small (a few KB to a few MB), so the
// kernels are written for few launches and short dependent chains, not for bandwidth:
//   topk_chunk_kernel   grid (64 chunks, M rows): the chunk's softmax statistics and its k largest
//                       logits (a thread owns ~10 logits in registers; k rounds of a per-wavefront
//                       argmax, then a merge of the four wavefronts' lists);
//   topk_merge_kernel   one wavefront per row: k rounds of a 64-lane argmax over the heads of the
//                       chunk lists; the k best are written in order with their log-softmax from
//                       the row's statistics;
//   tree_expand_kernel  one workgroup: appends the candidates of a level to the pool with their
//                       cumulative scores and ranks them for the next frontier;
//   tree_select_kernel  one wavefront: finds the score of the `total`-th best entry bit by bit, keeps
//                       what reaches it, renumbers in pool order (population counts of ballots);
//                       tree_select_small_kernel ranks pools of up to 128 entries by counting.
// "Better" is always: higher value, then lower index -- the order of the oracle.
#include "common.hpp"
#include "draft_tree.hpp"

namespace sparrow {

namespace {

constexpr int kTopkThreads = 256;
constexpr int kTopkMaxPerThread = 16;   // logits a thread may own: chunks of up to 4096 tokens

__device__ __forceinline__ bool better(float va, int ia, float vb, int ib) {
  return va > vb || (va == vb && ia < ib);
}

// Lowest index among the lanes that hold the maximum wv (0x7fffffff: none).  As a rule one lane does, and
// its index is read directly; ties take the minimum across the lanes.
__device__ __forceinline__ int winner_index(bool mine, int idx) {
  const unsigned long long who = __builtin_amdgcn_ballot_w64(mine);
  if (who == 0ull) return 0x7fffffff;
  if ((who & (who - 1ull)) == 0ull) return __builtin_amdgcn_readlane(idx, __builtin_ctzll(who));
  return wave_min_valu(mine ? idx : 0x7fffffff);
}

// One workgroup of 4 wavefronts per (chunk of the vocabulary, row); a thread owns up to 16 logits
// in registers (kTopkPerThread, by the vocabulary: a round's scan is most of its time, and a vocabulary
// of 16,384 needs one).  The chunk's softmax statistics (max and sum of exp2 in the log2 domain) come from
// the same registers.  Top k: every wavefront takes the k best of its own logits by k rounds of a
// 64-lane argmax on the vector ALU (value by maximum, then the lowest index among the lanes that
// hold it; no barrier, no LDS crossbar), then wavefront 0 merges the four sorted lists.
// Measured with k = 13: 1,481 tokens 17.4 -> 9.4 us, 59,077 tokens 16.9 -> 11.2 (k = 8, 152,064 tokens
// 9.2 -> 8.0) against one instance of 16 logits and a minimum across the lanes in every round.
template <int kTopkPerThread>
__global__ void __launch_bounds__(kTopkThreads)
topk_chunk_kernel(TopkArgs a) {
  constexpr int kWaves = kTopkThreads / 64;
  __shared__ float red[kWaves];
  __shared__ float lv[kWaves][kTreeMaxWidth];
  __shared__ int li[kWaves][kTreeMaxWidth];
  const int c = blockIdx.x, r = blockIdx.y;
  const int per = (a.V + kStatChunks - 1) / kStatChunks;
  const int v0 = min(a.V, c * per), v1 = min(a.V, v0 + per);
  const float *lg = a.logits + (int64_t)r * a.V;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  float val[kTopkPerThread];
#pragma unroll
  for (int j = 0; j < kTopkPerThread; ++j) {
    const int v = v0 + threadIdx.x + j * kTopkThreads;
    val[j] = v < v1 ? lg[v] : -INFINITY;
  }
  // ---- statistics of the chunk (temperature 1): m = max of l log2 e, s = sum of exp2(l log2 e - m)
  {
    constexpr float kLog2e = 1.4426950408889634f;
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < kTopkPerThread; ++j) m = fmaxf(m, val[j]);
    m = wave_max_valu(m);
    if (lane == 0) red[w] = m;
    __syncthreads();
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    const float ms = v1 > v0 ? m * kLog2e : kNegBig;       // an empty chunk: (kNegBig, 0)
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < kTopkPerThread; ++j) s += fast_exp2(fmaf(val[j], kLog2e, -ms));   // exp2(-inf) = 0
    s = wave_sum_valu(s);
    if (lane == 0) red[w] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
      float *o = a.stats + ((int64_t)r * kStatChunks + c) * 2;
      o[0] = ms;
      o[1] = v1 > v0 ? red[0] + red[1] + red[2] + red[3] : 0.f;
    }
  }
  // ---- the wavefront's k best, in decreasing order (ties: lower index first)
  for (int round = 0; round < a.k; ++round) {
    float bv = -INFINITY;
    int bj = 0;
#pragma unroll
    for (int j = 0; j < kTopkPerThread; ++j)
      if (val[j] > bv) { bv = val[j]; bj = j; }             // ascending index: the lowest wins a tie
    const float wv = wave_max_valu(bv);
    const int bi = v0 + (int)threadIdx.x + bj * kTopkThreads;
    const int wi = winner_index(bv == wv && bv > -INFINITY, bi);
    // the winner leaves its owner's registers (an exhausted wavefront yields -inf / 0x7fffffff)
#pragma unroll
    for (int j = 0; j < kTopkPerThread; ++j)
      if (j == bj && bi == wi) val[j] = -INFINITY;
    if (lane == 0) { lv[w][round] = wi == 0x7fffffff ? -INFINITY : wv; li[w][round] = wi; }
  }
  __syncthreads();
  // ---- merge of the four lists: lane l < 4 walks list l, every round the best head wins
  if (w == 0) {
    int pos = 0;
    float hv = lane < kWaves ? lv[lane][0] : -INFINITY;
    int hi = lane < kWaves ? li[lane][0] : 0x7fffffff;
    for (int round = 0; round < a.k; ++round) {
      const float wv = wave_max_valu(hv);
      const int wi = winner_index(hv == wv && hi != 0x7fffffff, hi);
      if (lane == 0) {
        const int64_t o = ((int64_t)r * kStatChunks + c) * a.k + round;
        a.cand_val[o] = wi == 0x7fffffff ? -INFINITY : wv;
        a.cand_idx[o] = wi;
      }
      if (hi == wi && wi != 0x7fffffff) {                   // the owner of the winner moves on
        ++pos;
        hv = pos < a.k ? lv[lane][pos] : -INFINITY;
        hi = pos < a.k ? li[lane][pos] : 0x7fffffff;
      }
    }
  }
}

__global__ void __launch_bounds__(64)
topk_merge_kernel(TopkArgs a) {
  // one wavefront per row: lane c walks chunk c's list (already in decreasing order); every round
  // the best list head of the 64 lanes is the row's next token
  const int r = blockIdx.x, lane = threadIdx.x;
  const float pm = a.stats[((int64_t)r * kStatChunks + lane) * 2];
  const float ps = a.stats[((int64_t)r * kStatChunks + lane) * 2 + 1];
  // the lane's whole list goes to LDS first (all loads in flight at once: one round trip); the
  // walk then costs an LDS read per round instead of a dependent global load
  __shared__ float sv[kTreeMaxWidth][64];
  __shared__ int si[kTreeMaxWidth][64];
  const float *cv = a.cand_val + ((int64_t)r * kStatChunks + lane) * a.k;
  const int32_t *ci = a.cand_idx + ((int64_t)r * kStatChunks + lane) * a.k;
#pragma unroll
  for (int j = 0; j < kTreeMaxWidth; ++j) {
    sv[j][lane] = j < a.k ? cv[j] : -INFINITY;
    si[j][lane] = j < a.k ? ci[j] : 0x7fffffff;
  }
  const float m = wave_max_valu(pm);
  const float Z = wave_sum_valu(ps * fast_exp2(pm - m));
  const float lse = (m + fast_log2(Z)) * kLn2;       // m is in the log2 domain (l log2 e)
  int pos = 0;
  float hv = sv[0][lane];                            // (a lane reads only what it wrote itself)
  int hi = si[0][lane];
  for (int round = 0; round < a.k; ++round) {
    const float wv = wave_max_valu(hv);
    const int wi = winner_index(hv == wv && hi != 0x7fffffff, hi);
    if (wi == 0x7fffffff) break;                     // every list exhausted (uniform)
    if (lane == 0) {
      a.ids[(int64_t)r * a.k + round] = wi;
      a.logp[(int64_t)r * a.k + round] = wv - lse;
    }
    if (hi == wi) {                                  // the owner of the winner moves on
      ++pos;
      hv = pos < a.k ? sv[pos][lane] : -INFINITY;
      hi = pos < a.k ? si[pos][lane] : 0x7fffffff;
    }
  }
}

__global__ void __launch_bounds__(256)
tree_expand_kernel(ExpandArgs a) {
  __shared__ float sc[kTreeMaxWidth * kTreeMaxWidth];
  const int tid = threadIdx.x;
  const int n_new = a.n_front * a.width;
  if (tid < n_new) {
    const int f = tid / a.width;
    const int p = a.front_in ? a.front_in[f] : -1;
    const float s = (p >= 0 ? a.pool_score[p] : 0.f) + a.cand_logp[tid];
    a.pool_tok[a.n_pool + tid] = a.cand_ids[tid];
    a.pool_par[a.n_pool + tid] = p;
    a.pool_score[a.n_pool + tid] = s;
    sc[tid] = s;
  }
  __syncthreads();
  if (tid < n_new) {
    const float s = sc[tid];
    int rank = 0;
    for (int j = 0; j < n_new; ++j) rank += better(sc[j], j, s, tid) ? 1 : 0;
    if (rank < a.width) a.front_out[rank] = a.n_pool + tid;
  }
}

// Order-preserving integer key of a score (+ 0: the two zeros are one score).
__device__ __forceinline__ unsigned int score_key(float score) {
  const unsigned int u = __float_as_uint(score + 0.0f);
  return (u & 0x80000000u) ? ~u : u | 0x80000000u;
}

// Pools of up to 128 entries, two per lane: every entry's rank is counted, the others' keys read across the
// lanes; a kept entry's new number and its parent's are population counts of the ballots of kept ones.  One
// memory round trip, no LDS: 72 entries 3.8 us, against 5.7 to 7.1 with the kernel for larger pools and 5.1
// with a workgroup that ranked by counting (8 entries 2.0, 3.7 to 5.0 and 2.9).
constexpr int kSelectSmall = 128;
__global__ void __launch_bounds__(64)
tree_select_small_kernel(SelectArgs a) {
  const int lane = threadIdx.x, n = a.n_pool, keep = min(a.total, n);
  unsigned int key[2];
  unsigned long long order[2];          // key, then the lower index: no two entries are equal
  int par[2], tok[2], rank[2] = {0, 0};
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int i = 64 * u + lane;
    key[u] = i < n ? score_key(a.pool_score[i]) : 0u;
    order[u] = (unsigned long long)key[u] << 32 | (0xffffffffu - (unsigned int)i);
    par[u] = i < n ? a.pool_par[i] : -1;
    tok[u] = i < n ? a.pool_tok[i] : 0;
  }
#pragma unroll
  for (int v = 0; v < 2; ++v)
    for (int j0 = 0; j0 < min(n - 64 * v, 64); j0 += 8)   // (entries past the pool rank behind all others)
#pragma unroll
      for (int j = j0; j < j0 + 8; ++j) {
        const unsigned int kj = (unsigned int)__builtin_amdgcn_readlane((int)key[v], j);
        const unsigned long long oj = (unsigned long long)kj << 32 | (0xffffffffu - (unsigned int)(64 * v + j));
#pragma unroll
        for (int u = 0; u < 2; ++u) rank[u] += oj > order[u] ? 1 : 0;
      }
  unsigned long long kept[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) kept[u] = __builtin_amdgcn_ballot_w64(64 * u + lane < n && rank[u] < keep);
  auto new_id = [&](int i) {            // -1: not kept
    const unsigned long long m = kept[i >> 6], bit = 1ull << (i & 63);
    return (m & bit) == 0ull ? -1 : (i >= 64 ? __popcll(kept[0]) : 0) + __popcll(m & (bit - 1ull));
  };
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int i = 64 * u + lane;
    if (i >= n) continue;
    const int id = new_id(i);
    if (id < 0) continue;
    a.parent[id] = (par[u] >= 0 && par[u] < n) ? new_id(par[u]) : -1;
    a.ids[id] = tok[u];
    a.pool_index[id] = i;
  }
}

// Larger pools.  Entry 64 r + l of the pool sits in register r of lane l.  The score of the keep-th best is
// found bit by bit on order-preserving integer keys (the number of entries that reach a candidate: one ballot
// per register); entries above it are kept, and of those equal to it the first in pool order.  No barrier and
// no rank counting: 200 entries 8 us, 689 entries 9.4 to 12, against 9.5 and 30 for a workgroup that ranked by
// counting.  With four registers for up to 256 entries, without a test for each of 32, 200 entries
// take 5.8 in a trace (32 registers 11.5).
template <int kRegs>
__global__ void __launch_bounds__(64)
tree_select_kernel(SelectArgs a) {
  __shared__ int new_id[64 * kRegs];
  const int lane = threadIdx.x;
  const int n = a.n_pool, keep = min(a.total, n), regs = kRegs <= 4 ? kRegs : (n + 63) / 64;
  unsigned int key[kRegs];                // 0 for lanes past the pool: below every score's key
#pragma unroll
  for (int r = 0; r < kRegs; ++r) {
    key[r] = 0u;
    if (r < regs && 64 * r + lane < n) key[r] = score_key(a.pool_score[64 * r + lane]);
  }
  auto reach = [&](unsigned int t) {
    int cnt = 0;
#pragma unroll
    for (int r = 0; r < kRegs; ++r)
      if (r < regs) cnt += __popcll(__builtin_amdgcn_ballot_w64(key[r] >= t));
    return cnt;
  };
  unsigned int thr = 0u;                  // the largest value that at least `keep` keys reach
  for (int bit = 31; bit >= 0; --bit) {
    const unsigned int t = thr | (1u << bit);
    const int cnt = reach(t);
    if (cnt >= keep) thr = t;
    if (cnt == keep) break;               // exactly the kept ones reach it
  }
  int above = 0;                          // strictly better entries
#pragma unroll
  for (int r = 0; r < kRegs; ++r)
    if (r < regs) above += __popcll(__builtin_amdgcn_ballot_w64(key[r] > thr));
  const unsigned long long below = (1ull << lane) - 1ull;
  int eq = 0, pos = 0;                    // equal entries / kept entries in the registers before r
#pragma unroll
  for (int r = 0; r < kRegs; ++r) {
    if (r < regs) {
      const bool in = 64 * r + lane < n;
      const unsigned long long eq_m = __builtin_amdgcn_ballot_w64(in && key[r] == thr);
      const bool kept = in && (key[r] > thr || (key[r] == thr && above + eq + __popcll(eq_m & below) < keep));
      const unsigned long long kept_m = __builtin_amdgcn_ballot_w64(kept);
      if (in) new_id[64 * r + lane] = kept ? pos + __popcll(kept_m & below) : -1;
      eq += __popcll(eq_m);
      pos += __popcll(kept_m);
    }
  }
  __syncthreads();
  for (int i = lane; i < n; i += 64) {
    const int id = new_id[i];
    if (id < 0) continue;
    const int p = a.pool_par[i];
    a.parent[id] = (p >= 0 && p < n) ? new_id[p] : -1;
    a.ids[id] = a.pool_tok[i];
    a.pool_index[id] = i;
  }
}

}  // namespace

hipError_t launch_topk(const TopkArgs &a, hipStream_t st) {
  const int per = (a.V + kStatChunks - 1) / kStatChunks;
  const dim3 grid(kStatChunks, a.M);
  if (per <= 1 * kTopkThreads) hipLaunchKernelGGL(topk_chunk_kernel<1>, grid, dim3(kTopkThreads), 0, st, a);
  else if (per <= 4 * kTopkThreads) hipLaunchKernelGGL(topk_chunk_kernel<4>, grid, dim3(kTopkThreads), 0, st, a);
  else if (per <= 10 * kTopkThreads) hipLaunchKernelGGL(topk_chunk_kernel<10>, grid, dim3(kTopkThreads), 0, st, a);
  else hipLaunchKernelGGL(topk_chunk_kernel<kTopkMaxPerThread>, grid, dim3(kTopkThreads), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(topk_merge_kernel, dim3(a.M), dim3(64), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_tree_expand(const ExpandArgs &a, hipStream_t st) {
  hipLaunchKernelGGL(tree_expand_kernel, dim3(1), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_tree_select(const SelectArgs &a, hipStream_t st) {
  if (a.n_pool <= kSelectSmall) hipLaunchKernelGGL(tree_select_small_kernel, dim3(1), dim3(64), 0, st, a);
  else if (a.n_pool <= 256) hipLaunchKernelGGL(tree_select_kernel<4>, dim3(1), dim3(64), 0, st, a);
  else hipLaunchKernelGGL(tree_select_kernel<kTreeMaxPool / 64>, dim3(1), dim3(64), 0, st, a);
  return hipGetLastError();
}

}  // namespace sparrow
