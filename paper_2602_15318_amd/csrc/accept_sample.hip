// Stochastic (temperature > 0) tree acceptance on the logits stored by the lm_head pass.
//
//   logit_stats_kernel   the whole chip reads the M x V logits once (64 chunks per row): per
//                        chunk the max and the sum of exponentials of logits / T, and per block of
//                        256 tokens the sum of exponentials relative to the chunk's max;
//   accept_sample_kernel one workgroup per sequence: merges the 64 chunk statistics of all its rows and fetches what
//                        decides every node at once, lets one wavefront apply the sequential rejection rule down the
//                        tree (u * S <= p[x] accepts; a rejected token is struck out and its mass leaves S), and
//                        draws the bonus token from what is left at the last node by inverse CDF in vocabulary order:
//                        a scan over the row's block sums (struck-out tokens taken out), then a search inside the
//                        one block that holds the target -- the only 256 logits of the row it reads;
//   accept_sample_q_kernel, residual_sums_kernel   the same against a sampled draft, see below.
// Exponentials are exp2 of logits pre-multiplied by log2(e) / T in fp32; sums across blocks fp64.
#include "accept.hpp"
#include "common.hpp"

namespace sparrow {

namespace {

constexpr int kStatThreads = 256;
constexpr int kWalkThreads = 1024;
constexpr int kBonusBlock = 256;              // tokens per block of the bonus draw
constexpr int kBonusMaxBlocks = kSampleMaxVocab / kBonusBlock;

// Philox4x32 with 10 rounds (Salmon et al., SC'11): round (c0, c1, c2, c3), key (k0, k1) ->
// (hi(M1 c2) ^ c1 ^ k0, lo(M1 c2), hi(M0 c0) ^ c3 ^ k1, lo(M0 c0)); the key grows by the Weyl
// constants after every round.  Only the first output word is used here.
__device__ __forceinline__ unsigned int philox4x32_10_word0(unsigned int c0, unsigned int c1,
                                                            unsigned int c2, unsigned int c3,
                                                            unsigned int k0, unsigned int k1) {
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    const unsigned int h0 = __umulhi(0xD2511F53u, c0), l0 = 0xD2511F53u * c0;
    const unsigned int h1 = __umulhi(0xCD9E8D57u, c2), l1 = 0xCD9E8D57u * c2;
    const unsigned int n0 = h1 ^ c1 ^ k0, n2 = h0 ^ c3 ^ k1;
    c0 = n0; c1 = l1; c2 = n2; c3 = l0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c0;
}
// The uniform that decides node j of sequence b (j = -1: the bonus draw): the caller's, or the
// top 24 bits of the Philox block (offset, b, j) under the key `seed`, times 2^-24.
__device__ __forceinline__ float uniform_of(const SampleArgs &a, int b, int j) {
  if (j >= 0 && a.u_accept != nullptr) return a.u_accept[(int64_t)b * a.n_q + j];
  if (j < 0 && a.u_bonus != nullptr) return a.u_bonus[b];
  const unsigned int w = philox4x32_10_word0((unsigned int)a.offset, (unsigned int)(a.offset >> 32),
                                             (unsigned int)b, j >= 0 ? (unsigned int)j : 0xFFFFFFFFu,
                                             (unsigned int)a.seed, (unsigned int)(a.seed >> 32));
  return (float)(w >> 8) * (1.0f / 16777216.0f);
}

// A chunk's blocks of 256 tokens are dealt to kWaves wavefronts, 1 or 4, a lane owns four consecutive tokens of each: the
// chunk is read once, 16 bytes per lane, all loads in flight together, and stays in registers for the maximum and for
// the sums.  One wavefront exchanges nothing through LDS, and the wavefronts of a workgroup serve four chunks.  Four / one
// wavefront, us: 315 rows of 6,828 31.0 / 9.9 (a chunk is one block at most, three wavefronts in four had none), 156 of
// 16,724 18.2 / 7.4, 180 of 152,064 31.7 / 23.5, 36 of 64,003 7.9 / 5.0, 30 of 56,772 5.6 / 4.5; with long chunks of few
// rows the chip is short of wavefronts: 24 of 152,064 6.9 / 7.4, 16 of 122,762 5.7 / 6.1.
constexpr int kStatAhead = 16;
constexpr int kStatWaves = kStatThreads / 64;
typedef f32x4 __attribute__((aligned(4))) f32x4u;       // rows of odd vocabularies start at any multiple of 4 bytes

int stat_blocks_per_chunk(int V) {
  const int n_blk = (V + kBonusBlock - 1) / kBonusBlock;
  return (n_blk + kStatChunks - 1) / kStatChunks;
}

template <int kWaves>
__global__ void __launch_bounds__(kStatThreads)
logit_stats_kernel(SampleArgs a) {
  __shared__ float red[kStatWaves];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = kWaves == 1 ? 0 : wave;                             // wavefront within the chunk
  const int c = kWaves == 1 ? blockIdx.x * kStatWaves + wave : blockIdx.x, r = blockIdx.y;
  const int n_blk = (a.V + kBonusBlock - 1) / kBonusBlock;
  const int bpc = (n_blk + kStatChunks - 1) / kStatChunks;          // blocks per chunk
  const int b0 = min(n_blk, c * bpc), b1 = min(n_blk, b0 + bpc);
  const float *lg = a.logits + (int64_t)r * a.V;
  // scaled logits of this lane: x[k][i] = token (b0 + w + kWaves k) * 256 + 4 lane + i, kNegBig past V
  float x[kStatAhead][4];
#pragma unroll
  for (int k = 0; k < kStatAhead; ++k) {
    const int ib = b0 + w + kWaves * k;
    const int v = ib * kBonusBlock + 4 * lane;
#pragma unroll
    for (int i = 0; i < 4; ++i) x[k][i] = kNegBig;
    if (ib < b1) {
      if (v + 3 < a.V) {
        const f32x4 q = *reinterpret_cast<const f32x4u *>(lg + v);
#pragma unroll
        for (int i = 0; i < 4; ++i) x[k][i] = q[i] * a.inv_temp_log2;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (v + i < a.V) x[k][i] = lg[v + i] * a.inv_temp_log2;
      }
    }
  }
  float m = kNegBig;
#pragma unroll
  for (int k = 0; k < kStatAhead; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) m = fmaxf(m, x[k][i]);
  m = wave_max_valu(m);
  if constexpr (kWaves > 1) {
    if (lane == 0) red[w] = m;
    __syncthreads();
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
  }
  // block sums relative to the chunk's max; four running sums whatever the number of wavefronts
  constexpr int kSums = kStatWaves / kWaves;
  float s[kSums];
#pragma unroll
  for (int k = 0; k < kSums; ++k) s[k] = 0.f;
#pragma unroll
  for (int k = 0; k < kStatAhead; ++k) {
    const int ib = b0 + w + kWaves * k;
    if (ib < b1) {                              // uniform over the wavefront
      const int v = ib * kBonusBlock + 4 * lane;
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (v + i < a.V) t += fast_exp2(x[k][i] - m);
      t = wave_sum_valu(t);
      if (lane == 0) a.blk_sum[(int64_t)r * n_blk + ib] = t;
      s[k % kSums] += t;                        // the same value in every lane
    }
  }
  float *o = a.stats + ((int64_t)r * kStatChunks + c) * 2;         // kNegBig and sum 0 for an empty chunk
  if constexpr (kWaves == 1) {
    if (lane == 0) { o[0] = m; o[1] = s[0] + s[1] + s[2] + s[3]; }
  } else {
    if (lane == 0) red[w] = s[0];
    __syncthreads();
    if (threadIdx.x == 0) { o[0] = m; o[1] = red[0] + red[1] + red[2] + red[3]; }
  }
}

// Maximum and sum of exponentials of every row of a sequence from the rows' 64 chunk statistics: wavefront w of the
// workgroup takes rows w, w + 16, ..., all loads in flight together.
__device__ __forceinline__ void row_statistics(const SampleArgs &a, int64_t row0, float *row_m, float *row_z) {
  constexpr int kWaves = kWalkThreads / 64, kRows = (SPARROW_MAX_NQ + 1 + kWaves - 1) / kWaves;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const float2 *st = reinterpret_cast<const float2 *>(a.stats) + row0 * kStatChunks + lane;
  float2 ps[kRows];
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    ps[u] = make_float2(kNegBig, 0.f);
    if (w + kWaves * u <= a.n_q) ps[u] = st[(w + kWaves * u) * kStatChunks];
  }
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    if (w + kWaves * u > a.n_q) break;                       // uniform over the wavefront
    const float m = wave_max_valu(ps[u].x);
    const float Z = wave_sum_valu(ps[u].y * fast_exp2(ps[u].x - m));
    if (lane == 0) { row_m[w + kWaves * u] = m; row_z[w + kWaves * u] = Z; }
  }
}

// What decides whether a node is accepted, fetched for all nodes at once, lane j of a wavefront for node j (n_q <= 64):
// the walk then reads registers, where fetched level by level every level paid two memory round trips.  Walk and draw of
// deterministic children level by level / at once, us: 6 chains of 4 over 56,772 14.8 / 5.6, 6 trees of 29 over 152,064
// 20.5 / 8.2.  parent = -2: not a node, or its token or parent is out of range (never accepted).
struct Node {
  int parent, token;
  float logit, q, u;                            // of its token in the parent's row; the uniform that decides it
};
__device__ __forceinline__ Node fetch_node(const SampleArgs &a, int b, int64_t row0, int j) {
  Node nd = {-2, -1, 0.f, 0.f, 0.f};
  if (j < a.n_q) {
    const int p = a.parent ? a.parent[(int64_t)b * a.parent_stride + j] : j - 1;
    nd.token = a.draft_ids[(int64_t)b * a.n_q + j];
    if (p >= -1 && p < a.n_q && nd.token >= 0 && nd.token < a.V) {
      nd.parent = p;
      nd.logit = a.logits[(row0 + p + 1) * a.V + nd.token];
      if (a.draft_q != nullptr) nd.q = a.draft_q[(row0 + p + 1) * a.V + nd.token];
    }
    nd.u = uniform_of(a, b, j);
  }
  return nd;
}
__device__ __forceinline__ float lane_f32(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// The bonus draw's scan, by one wavefront: the block of 256 tokens in which the running sum reaches the target, and the
// sum of the blocks before it.  Lane l owns n_blk / 64 consecutive blocks; nothing waits for another wavefront (with
// the scan spread over the workgroup's 16, six barriers took as long as the rest of the kernel).
// target_of: the target from the sum of all blocks.  block = -1: no live block.
struct Drawn {
  int block;
  double before, target;
};
template <class F> __device__ __forceinline__ Drawn find_block(const double *blk_tot, int n_blk, F target_of) {
  const int lane = threadIdx.x & 63;
  const int per = (n_blk + 63) / 64, i0 = min(n_blk, lane * per), i1 = min(n_blk, i0 + per);
  double local = 0.0;
  int last = -1;                                             // last live block of the lane
  for (int i = i0; i < i1; ++i) {
    const double t = blk_tot[i];
    local += t;
    if (t > 0.0) last = i;
  }
  double incl = local;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  Drawn d;
  d.target = target_of(__shfl(incl, 63, 64));
  const unsigned long long hit = __builtin_amdgcn_ballot_w64(local > 0.0 && incl >= d.target);
  if (hit == 0ull) {               // rounding left the total a hair below the target: the row's last live block, with
    d.block = last;                // nothing to find in it
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) d.block = max(d.block, __shfl_xor(d.block, o, 64));
    d.before = -1.0e300;
    return d;
  }
  double run = incl - local;
  int blk = -1;
  for (int i = i0; i < i1 && blk < 0; ++i) {
    const double t = blk_tot[i];
    if (t > 0.0) {
      if (run + t >= d.target) blk = i; else run += t;
    }
  }
  if (blk < 0) { blk = last; run = -1.0e300; }               // rounding between the two orders of summation
  const int owner = __builtin_ctzll(hit);
  d.block = __shfl(blk, owner, 64);
  d.before = __shfl(run, owner, 64);
  return d;
}

// The token of that block at which the running sum reaches the target, by one wavefront, four tokens of weights e per
// lane; its last live token if rounding left nothing to find.
__device__ __forceinline__ int find_token(const Drawn &d, const float *e) {
  const int lane = threadIdx.x & 63;
  const float mine = (e[0] + e[1]) + (e[2] + e[3]);
  float li = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const float up = __shfl_up(li, o, 64);
    if (lane >= o) li += up;
  }
  double run = d.before + (double)(li - mine);
  int found = -1, lastp = -1;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (e[i] > 0.f) {
      lastp = d.block * kBonusBlock + 4 * lane + i;
      run += (double)e[i];
      if (found < 0 && run >= d.target) found = lastp;
    }
  }
  // first lane that found its element wins (vocabulary order = lane order)
  const unsigned long long hit = __builtin_amdgcn_ballot_w64(found >= 0);
  if (hit != 0ull) return __shfl(found, __builtin_ctzll(hit), 64);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) lastp = max(lastp, __shfl_xor(lastp, o, 64));
  return lastp;
}

__global__ void __launch_bounds__(kWalkThreads)
accept_sample_kernel(SampleArgs a) {
  __shared__ float row_m[SPARROW_MAX_NQ + 1], row_z[SPARROW_MAX_NQ + 1];
  __shared__ int struck[SPARROW_MAX_NQ];        // tokens rejected at the last node
  __shared__ int sh_cur;
  __shared__ double blk_tot[kBonusMaxBlocks];   // sum of the live exponentials of 256 tokens
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int n_q = a.n_q, V = a.V;
  const int64_t row0 = (int64_t)b * (n_q + 1);
  int32_t *path = a.accept_path + (int64_t)b * n_q;
  Node nd = {-2, -1, 0.f, 0.f, 0.f};
  if (w == 0) nd = fetch_node(a, b, row0, lane);
  row_statistics(a, row0, row_m, row_z);
  __syncthreads();
  int cur = -1, len = 0;
  float S = 1.f;
  unsigned long long out = 0ull;                // children rejected at the current node
  if (w == 0) {                                 // the walk, by one wavefront
    float p = -1.f;
    if (nd.parent >= -1) p = fast_exp2(nd.logit * a.inv_temp_log2 - row_m[nd.parent + 1]) / row_z[nd.parent + 1];
    int mine = -1;
    bool ended = false;
    // at most n_q + 1 levels: cur strictly increases along a path
    for (int level = 0; level <= n_q && !ended; ++level) {
      unsigned long long kids = __builtin_amdgcn_ballot_w64(nd.parent == cur);
      int next = -1;
      S = 1.f;
      out = 0ull;
      while (kids != 0ull && next < 0) {
        const int j = __builtin_ctzll(kids);
        kids &= kids - 1;
        const float pj = lane_f32(p, j);
        const bool gone = (__builtin_amdgcn_ballot_w64(nd.token == __builtin_amdgcn_readlane(nd.token, j)) & out) != 0ull;
        if (gone || pj == 0.f) continue;
        if (lane_f32(nd.u, j) * S <= pj) next = j;
        else { S -= pj; out |= 1ull << j; }
      }
      if (next < 0) { ended = true; break; }
      if (lane == len) mine = next;
      ++len;
      cur = next;
    }
    if (lane < n_q) path[lane] = mine;
    if ((out >> lane) & 1ull) struck[__popcll(out & ((1ull << lane) - 1ull))] = nd.token;
    if (!ended) cur = -2;
    if (lane == 0) {
      sh_cur = cur;
      a.accept_len[b] = len;
      if (!ended) a.bonus_id[b] = 0;            // only with a malformed tree (the walk did not end within n_q + 1 levels)
    }
  }
  __syncthreads();
  cur = sh_cur;
  if (cur < -1) return;
  // ---- bonus token: inverse CDF over what is left of the row's distribution.  The sums of
  // the row's 256-token blocks come from the statistics pass (relative to their chunk's max);
  // rescaled to the row's max, minus the struck-out tokens, they are scanned in fp64 (fp32
  // inside a block, whose sum is a small part of the mass), so the draw is decided by the fp32
  // exponentials alone (~1e-7 of the remaining mass).  Only the block that holds the target
  // is read from the logits.
  const int64_t row = row0 + cur + 1;
  const float *lg = a.logits + row * V;
  const float m = row_m[cur + 1], Z = row_z[cur + 1];
  const int n_blk = (V + kBonusBlock - 1) / kBonusBlock;
  const int bpc = (n_blk + kStatChunks - 1) / kStatChunks;
  const float *bs = a.blk_sum + row * n_blk;
  for (int ib = tid; ib < n_blk; ib += kWalkThreads)
    blk_tot[ib] = (double)bs[ib] * (double)fast_exp2(a.stats[(row * kStatChunks + ib / bpc) * 2] - m);
  __syncthreads();
  if (w != 0) return;
  const int ns = __popcll(out);
  const float nd_e = fast_exp2(nd.logit * a.inv_temp_log2 - m);
  while (out != 0ull) {            // struck-out tokens leave their blocks
    const int j = __builtin_ctzll(out), x = __builtin_amdgcn_readlane(nd.token, j);
    out &= out - 1;
    const double left = blk_tot[x / kBonusBlock] - (double)lane_f32(nd_e, j);
    blk_tot[x / kBonusBlock] = left > 0.0 ? left : 0.0;      // (every lane stores the same value)
  }
  const Drawn d = find_block(blk_tot, n_blk, [&](double) {
    return (double)uniform_of(a, b, -1) * (double)S * (double)Z;        // unnormalised units
  });
  int pick = -1;
  if (d.block >= 0) {
    float e[4];                    // 0 past the end of the vocabulary and for struck-out tokens
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int v = d.block * kBonusBlock + 4 * lane + i;
      e[i] = 0.f;
      if (v < V) {
        e[i] = fast_exp2(lg[v] * a.inv_temp_log2 - m);
        for (int k = 0; k < ns; ++k)
          if (struck[k] == v) e[i] = 0.f;
      }
    }
    pick = find_token(d, e);
  }
  if (lane == 0) a.bonus_id[b] = max(pick, 0);
}

// Acceptance against a SAMPLED draft: the children of a node were drawn from the draft's
// distribution q (row of draft_q), and child j with token x is accepted with probability
// min(1, (R[x] / S) / q[x]), where R is the residual of the target's p after the rejections so far
// at this node (R <- max(R - S q, 0) on every rejection, S its sum); the bonus token comes from R.
// One workgroup per sequence.  R is never stored: a token's residual after k rejections follows
// from its p, its q and the k sums S_0 .. S_{k-1}, so a rejection costs one pass over the row
// (logits and q) for the next sum, which also leaves the sums per block of 256 tokens in LDS for
// the bonus draw: scan over the blocks, then a search inside the block that holds the target.
// A pass is one workgroup's read of 8 V bytes and bound by its latency and by the exponentials: four blocks per
// wavefront are in flight, and rows of odd vocabularies, which start at any multiple of 4 bytes, are read by the same
// 16-byte loads.
// kStage = 0: that workgroup does everything.  Where a pass takes it longer than two more launches, three kernels: 1,
// the walk up to the first residual sum; residual_sums_kernel, that pass by the whole chip; 2, the rest from there
// (further rejections at the same node, and nodes further down, again by one workgroup).  One kernel that fetched level
// by level / as here, us of kernels: 4 chains of 8 over 64,003 27.7 / 13.2, 6 of 3 over 152,064 38.4 / 14.4; in one
// kernel, 5 trees of 62 over 6,828 29.0 / 17.0.
constexpr int kMaxRejections = SPARROW_MAX_NQ;
constexpr int kAhead = 4;

struct WalkState {
  int32_t cur, len;         // node, accepted so far (cur = -2: malformed tree, nothing to draw)
  int32_t k, j;             // rejections at the node (0 or 1), the first child that is still to be tested
  float m, Z;               // of the node's row
};
// The walk up to the first node that has to know a residual sum, by one wavefront: children are tested against the
// row's own distribution until one is rejected, or a node has no child left.
__device__ __forceinline__ WalkState walk_unrejected(const SampleArgs &a, const Node &nd, const float *row_m,
                                                     const float *row_z, int32_t *path) {
  const int lane = threadIdx.x & 63, n_q = a.n_q;
  float p = 0.f, Z = 0.f;
  if (nd.parent >= -1) {
    p = fast_exp2(nd.logit * a.inv_temp_log2 - row_m[nd.parent + 1]);
    Z = row_z[nd.parent + 1];
  }
  const bool pass = p > 0.f && nd.u * nd.q * Z <= p;         // as the first child tested at its parent
  const unsigned long long passes = __builtin_amdgcn_ballot_w64(pass);
  WalkState s = {-1, 0, 0, n_q, 0.f, 0.f};
  int mine = -1;
  bool ended = false;
  for (int level = 0; level <= n_q; ++level) {
    // (nodes after their parent only: the others of a malformed tree are never reached)
    const unsigned long long kids = __builtin_amdgcn_ballot_w64(nd.parent == s.cur && lane > s.cur);
    const int j = kids != 0ull ? __builtin_ctzll(kids) : n_q;
    if (j == n_q || ((passes >> j) & 1ull) == 0ull) {
      s.k = j < n_q;
      s.j = (kids & (kids - 1)) != 0ull ? j + 1 : n_q;       // n_q: no sibling left to test, the walk goes no further
      ended = true;
      break;
    }
    if (lane == s.len) mine = j;
    ++s.len;
    s.cur = j;
  }
  if (lane < n_q) path[lane] = mine;
  if (ended) { s.m = row_m[s.cur + 1]; s.Z = row_z[s.cur + 1]; }
  else s.cur = -2;
  return s;
}

template <int kStage>
__global__ void __launch_bounds__(kWalkThreads)
accept_sample_q_kernel(SampleArgs a) {
  __shared__ float row_m[SPARROW_MAX_NQ + 1], row_z[SPARROW_MAX_NQ + 1];
  __shared__ Node nodes[SPARROW_MAX_NQ];
  __shared__ WalkState sh_state;
  __shared__ float S_s[kMaxRejections + 1];     // residual sums at the current node
  __shared__ double blk_tot[kStage == 1 ? 1 : kBonusMaxBlocks];   // sums of the current residual per 256 tokens
  __shared__ double wave_tot[kWalkThreads / 64];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int n_q = a.n_q, V = a.V;
  const int64_t row0 = (int64_t)b * (n_q + 1);
  int32_t *path = a.accept_path + (int64_t)b * n_q;
  WalkState *const state = reinterpret_cast<WalkState *>(a.state) + b;
  // nodes and row statistics (in LDS behind the next barrier), in the kernels that test children
  auto fetch = [&]() {
    Node nd = {-2, -1, 0.f, 0.f, 0.f};
    if (w == 0) {
      nd = fetch_node(a, b, row0, lane);
      if (lane < n_q) nodes[lane] = nd;
    }
    row_statistics(a, row0, row_m, row_z);
    return nd;
  };
  if constexpr (kStage < 2) {
    const Node nd = fetch();
    __syncthreads();
    if (w == 0) {
      const WalkState s = walk_unrejected(a, nd, row_m, row_z, path);
      if (lane == 0) { if constexpr (kStage == 1) *state = s; else sh_state = s; }
    }
    if constexpr (kStage == 1) return;
    __syncthreads();
  }
  const int n_blk = (V + kBonusBlock - 1) / kBonusBlock;
  WalkState s;
  if constexpr (kStage == 2) s = *state; else s = sh_state;
  int cur = s.cur, len = s.len;
  if (cur < -1) {                                             // malformed tree only
    if (tid == 0) { a.accept_len[b] = len; a.bonus_id[b] = 0; }
    return;
  }
  bool entered = kStage != 2;                                 // stage 2: the sums that the walk stopped for are there
  int k = s.k, first = s.j;                                   // rejections at this node so far, next child to test
  float m = s.m;
  if (kStage == 2 && first < n_q) (void)fetch();
  if (tid == 0) S_s[0] = s.Z;
  __syncthreads();
  for (int level = 0; level <= n_q; ++level) {
    const int64_t row = row0 + cur + 1;
    const float *lg = a.logits + row * V;
    const float *q = a.draft_q + row * V;
    // residual of token v after k rejections (unnormalised: p = exp2(..) / S_0)
    auto residual = [&](float lv, float qv, int kk) {
      float r = fast_exp2(lv * a.inv_temp_log2 - m);
      for (int i = 0; i < kk; ++i) r = fmaxf(r - S_s[i] * qv, 0.f);
      return r;
    };
    // one pass over the row: sums of the residual after kk rejections per block of 256 tokens
    // (into blk_tot) and in total (into S_s[kk])
    auto block_sums = [&](int kk) {
      double mine = 0.0;
      for (int ib0 = w; ib0 < n_blk; ib0 += kAhead * (kWalkThreads / 64)) {
        f32x4u l4[kAhead], q4[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const int v = (ib0 + u * (kWalkThreads / 64)) * kBonusBlock + 4 * lane;
          if (v + 3 < V) {
            l4[u] = *reinterpret_cast<const f32x4u *>(lg + v);
            q4[u] = *reinterpret_cast<const f32x4u *>(q + v);
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              l4[u][i] = v + i < V ? lg[v + i] : 0.f;
              q4[u][i] = v + i < V ? q[v + i] : 0.f;
            }
          }
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const int ib = ib0 + u * (kWalkThreads / 64), v = ib * kBonusBlock + 4 * lane;
          if (ib >= n_blk) break;                             // uniform over the wavefront
          float t = 0.f;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (v + i < V) t += residual(l4[u][i], q4[u][i], kk);
          t = wave_sum_valu(t);
          if (lane == 0) blk_tot[ib] = (double)t;
          mine += (double)t;                                  // the same value in every lane
        }
      }
      if (lane == 0) wave_tot[w] = mine;
      __syncthreads();
      if (tid == 0 && kk > 0) {
        double tot = 0.0;
        for (int i = 0; i < kWalkThreads / 64; ++i) tot += wave_tot[i];
        S_s[kk] = (float)tot;
      }
      __syncthreads();                                        // (wave_tot is reused by the next pass)
    };
    if (!entered) {
      entered = true;
      const float *bs = a.blk_sum + row * n_blk;
      double mine = 0.0;
      for (int ib = tid; ib < n_blk; ib += kWalkThreads) {
        const double t = (double)bs[ib];
        blk_tot[ib] = t;
        mine += t;
      }
      if (first < n_q) {                                      // the total, for the siblings (the draw finds its own)
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) mine += __shfl_xor(mine, o, 64);
        if (lane == 0) wave_tot[w] = mine;
        __syncthreads();
        if (tid == 0 && k > 0) {
          double tot = 0.0;
          for (int i = 0; i < kWalkThreads / 64; ++i) tot += wave_tot[i];
          S_s[k] = (float)tot;
        }
      }
      __syncthreads();
    } else {
      block_sums(k);
    }
    int next = -1;
    for (int j = first; j < n_q && next < 0; ++j) {           // uniform: the nodes are shared
      if (nodes[j].parent != cur) continue;
      const float r = residual(nodes[j].logit, nodes[j].q, k);
      if (r > 0.f && nodes[j].u * nodes[j].q * S_s[k] <= r) { next = j; break; }
      if (k == kMaxRejections) continue;                      // (cannot happen: at most n_q children)
      block_sums(++k);                                        // rejected: the next residual's sum
    }
    if (next < 0) {
      // ---- bonus token: inverse CDF of the residual after k rejections, in vocabulary order
      if (w != 0) return;
      const Drawn d = find_block(blk_tot, n_blk, [&](double total) {
        return (double)uniform_of(a, b, -1) * (double)(k > 0 ? (float)total : S_s[0]);
      });
      int pick = -1;
      if (d.block >= 0) {
        float e[4];
        const int v = d.block * kBonusBlock + 4 * lane;
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = v + i < V ? residual(lg[v + i], q[v + i], k) : 0.f;
        pick = find_token(d, e);
      }
      if (lane == 0) {
        a.bonus_id[b] = max(pick, 0);
        a.accept_len[b] = len;
      }
      return;
    }
    // accepted after a rejection at its parent: the nodes below, up to the next one that has to know a sum
    __syncthreads();                                          // S_s and blk_tot are rewritten at the next node
    if (tid == 0) path[len] = next;
    ++len;
    cur = next;
    for (k = 0, first = n_q;;) {
      int j = cur + 1;
      while (j < n_q && nodes[j].parent != cur) ++j;
      m = row_m[cur + 1];
      if (j == n_q) break;                                    // no child: the draw from the row itself
      const float r = fast_exp2(nodes[j].logit * a.inv_temp_log2 - m);
      if (!(r > 0.f && nodes[j].u * nodes[j].q * row_z[cur + 1] <= r)) {
        k = 1;
        first = j + 1;
        break;
      }
      if (tid == 0) path[len] = j;
      ++len;
      cur = j;
    }
    if (tid == 0) S_s[0] = row_z[cur + 1];
    __syncthreads();
  }
  if (tid == 0) { a.accept_len[b] = len; a.bonus_id[b] = 0; }   // malformed tree only
}

// Sums of the residual at the node where a sequence's walk stopped, per block of 256 tokens, in place of the row's
// own block sums.  Two blocks per wavefront: 64,003 tokens are 32 workgroups per sequence, and the pass is one round
// trip for the state and one for the row.
constexpr int kSumBlocks = 2;
__global__ void __launch_bounds__(256)
residual_sums_kernel(SampleArgs a) {
  const int b = blockIdx.y, lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  const int V = a.V, n_blk = (V + kBonusBlock - 1) / kBonusBlock;
  const WalkState s = reinterpret_cast<const WalkState *>(a.state)[b];
  if (s.cur < -1) return;
  const int64_t row = (int64_t)b * (a.n_q + 1) + s.cur + 1;
  const float *lg = a.logits + row * V;
  const float *q = a.draft_q + row * V;
  float l4[kSumBlocks][4], q4[kSumBlocks][4];
#pragma unroll
  for (int u = 0; u < kSumBlocks; ++u) {
    const int v = (w * kSumBlocks + u) * kBonusBlock + 4 * lane;
    if (v + 3 < V) {
      const f32x4 x = *reinterpret_cast<const f32x4u *>(lg + v), y = *reinterpret_cast<const f32x4u *>(q + v);
#pragma unroll
      for (int i = 0; i < 4; ++i) { l4[u][i] = x[i]; q4[u][i] = y[i]; }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        l4[u][i] = v + i < V ? lg[v + i] : 0.f;
        q4[u][i] = v + i < V ? q[v + i] : 0.f;
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kSumBlocks; ++u) {
    const int ib = w * kSumBlocks + u, v = ib * kBonusBlock + 4 * lane;
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (v + i < V) {
        const float e = fast_exp2(l4[u][i] * a.inv_temp_log2 - s.m);
        t += s.k > 0 ? fmaxf(e - s.Z * q4[u][i], 0.f) : e;
      }
    t = wave_sum_valu(t);
    if (lane == 0 && ib < n_blk) a.blk_sum[row * n_blk + ib] = t;
  }
}

}  // namespace

size_t sample_state_bytes(int B) { return (size_t)B * sizeof(WalkState); }

hipError_t launch_logit_stats(const SampleArgs &a, hipStream_t st) {
  // (rows and blocks between the measured sizes above; more than 16 blocks do not fit one wavefront's registers)
  const int bpc = stat_blocks_per_chunk(a.V);
  if (bpc <= 4 || (bpc <= kStatAhead && a.M >= 32))
    hipLaunchKernelGGL(logit_stats_kernel<1>, dim3(kStatChunks / kStatWaves, a.M), dim3(kStatThreads), 0, st, a);
  else
    hipLaunchKernelGGL(logit_stats_kernel<kStatWaves>, dim3(kStatChunks, a.M), dim3(kStatThreads), 0, st, a);
  return hipGetLastError();
}

// Up to here one workgroup walks a sequence alone: two rounds of loads for its 16 wavefronts, against two launches more.
// One kernel / three, us a call with its lm_head (256 columns): four chains of 8 over 16,000 18.8 / 20.9, 18,000 20.9 / 22.8,
// 24,000 22.6 / 23.1, 32,000 23.4 / 23.4, 48,000 28.7 / 26.8, 64,003 32.5 / 29.2; six trees of 25 over 24,000 39.7 / 41.0,
// 32,000 40.9 / 41.8; one chain of 5 over 24,000 18.9 / 19.0, 32,000 20.6 / 20.6, 64,003 28.4 / 25.2.
constexpr int kOneWorkgroupVocab = 32768;

hipError_t launch_accept_sample(const SampleArgs &a, hipStream_t st) {
  if (a.draft_q == nullptr) {
    hipLaunchKernelGGL(accept_sample_kernel, dim3(a.B), dim3(kWalkThreads), 0, st, a);
  } else if (a.state != nullptr && a.V > kOneWorkgroupVocab) {
    const int n_blk = (a.V + kBonusBlock - 1) / kBonusBlock;
    hipLaunchKernelGGL(accept_sample_q_kernel<1>, dim3(a.B), dim3(kWalkThreads), 0, st, a);
    hipLaunchKernelGGL(residual_sums_kernel, dim3((n_blk + 4 * kSumBlocks - 1) / (4 * kSumBlocks), a.B), dim3(256), 0, st, a);
    hipLaunchKernelGGL(accept_sample_q_kernel<2>, dim3(a.B), dim3(kWalkThreads), 0, st, a);
  } else {
    hipLaunchKernelGGL(accept_sample_q_kernel<0>, dim3(a.B), dim3(kWalkThreads), 0, st, a);
  }
  return hipGetLastError();
}

}  // namespace sparrow
