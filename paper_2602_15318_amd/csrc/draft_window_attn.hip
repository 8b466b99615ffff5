// Draft model's text-anchored window attention (VATA, Eq. 2): one query per sequence attends
// only to the `window` most recent text positions.  The kernel walks the precomputed
// text-position index, so keys and values at visual positions are never addressed.
//
// The whole job is at most a few hundred KB, so it is latency-bound: a single launch, workgroups of 16 wavefronts, one to
// four per (sequence, query head), spread over as many compute units as there are; each re-reads its KV head's window
// from L2.  A group of LPT lanes owns one token (each lane one 16-byte slice of the K row and its part of the V row); every
// lane group keeps its own online-softmax stream (m, l, o), updated once per round of kUnroll gathered tokens in flight;
// streams are merged once at the end (lane groups by shuffles, wavefronts through LDS).
//
// What a workgroup takes beyond a launch and two dependent round trips (positions, rows) is the way of its rows into one
// compute unit and the arithmetic of 16 wavefronts on four SIMDs, so both are cut: heads share out the values' columns
// where compute units are idle, short windows run without the rounds' empty tokens, and a round has one softmax update
// instead of eight.  us a call, one update per token / per round / columns shared out / and rounds of two for short windows:
//   28/4 heads of 128, one sequence, window 512 6.7 / 6.2 / 5.1 / 5.1, 64 6.7 / 6.2 / 5.0 / 3.7, 1,000 10.2 / 9.6 / 7.5 / 7.5;
//   six sequences, 40/8 heads of 64, window 256 7.3 / 6.8 / 6.8 / 4.8; four, 32/8 of 128, 512 7.0 / 6.4 / 6.0 / 6.0;
//   fp32, one sequence, 28/4 of 128, 512 9.1 / 8.3 / 6.8 / 6.8, 4/1 of 64, 32 4.2 / 3.9 / 3.7 / 3.0.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "draft_window_attn.hpp"

namespace sparrow {

constexpr int kDraftWaves = 16;

// kDS = workgroups per query head: each takes all keys of the window and D / kDS of the values' columns.
// kUnroll = tokens in flight per lane group, a round.
template <typename T, int D, int kDS, int kUnroll>
__global__ void __launch_bounds__(kDraftWaves * 64)
draft_window_attn_kernel(DraftArgs a, DraftTable tab) {
  constexpr int PER = Elem<T>::kPer16B;       // elements per 16-byte slice
  constexpr int LPT = D / PER;                // lanes per token
  constexpr int TPW = 64 / LPT;               // tokens per wavefront per step
  constexpr int STEP = kDraftWaves * TPW;     // tokens per workgroup per step
  constexpr int VPER = PER / kDS;             // value columns of a lane
  typedef typename std::conditional<kDS == 1, u32x4, typename std::conditional<kDS == 2, u32x2, unsigned int>::type>::type vword_t;
  static_assert(kDS == 1 || kDS == 2 || kDS == 4, "16, 8 or 4 bytes of values per lane and token");
  __shared__ float Om[kDraftWaves][D / kDS];
  __shared__ float Mm[kDraftWaves];
  __shared__ float Lm[kDraftWaves];

  const int b = blockIdx.x, c = blockIdx.y;
  const int g = a.Hq / a.Hkv;
  const int r0 = (int)blockIdx.z / kDS, part = (int)blockIdx.z % kDS;   // head of the group, part of the columns
  const int h = c * g + r0;
  const int tid = threadIdx.x, w = tid / 64, lane = tid % 64;
  const int sub = lane / LPT, vec = lane % LPT;

  const int n_text = tab.cu_text[b + 1] - tab.cu_text[b];
  const int n = min(n_text, a.window);
  const int32_t *idx = a.text_idx + tab.cu_text[b] + (n_text - n);
  const int64_t tok_base = tab.cu_len[b];
  const T *K = (const T *)a.k + c * a.stride_head + vec * PER;
  const T *V = (const T *)a.v + c * a.stride_head + part * (D / kDS) + vec * VPER;

  // positions of a round of kUnroll tokens; the next round's are asked for with this round's rows
  int pos[kUnroll];
  auto positions = [&](int j0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) pos[u] = idx[min(j0 + u * STEP, n - 1)];   // clamped: always a valid text position
  };
  int j0 = w * TPW + sub;
  positions(j0);
  // this lane's slice of the query (raw storage words; the scale is applied to the scores)
  constexpr bool kBf16 = std::is_same<T, bf16_t>::value;
  const u32x4 qw = *(const u32x4 *)((const T *)a.q + ((int64_t)b * a.Hq + h) * D + vec * PER);
  float qf[PER];
  Elem<T>::unpack(qw, qf);

  float m = kNegBig, l = 0.f, acc[VPER];
#pragma unroll
  for (int u = 0; u < VPER; ++u) acc[u] = 0.f;

  for (; j0 < n; j0 += STEP * kUnroll) {
    u32x4 kw[kUnroll];
    vword_t vw[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int64_t off = (tok_base + pos[u]) * a.stride_tok;
      kw[u] = *(const u32x4 *)(K + off);
      vw[u] = vword_t{};                   // past the end no value: a duplicate of an infinite one would give 0 * inf
      if (j0 + u * STEP < n) vw[u] = *(const vword_t *)(V + off);
    }
    if (j0 + STEP * kUnroll < n) positions(j0 + STEP * kUnroll);
    // one softmax update for the round
    float s[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      float d = 0.f;
      if (kBf16) {   // packed bf16 dot products with fp32 accumulation, no unpacking of K
        typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
        const unsigned qe[4] = {qw.x, qw.y, qw.z, qw.w};
        const unsigned ke[4] = {kw[u].x, kw[u].y, kw[u].z, kw[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, qe[e]), __builtin_bit_cast(bf16x2, ke[e]), d, false);
      } else {
        float kf[PER];
        Elem<T>::unpack(kw[u], kf);
#pragma unroll
        for (int e = 0; e < PER; ++e) d = fmaf(qf[e], kf[e], d);
      }
      s[u] = group_sum<LPT>(d) * a.scale_log2;
      if (j0 + u * STEP >= n) s[u] = -INFINITY;
    }
    float m_new = m;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) m_new = fmaxf(m_new, s[u]);
    const float alpha = fast_exp2(m - m_new);
    m = m_new;
    l *= alpha;
#pragma unroll
    for (int e = 0; e < VPER; ++e) acc[e] *= alpha;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const float p = fast_exp2(s[u] - m);
      l += p;
      float vf[VPER];
      unsigned int word[4 / kDS];
      __builtin_memcpy(word, &vw[u], sizeof(vword_t));
#pragma unroll
      for (int e = 0; e < VPER; ++e)
        vf[e] = kBf16 ? (e & 1 ? bf16hi_to_f32(word[e >> 1]) : bf16lo_to_f32(word[e >> 1])) : __uint_as_float(word[kBf16 ? 0 : e]);
#pragma unroll
      for (int e = 0; e < VPER; ++e) acc[e] = fmaf(p, vf[e], acc[e]);
    }
  }

  // merge the TPW lane-group streams of this wavefront
  auto merge_with = [&](auto xor_tag) {
    constexpr int O = decltype(xor_tag)::value;
    const float m_o = lane_xor<O>(m, lane);
    const float l_o = lane_xor<O>(l, lane);
    const float m_new = fmaxf(m, m_o);
    const float wa = fast_exp2(m - m_new), wb = fast_exp2(m_o - m_new);
    l = l * wa + l_o * wb;
    m = m_new;
#pragma unroll
    for (int e = 0; e < VPER; ++e) {
      const float a_o = lane_xor<O>(acc[e], lane);
      acc[e] = acc[e] * wa + a_o * wb;
    }
  };
  if (LPT <= 8) merge_with(std::integral_constant<int, 8>{});
  if (LPT <= 16) merge_with(std::integral_constant<int, 16>{});
  merge_with(std::integral_constant<int, 32>{});
  if (sub == 0) {
#pragma unroll
    for (int e = 0; e < VPER; ++e) Om[w][vec * VPER + e] = acc[e];
    if (vec == 0) { Mm[w] = m; Lm[w] = l; }
  }
  __syncthreads();
  // merge the wavefronts: a thread per column
  if (tid >= D / kDS) return;
  float mm = kNegBig;
#pragma unroll
  for (int ww = 0; ww < kDraftWaves; ++ww) mm = fmaxf(mm, Mm[ww]);
  float ll = 0.f, oo = 0.f;
#pragma unroll
  for (int ww = 0; ww < kDraftWaves; ++ww) {
    const float wt = fast_exp2(Mm[ww] - mm);
    ll = fmaf(Lm[ww], wt, ll);
    oo = fmaf(Om[ww][tid], wt, oo);
  }
  Elem<T>::store((T *)a.out + ((int64_t)b * a.Hq + h) * D + part * (D / kDS) + tid, oo / ll);
  if (a.lse != nullptr && tid == 0 && part == 0) a.lse[(int64_t)b * a.Hq + h] = (mm + fast_log2(ll)) * kLn2;
}

// Rounds of two tokens per lane group where they cover every window of the call: the tokens of a round are all fetched and
// worked on, and with eight a window of 64 took as long as one of 512.
template <typename T, int D, int kDS>
static hipError_t launch(const DraftArgs &a, const DraftTable &tab, int longest, hipStream_t st) {
  const dim3 grid(a.B, a.Hkv, kDS * (a.Hq / a.Hkv)), block(kDraftWaves * 64);
  constexpr int kStep = kDraftWaves * 64 * Elem<T>::kPer16B / D;             // tokens that a workgroup takes side by side
  if (longest <= 2 * kStep) hipLaunchKernelGGL((draft_window_attn_kernel<T, D, kDS, 2>), grid, block, 0, st, a, tab);
  else hipLaunchKernelGGL((draft_window_attn_kernel<T, D, kDS, 8>), grid, block, 0, st, a, tab);
  return hipGetLastError();
}

// As many workgroups per head as leave one to a compute unit: the keys are read and multiplied by each of them.  Two where
// that makes more than 256: 28 heads of 128, six sequences, window 100 6.4 -> 9.1 us, 40 of 64, six, 256 6.8 -> 9.8.
template <typename T, int D>
static hipError_t launch(const DraftArgs &a, const DraftTable &tab, hipStream_t st) {
  int longest = 0;
  for (int b = 0; b < a.B; ++b) longest = std::max(longest, std::min(tab.cu_text[b + 1] - tab.cu_text[b], a.window));
  const int heads = a.B * a.Hq;
  if (heads <= 64) return launch<T, D, 4>(a, tab, longest, st);
  return heads <= 128 ? launch<T, D, 2>(a, tab, longest, st) : launch<T, D, 1>(a, tab, longest, st);
}

hipError_t launch_draft_window_attn(int dtype, const DraftArgs &a, const DraftTable &tab,
                                    hipStream_t st) {
  if (dtype == SPARROW_F32)
    return a.d == 64 ? launch<float, 64>(a, tab, st) : launch<float, 128>(a, tab, st);
  return a.d == 64 ? launch<bf16_t, 64>(a, tab, st) : launch<bf16_t, 128>(a, tab, st);
}

}  // namespace sparrow
