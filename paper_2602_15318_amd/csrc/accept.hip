// Greedy acceptance, plain-ALU lm_head pass and the finalize pass.
//
// Step 1 (this file: hidden sizes beyond the matrix-core kernels of accept_mfma.hip, bf16 above 8,192 and fp32
// above 2^20, which the entry points accept as they always did): logits of the
// B*(n_q+1) verified rows against the whole vocabulary, never written out: every wavefront keeps,
// per row, the best (value, lowest index) of the vocabulary range it owns and writes one
// candidate per row.  Step 2: reduce the candidates to the target's greedy token per row
// (lowest index wins ties), then walk the draft chain / tree from the last accepted token,
// taking the lowest-numbered child whose drafted token equals the target token of the current
// row (lossless greedy acceptance at temperature 0).
#include "accept.hpp"
#include "common.hpp"

namespace sparrow {

constexpr int kGenVW = 4;        // vocabulary rows per wavefront step
constexpr int kGenMC = 8;        // hidden rows per pass
constexpr int kGenBlocks = 512;  // workgroups of 4 wavefronts

template <typename T>
__global__ void __launch_bounds__(256) lm_head_generic_kernel(AcceptArgs a) {
  constexpr int PER = Elem<T>::kPer16B;
  const int lane = threadIdx.x % 64;
  const int gw = blockIdx.x * 4 + threadIdx.x / 64;   // global wavefront = candidate slot
  const int n_w = gridDim.x * 4;
  const int per = (a.V + n_w - 1) / n_w;
  const int v0 = min(a.V, gw * per), v1 = min(a.V, v0 + per);
  const T *Wm = (const T *)a.lm_head;
  const T *Hd = (const T *)a.hidden;

  for (int r0 = 0; r0 < a.M; r0 += kGenMC) {
    float best[kGenMC];
    int best_i[kGenMC];
#pragma unroll
    for (int r = 0; r < kGenMC; ++r) { best[r] = -INFINITY; best_i[r] = 0x7fffffff; }
    for (int vb = v0; vb < v1; vb += kGenVW) {
      float acc[kGenVW][kGenMC];
#pragma unroll
      for (int j = 0; j < kGenVW; ++j)
#pragma unroll
        for (int r = 0; r < kGenMC; ++r) acc[j][r] = 0.f;
      for (int x = lane * PER; x < a.H; x += 64 * PER) {
        float wf[kGenVW][PER];
#pragma unroll
        for (int j = 0; j < kGenVW; ++j) {
          const int v = min(vb + j, v1 - 1);
          u32x4 ww = *(const u32x4 *)(Wm + (int64_t)v * a.H + x);
          Elem<T>::unpack(ww, wf[j]);
        }
#pragma unroll
        for (int r = 0; r < kGenMC; ++r) {
          const int row = min(r0 + r, a.M - 1);
          u32x4 hw = *(const u32x4 *)(Hd + (int64_t)row * a.H + x);
          float hf[PER];
          Elem<T>::unpack(hw, hf);
#pragma unroll
          for (int j = 0; j < kGenVW; ++j)
#pragma unroll
            for (int e = 0; e < PER; ++e) acc[j][r] = fmaf(wf[j][e], hf[e], acc[j][r]);
        }
      }
#pragma unroll
      for (int j = 0; j < kGenVW; ++j) {
        const int v = vb + j;
#pragma unroll
        for (int r = 0; r < kGenMC; ++r) {
          const float s = wave_sum(acc[j][r]);
          if (v < v1 && s > best[r]) { best[r] = s; best_i[r] = v; }   // ascending v: lowest wins
          if (a.logits != nullptr && lane == 0 && v < v1 && r0 + r < a.M)
            a.logits[(int64_t)(r0 + r) * a.V + v] = s;
        }
      }
    }
    if (lane == 0) {
#pragma unroll
      for (int r = 0; r < kGenMC; ++r) {
        if (r0 + r < a.M) {
          a.cand_val[(int64_t)(r0 + r) * a.n_cand + gw] = best[r];
          a.cand_idx[(int64_t)(r0 + r) * a.n_cand + gw] = best_i[r];
        }
      }
    }
  }
}

// One workgroup of 16 wavefronts per sequence: wavefront w reduces the candidates of its rows w,
// w+16, ... (64 lanes stride over the row's candidates, then a butterfly), then one wavefront walks the
// sequence's chain / tree.  (One workgroup for all sequences took 18 us at 8 x 31 rows.)
// What bounds it: the loads of one compute unit (16 cycles an instruction; four candidates by one where rows are whole
// 16 bytes) and the walk, in which lane j now holds node j and a ballot finds the child (a thread that looked through the
// nodes in LDS paid some 100 cycles for each).  us in a trace, before / now: 8 trees of 30 nodes, 256 candidates
// a row 8.2 / 4.8, a chain of 4, 16 candidates 3.6 / 2.2, of 8, 256 candidates 4.3 / 4.2.
__global__ void __launch_bounds__(1024) accept_finalize_kernel(AcceptArgs a) {
  __shared__ int32_t tgt[SPARROW_MAX_NQ + 1];
  __shared__ int32_t dr_s[SPARROW_MAX_NQ], par_s[SPARROW_MAX_NQ];
  const int tid = threadIdx.x, b = blockIdx.x;
  const int w = tid >> 6, lane = tid & 63;
  const int n_rows = a.n_q + 1, base = b * n_rows;
  // draft tokens and parents of the sequence into LDS while the candidates are being reduced:
  // the walk below is a chain of dependent reads and should not pay a memory round trip each
  if (tid < a.n_q) {
    dr_s[tid] = a.draft_ids[b * a.n_q + tid];
    par_s[tid] = a.parent ? a.parent[(int64_t)b * a.parent_stride + tid] : tid - 1;
  }
  // two rows per wavefront at a time (rows r and r + 16): their candidate loads are in flight
  // together, and the 64-lane argmax runs on the vector ALU (maximum, then the lowest index
  // among the lanes that hold it)
  const int per = (a.n_cand & 3) == 0 ? 256 : 64;        // candidates of a load: rows of whole 16 bytes, or not
  for (int r0 = w; r0 < n_rows; r0 += 32) {
    const int rows = r0 + 16 < n_rows ? 2 : 1;
    float bv[2] = {-INFINITY, -INFINITY};
    int bi[2] = {0x7fffffff, 0x7fffffff};
    constexpr int kU = 4;                                // loads in flight per row; those past the row's end are left out
    for (int c0 = 0; c0 < a.n_cand; c0 += per * kU) {
      f32x4 v[2][kU];
      u32x4 x[2][kU];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          if (h >= rows || c0 + per * u >= a.n_cand) continue;             // (uniform)
          const int64_t at = (int64_t)(base + r0 + 16 * h) * a.n_cand;
          const int c = c0 + per * u + (per == 256 ? 4 * lane : lane);
          v[h][u] = (f32x4){-INFINITY, -INFINITY, -INFINITY, -INFINITY};
          x[h][u] = (u32x4){0x7fffffffu, 0x7fffffffu, 0x7fffffffu, 0x7fffffffu};
          if (c >= a.n_cand) continue;
          if (per == 256) {
            v[h][u] = *reinterpret_cast<const f32x4 *>(a.cand_val + at + c);
            x[h][u] = *reinterpret_cast<const u32x4 *>(a.cand_idx + at + c);
          } else {
            v[h][u][0] = a.cand_val[at + c];
            x[h][u][0] = (unsigned int)a.cand_idx[at + c];
          }
        }
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          if (h >= rows || c0 + per * u >= a.n_cand) continue;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int i = (int)x[h][u][e];
            if (v[h][u][e] > bv[h] || (v[h][u][e] == bv[h] && i < bi[h])) { bv[h] = v[h][u][e]; bi[h] = i; }
          }
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h >= rows) continue;
      const int r = r0 + 16 * h;
      const float wv = wave_max_valu(bv[h]);
      const int wi = wave_min_valu(bv[h] == wv ? bi[h] : 0x7fffffff);
      if (lane == 0) { tgt[r] = wi; a.target_ids[base + r] = wi; }
    }
  }
  __syncthreads();
  if (w == 0) {
    // lane j: node j and its row's token.  The child is the lowest node that fits; it has a larger index than its
    // parent, so there are at most n_q steps.
    const bool node = lane < a.n_q;
    const int dr = node ? dr_s[lane] : -1, par = node ? par_s[lane] : -2, mine = node ? tgt[lane + 1] : 0;
    int cur = -1, len = 0, tok = __builtin_amdgcn_readfirstlane(tgt[0]), path = -1;
    for (;;) {
      const unsigned long long fit = __builtin_amdgcn_ballot_w64(node && lane > cur && par == cur && dr == tok);
      if (fit == 0ull) break;
      cur = __builtin_ctzll(fit);
      if (lane == len) path = cur;
      ++len;
      tok = __builtin_amdgcn_readlane(mine, cur);
    }
    if (node) a.accept_path[(int64_t)b * a.n_q + lane] = path;
    if (lane == 0) {
      a.accept_len[b] = len;
      a.bonus_id[b] = tok;
    }
  }
}

hipError_t launch_lm_head_generic(int dtype, const AcceptArgs &a, hipStream_t st) {
  const int blocks = a.n_cand / 4;
  if (dtype == SPARROW_F32)
    hipLaunchKernelGGL(lm_head_generic_kernel<float>, dim3(blocks), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL(lm_head_generic_kernel<bf16_t>, dim3(blocks), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_accept_finalize(const AcceptArgs &a, hipStream_t st) {
  hipLaunchKernelGGL(accept_finalize_kernel, dim3(a.B), dim3(1024), 0, st, a);
  return hipGetLastError();
}

int generic_num_candidates(int V) {
  int blocks = kGenBlocks;
  while (blocks > 1 && blocks * 4 * kGenVW > V) blocks /= 2;
  return blocks * 4;
}

}  // namespace sparrow
