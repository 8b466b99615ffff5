// Internal interface of the verification-attention kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/sparrow.h"
#include "common.hpp"

namespace sparrow {

// Per-call schedule, passed to the kernels by value (no device-side schedule buffer, so a call is
// a pure function of its arguments and can be captured in a graph).  The context of every
// sequence is cut into splits of `chunk` tokens; split slots are numbered across sequences.
struct SeqTable {
  int32_t cu_len[SPARROW_MAX_BATCH + 1];    // token offsets (L_b + n_q rows per sequence)
  int32_t cu_split[SPARROW_MAX_BATCH + 1];  // split-slot offsets
};

struct VerifyArgs {
  const void *q, *k, *v;
  const int32_t *parent;  // device, or nullptr for a chain
  int32_t parent_stride;  // 0: one tree [n_q] for all sequences; else sequence b's tree at parent + b*stride
  int32_t B, n_q, Hq, Hkv, d;
  int32_t g;              // Hq / Hkv
  float inv_g;            // 1 / g
  int32_t chunk;          // longest split of the call, in tokens (the kernels derive each
                          // sequence's own split length from SeqTable)
  int32_t n_slots;        // cu_split[B]
  int32_t direct;         // matrix-core path: one split per sequence, the partial pass writes out and lse
  float scale_log2;       // softmax scale * log2(e)
  int64_t stride_tok, stride_head;
  // plain-ALU path: part_o [n_slots, n_q, Hq, d], part_ml [n_slots, n_q, Hq, 2];
  // matrix-core path: tiled per (split, KV head, row block), see verify_attn_mfma.hip
  float *part_o;          // partial outputs (plain-ALU path: unnormalised fp32; matrix-core path:
                          // normalised, fp32, or fp16 for bf16 heads of 128)
  float *part_ml;         // reference point (log2 domain) and partial sum; matrix-core path: and
                          // the scale of fp16 outputs
  void *out;              // [B*n_q, Hq, d]
  float *lse;             // [B*n_q, Hq] or nullptr
};

// Token range [t0, t1) of a split: a sequence of `len` rows with `ns` splits is cut into pieces of
// ceil(len / ns) rounded up to a whole 32-token tile (the last piece takes what is left, possibly
// nothing), so that all workgroups of a sequence stream the same number of bytes.
__host__ __device__ __forceinline__ int split_len(int len, int ns) {
  return ((len + ns - 1) / ns + 31) / 32 * 32;
}

// Which sequence owns split slot `slot`: as many as end at or before it.  Sixteen ends come with one load and are counted on
// the scalar unit (one after the other they were a round trip each ahead of a workgroup's first load); those past the
// call's sequences are out of any slot's reach.
__device__ __forceinline__ int seq_of_slot(const SeqTable &tab, int slot) {
  int b = 0;
  do {
    const int b0 = b;
#pragma unroll
    for (int k = 1; k <= 16; ++k) b += (unsigned int)(tab.cu_split[b0 + k] - slot - 1) >> 31;      // ends <= slot
  } while ((b & 15) == 0 && b > 0 && b < SPARROW_MAX_BATCH && tab.cu_split[b + 1] <= slot);
  return b;
}

// a / n and the rest by the reciprocal of n (one bit off at most).  Half a step is more than the roundings are off while a < 2^20,
// and for the rows of a KV head (a / n < 64) while n < 32,768; `large` (uniform) says that this does not hold, and the quotient
// may be one off either way (a launch has fewer than 2^23 groups; n = 1 is exact).  Corrected in every call it lies ahead of
// the query's loads: 6.8 -> 6.9 us a call over 200 tokens.
struct QuotRest { int quot, rest; };
__device__ __forceinline__ QuotRest div_by_rcp(int a, int n, float inv_n, bool large) {
  int q = (int)(((float)a + 0.5f) * inv_n), r = a - q * n;
  if (__builtin_expect(large, 0)) {
    asm volatile("" : "+v"(q));                    // (empty: keeps it a branch)
    if (r < 0) { --q; r += n; }
    else if (r >= n) { ++q; r -= n; }
  }
  return {q, r};
}
// Draft row and head (within the group of g) of row rho of a KV head
__device__ __forceinline__ QuotRest row_and_head(int rho, int g, float inv_g) { return div_by_rcp(rho, g, inv_g, g >= 32768); }
// The same of uniform numbers: of a group (split slot, KV head) or unit (KV head, row block)
__device__ __forceinline__ QuotRest div_uniform(int a, int n) {
  const QuotRest d = div_by_rcp(a, n, __builtin_amdgcn_rcpf((float)n), a >= 1 << 20);
  return {__builtin_amdgcn_readfirstlane(d.quot), __builtin_amdgcn_readfirstlane(d.rest)};
}

// Natural-log sum-exp of a row: reference point m (log2 units) and sum l.  kWide: rounded once at its full
// size.  (m may lie below the row's maximum; log2(l) is then larger than in the plain-ALU kernels and so are
// the roundings of the other form.  Root mean square error over 6,000 fp32 tokens, 60 rows, heads of 128:
// 4.9e-7 against 4.65e-7 there, 4.6e-7 in this form.)
template <bool kWide> __device__ __forceinline__ float lse_of(float m, float l) {
  return kWide ? fmaf(m, kLn2, fast_log2(l) * kLn2) : (m + fast_log2(l)) * kLn2;
}

// Partial pass, plain-ALU version: any supported dtype / head_dim.
hipError_t launch_verify_partial_generic(int dtype, const VerifyArgs &a, const SeqTable &tab,
                                         hipStream_t st);
// Partial pass, matrix-core versions (fp32 has a kernel of its own).
bool verify_partial_mfma_supported(int dtype, int head_dim);
hipError_t launch_verify_partial_mfma(int dtype, const VerifyArgs &a, const SeqTable &tab, hipStream_t st);
hipError_t launch_verify_partial_f32(const VerifyArgs &a, const SeqTable &tab, hipStream_t st);
int verify_f32_row_blocks(int R);
// Workgroups per (split, KV head) for R = n_q * (Hq / Hkv) rows.
int verify_mfma_row_blocks(int dtype, int R);
// Its partials use a tiled layout of their own: workspace floats per (split, KV head, block of 64
// rows) unit, and the matching combine pass.
constexpr int kMlFloats = 3;              // per row of a partial: max, sum, output scales of the two stored halves (two bf16)
int64_t verify_mfma_unit_floats_o(int dtype, int head_dim);
int64_t verify_mfma_unit_floats_ml();
// Splits of a sequence whose partials the combine pass can address, of `units` (KV heads x blocks of 64 rows) each.
int verify_mfma_max_splits(int dtype, int head_dim, int64_t units);
hipError_t launch_verify_combine_mfma(int dtype, const VerifyArgs &a, const SeqTable &tab, hipStream_t st);
// Second pass: merge the per-split partials of every (row, head).
hipError_t launch_verify_combine(int dtype, const VerifyArgs &a, const SeqTable &tab,
                                 hipStream_t st);

}  // namespace sparrow
