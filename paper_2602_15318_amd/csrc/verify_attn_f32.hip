// Verification attention in fp32, matrix-core partial pass: head_dim 128 or 64, gfx950.
//
// The fp32 matrix instruction (v_mfma_f32_16x16x4_f32) multiplies and adds in fp32, at 157 TFLOP/s over
// the chip.  One workgroup of 4 wavefronts owns one (context split, KV head, block of 64 kQT rows); a
// row is a (draft row, query head of the group) pair, wavefront w owns rows 16 w .. 16 w + 15 of each of
// its kQT row tiles.  K/V tiles of 32 tokens travel memory -> registers (one step ahead) -> LDS
// (16-byte chunks XOR-swizzled, double buffered, one barrier per tile) -> operands:
//   S^T = K Q^T    A = K (lane: token n, four columns 16 ks + 4 c4 .. +4 by one 16-byte read: four
//                  k-steps of 4), B = Q^T in registers, cut the same way.  A lane then holds, for its
//                  query row, the scores of tokens 4 c4 + 0..3 of each 16-token slab.
//   O^T += V^T P^T B = the scores' own registers (k = c4 <-> token 4 c4 + i), A = V by 4-byte reads.
// Online softmax as in the bf16 kernel (lazy reference point), row sums on the vector ALU, partials in
// fp32 in the layout of its 64-wide heads.
// A tile costs a wavefront 128 matrix instructions of 32 cycles per row tile at d = 128: at 64 rows per
// KV head the matrix cores take 22 us for 26,112 tokens over 4 KV heads, their 107 MB take 17: near
// balance; trees are bound by the matrix cores.  Two workgroups share a compute unit so that one's
// softmax runs under the other's matrix instructions.
// Measured, both passes, against the plain-ALU kernels: 26,112 tokens, 28/4 heads of 128, chain of 8
// 47 (414) us, tree of 60 nodes 236 (3165) us = 93 TFLOP/s; 8,192 tokens, chain of 5 25 (111) us; four
// sequences of 6k, 16/4 heads of 64, chain of 8 25 (114) us; 512 tokens, 4/1 heads of 64 7.7 (13.2) us.
// One output chain over all tokens of a piece instead of one per 16: 1 to 5 % faster, and up to 1.17 times
// the plain-ALU kernels' error on short contexts.
// One workgroup per compute unit instead of two: within 2 %.
#include <algorithm>

#include "common.hpp"
#include "verify_attn.hpp"

namespace sparrow {

namespace {

constexpr int kTile = 32;                 // tokens per tile
constexpr float kSlack = 8.0f;            // log2 units a score may exceed a row's reference point

// Swizzles of the 16-byte chunk index by the token row.  K is read 16 rows at one chunk: rows r .. r+7
// on eight columns of the 256 bytes of a bank line.  V is read four rows (4 c4 + i) x 64 bytes: the rows
// of the four c4 on four columns of 64 bytes.
__device__ __forceinline__ int swz_k(int row) { return (row & 7) << 1; }
__device__ __forceinline__ int swz_v(int row) { return ((row >> 2) & 3) << 2; }

__device__ __forceinline__ float quad_max(float v) {          // over lanes l, l^16, l^32, l^48
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float quad_sum(float v) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <int kD, int kQT>
__global__ void __launch_bounds__(256, 2)
verify_partial_f32_kernel(const void *k_base, const void *v_base, int64_t stride_head, int stride_tok, int cl0_one, int len_one,
                          int ns_one, int piece_one, int n_slots, int rbs, VerifyArgs a, SeqTable tab) {
  constexpr int kRowBytes = 4 * kD, kChunks = kD / 4;      // of a K or V row
  constexpr int kLdRows = 256 / kChunks, kLd = kTile / kLdRows;   // rows of one load of the workgroup, loads
  constexpr int kKS = kD / 16, kMT = kD / 16;              // 16-column groups of a score, 16-wide d-tiles
  constexpr int kTileBytes = kTile * kRowBytes;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];    // [buf][K,V][32 rows]

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, c4 = lane >> 4;
  // row blocks of one split 8 workgroup indices apart: one XCD, whose L2 serves the second fetch
  const int xj = (int)blockIdx.x >> 3, rb = rbs > 1 ? xj % rbs : 0;
  const int slot = (rbs > 1 ? xj / rbs : xj) * 8 + ((int)blockIdx.x & 7);
  if (slot >= n_slots) return;                             // padding of the last round of 8 (uniform)
  const int c = blockIdx.y;
  // one sequence: what the first load needs came with the launch (leading scalars reach the registers), and no row number is
  // divided; chain of 4 over 512 tokens, heads of 64, in a trace 6.3 -> 5.6 us
  int b = 0, cl0 = cl0_one, len = len_one, first = 0, piece = piece_one;
  if (ns_one < n_slots) {
    b = seq_of_slot(tab, slot);
    cl0 = tab.cu_len[b]; len = tab.cu_len[b + 1] - cl0;
    first = tab.cu_split[b];
    piece = split_len(len, tab.cu_split[b + 1] - first);
  }
  const int t0 = min(len, (slot - first) * piece), t1 = min(len, t0 + piece);
  const int n_tiles = (t1 - t0 + kTile - 1) / kTile;
  const int64_t seq_off = (int64_t)cl0 * stride_tok + (int64_t)c * stride_head;
  const unsigned char *Kg = (const unsigned char *)((const float *)k_base + seq_off);
  const unsigned char *Vg = (const unsigned char *)((const float *)v_base + seq_off);
  const unsigned int row_bytes = (unsigned int)stride_tok * 4u;

  // loader: thread -> rows tid / kChunks + kLdRows j, 16-byte chunk tid % kChunks; rows past the end of
  // the split are clamped to its last token (their probability is zero)
  const int ld_row = tid / kChunks, ld_ch = tid % kChunks;
  u32x4 stage[2 * kLd];
  auto issue = [&](int t) {
    const int tb = t0 + t * kTile;
#pragma unroll
    for (int j = 0; j < kLd; ++j) {
      const int r = min(tb + ld_row + kLdRows * j, max(t1 - 1, 0));
      const unsigned int o = (unsigned int)r * row_bytes + (unsigned int)ld_ch * 16u;
      stage[j] = __builtin_nontemporal_load((const u32x4 *)(Kg + o));
      stage[kLd + j] = __builtin_nontemporal_load((const u32x4 *)(Vg + o));
    }
  };
  auto stash = [&](int t, int buf) {
    // values past the end of the split are zero, as in the plain-ALU kernel: a duplicate of an infinite
    // last row would give 0 * inf
    const int left = t1 - (t0 + t * kTile);
    if (left < kTile) {                                    // uniform over the workgroup
#pragma unroll
      for (int j = 0; j < kLd; ++j)
        if (ld_row + kLdRows * j >= left) stage[kLd + j] = (u32x4){0u, 0u, 0u, 0u};
    }
    unsigned char *kb = lds + buf * 2 * kTileBytes, *vb = kb + kTileBytes;
#pragma unroll
    for (int j = 0; j < kLd; ++j) {
      const int r = ld_row + kLdRows * j;
      *reinterpret_cast<u32x4 *>(kb + r * kRowBytes + ((ld_ch ^ swz_k(r)) << 4)) = stage[j];
      *reinterpret_cast<u32x4 *>(vb + r * kRowBytes + ((ld_ch ^ swz_v(r)) << 4)) = stage[kLd + j];
    }
  };
  issue(0);

  const int L = len - a.n_q;
  const int g = a.g, R = a.n_q * g;
  bool row_ok[kQT];
  int i_row[kQT], h[kQT];
  int n_act = 0;                                           // row tiles of this wavefront that hold rows
  u32x4 qreg[kQT][kKS];
  unsigned long long anc[kQT];
#pragma unroll
  for (int qt = 0; qt < kQT; ++qt) {
    const int rho = (rb * kQT + qt) * 64 + 16 * w + n;
    row_ok[qt] = rho < R;
    if ((rb * kQT + qt) * 64 + 16 * w < R) n_act = qt + 1;
    const QuotRest rh = row_and_head(rho, g, a.inv_g);
    i_row[qt] = row_ok[qt] ? rh.quot : 0;
    h[qt] = row_ok[qt] ? c * g + rh.rest : 0;
    // rows past R read row 0 (in bounds) and are zeroed
    const int64_t qrow = row_ok[qt] ? ((int64_t)b * a.n_q + i_row[qt]) * a.Hq + h[qt] : 0;
    const float *qp = (const float *)a.q + qrow * kD + 4 * c4;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) {
      const u32x4 v = *(const u32x4 *)(qp + 16 * ks);
      qreg[qt][ks] = row_ok[qt] ? v : (u32x4){0u, 0u, 0u, 0u};
    }
    // draft rows a row may attend (bit j <=> draft row j); only needed if the split reaches them
    anc[qt] = 0ull;
    if (t1 > L) {                                          // uniform over the workgroup
      anc[qt] = ancestor_mask_wave(a.parent ? a.parent + (int64_t)b * a.parent_stride : nullptr, a.n_q, i_row[qt], lane);
      if (!row_ok[qt]) anc[qt] = 0ull;
    }
  }

  float m_run[kQT], l_run[kQT];
  f32x4 o_acc[kQT][kMT];
#pragma unroll
  for (int qt = 0; qt < kQT; ++qt) {
    m_run[qt] = kNegBig;
    l_run[qt] = 0.f;
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt) o_acc[qt][mt] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }

  auto compute = [&](int t, int buf) {
    const unsigned char *Ks = lds + buf * 2 * kTileBytes, *Vs = Ks + kTileBytes;
    const int tb = t0 + t * kTile;
    f32x4 s[kQT][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int qt = 0; qt < kQT; ++qt) s[qt][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks) {
        const u32x4 ka = *reinterpret_cast<const u32x4 *>(Ks + (16 * j + n) * kRowBytes + (((4 * ks + c4) ^ swz_k(n)) << 4));
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int qt = 0; qt < kQT; ++qt)
            s[qt][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(ka[e]), __uint_as_float(qreg[qt][ks][e]), s[qt][j], 0, 0, 0);
      }
    }
    const bool edge = tb + kTile > min(t1, L);             // uniform: split end or draft rows in reach
#pragma unroll
    for (int qt = 0; qt < kQT; ++qt) {
      if (edge) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int tok = tb + 16 * j + 4 * c4 + i, dj = tok - L;
            const bool vis = (dj < 0) | (((anc[qt] >> (dj & 63)) & 1ull) != 0ull);
            s[qt][j][i] = ((tok < t1) & vis) ? s[qt][j][i] : -INFINITY;
          }
      }
      float mx = s[qt][0][0];
#pragma unroll
      for (int e = 1; e < 8; ++e) mx = fmaxf(mx, s[qt][e >> 2][e & 3]);
      mx *= a.scale_log2;
      if (__builtin_amdgcn_ballot_w64(mx > m_run[qt] + kSlack) != 0ull) {
        const float m_new = fmaxf(m_run[qt], quad_max(mx));
        const float alpha = fast_exp2(m_run[qt] - m_new);
        m_run[qt] = m_new;
        l_run[qt] *= alpha;
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt) o_acc[qt][mt] *= alpha;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) s[qt][e >> 2][e & 3] = fast_exp2(fmaf(s[qt][e >> 2][e & 3], a.scale_log2, -m_run[qt]));
      const f32x4 p4 = s[qt][0] + s[qt][1];
      l_run[qt] += (p4[0] + p4[1]) + (p4[2] + p4[3]);
    }
    // 16 tokens are added up from zero and then to the running output: chains of 16 roundings and of one
    // per 16 tokens instead of one over all tokens of the piece
    constexpr int kX = 2 / kQT;                            // d-tiles side by side: two chains are in flight
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int mt = 0; mt < kMT; mt += kX) {
        if (kD * kQT > 128 && mt == 0) __builtin_amdgcn_sched_barrier(0);   // (V reads further ahead spill registers)
        f32x4 part[kQT][kX];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 16 * j + 4 * c4 + i;
          const unsigned char *vr = Vs + r * kRowBytes + ((n & 3) << 2);
#pragma unroll
          for (int x = 0; x < kX; ++x) {
            const float va = *reinterpret_cast<const float *>(vr + (((4 * (mt + x) + (n >> 2)) ^ swz_v(r)) << 4));
#pragma unroll
            for (int qt = 0; qt < kQT; ++qt) {
              if (i == 0) part[qt][x] = (f32x4){0.f, 0.f, 0.f, 0.f};
              part[qt][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(va, s[qt][j][i], part[qt][x], 0, 0, 0);
            }
          }
        }
#pragma unroll
        for (int qt = 0; qt < kQT; ++qt)
#pragma unroll
          for (int x = 0; x < kX; ++x) o_acc[qt][mt + x] += part[qt][x];
      }
  };

  // double buffered: a wavefront may write tile t + 1 while others still read tile t, and reaches tile
  // t + 2's writes only after the barrier of tile t + 1, behind which tile t has been read by all
  for (int t = 0; t < n_tiles; ++t) {
    stash(t, t & 1);
    issue(min(t + 1, n_tiles - 1));
    __syncthreads();
    if (n_act > 0) compute(t, t & 1);
  }

  const int rbs64 = (R + 63) / 64;
#pragma unroll
  for (int qt = 0; qt < kQT; ++qt) {
    if (qt >= n_act) break;
    const float l_tot = quad_sum(l_run[qt]);
    const float inv_l = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    if (a.direct) {                                        // the split is the whole sequence
      if (!row_ok[qt]) continue;
      const int64_t orow = ((int64_t)b * a.n_q + i_row[qt]) * a.Hq + h[qt];
      float *out = (float *)a.out + orow * kD + 4 * c4;
#pragma unroll
      for (int mt = 0; mt < kMT; ++mt) *reinterpret_cast<f32x4 *>(out + 16 * mt) = o_acc[qt][mt] * inv_l;
      if (a.lse != nullptr && c4 == 0) a.lse[orow] = lse_of<true>(m_run[qt], l_tot);
      continue;
    }
    const int64_t unit = ((int64_t)slot * a.Hkv + c) * rbs64 + rb * kQT + qt;
    f32x4 *po = reinterpret_cast<f32x4 *>(a.part_o) + (unit * 4 + w) * (kMT * 64) + lane;
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt) __builtin_nontemporal_store(o_acc[qt][mt] * inv_l, &po[mt * 64]);
    if (c4 == 0) {
      float *pml = a.part_ml + (unit * 64 + 16 * w + n) * kMlFloats;
      __builtin_nontemporal_store(m_run[qt], &pml[0]);
      __builtin_nontemporal_store(l_tot, &pml[1]);
    }
  }
}

template <int kD, int kQT>
hipError_t launch_f32(const VerifyArgs &a, const SeqTable &tab, int rbs, hipStream_t st) {
  constexpr int lds = 2 * 2 * kTile * kD * 4;
  static_assert(lds <= 64 * 1024, "beyond 64 KB the kernel needs the dynamic-LDS attribute");
  const dim3 grid((a.n_slots + 7) / 8 * 8 * rbs, a.Hkv);
  hipLaunchKernelGGL((verify_partial_f32_kernel<kD, kQT>), grid, dim3(256), lds, st, a.k, a.v, a.stride_head, (int)a.stride_tok,
                     (int)tab.cu_len[0], (int)(tab.cu_len[1] - tab.cu_len[0]), (int)tab.cu_split[1],
                     split_len(tab.cu_len[1] - tab.cu_len[0], tab.cu_split[1]), a.n_slots, rbs, a, tab);
  return hipGetLastError();
}

}  // namespace

// Blocks of 64 rows, or of 128 (the K and V operands read from LDS then feed two row tiles).
int verify_f32_row_blocks(int R) { return R <= 64 ? 1 : (R + 127) / 128; }

hipError_t launch_verify_partial_f32(const VerifyArgs &a, const SeqTable &tab, hipStream_t st) {
  const int R = a.n_q * (a.Hq / a.Hkv), rbs = verify_f32_row_blocks(R);
  if (a.d == 128) return R <= 64 ? launch_f32<128, 1>(a, tab, rbs, st) : launch_f32<128, 2>(a, tab, rbs, st);
  return R <= 64 ? launch_f32<64, 1>(a, tab, rbs, st) : launch_f32<64, 2>(a, tab, rbs, st);
}

}  // namespace sparrow
