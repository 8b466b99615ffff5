// Input side of the draft model for any hidden size (a multiple of 8), bf16: the hidden-state-reuse
// projection (Eq. 1) and the draft layer's RMSNorm / QKV / rotary step with the K/V append.  gfx950.
// Hidden sizes of 7 and 8 whole slices of 512 have kernels of their own (hsr_input.hip), in which the
// number of slices is a compile-time constant and no column needs a check: QKV of 2 to 8 rows takes 12.3 to 12.9 us at
// 3,584 there and 17.2 to 18.6 here, at 4,096 14.7 to 15.3 and 18.9 to 20.5; FC of 6 rows at 3,584 11.1 and 12.3.
//
// Both steps are skinny GEMMs (at most 64 activation rows), bound by the weight stream:
//   - one workgroup per tile of 16 weight rows (grid.y = blocks of 16 activation rows);
//   - a weight row is cut into slices of 512 elements (1 KB; the last one may be short: columns past
//     its end read as zero by the bounds check of the buffer loads); wavefront w owns the slices w,
//     w + nw, ...: every load instruction reads the slice of one weight row, 16 loads in flight,
//     staged through a private, XOR-swizzled 16 KB LDS buffer into the A operand of
//     v_mfma_f32_16x16x32_bf16; the B operand is the wavefront's slice of the activation rows, held
//     in registers;
//   - the partial sums of the wavefronts meet in LDS and wavefront 0 runs the epilogue.
// For the QKV step the tile's 16 weight rows are features f..f+7 and f+d/2..f+d/2+7 of one head,
// so both halves of every rotary pair sit in the same tile (lanes l and l^32 of the result);
// RMSNorm is folded in: the activations enter the B operand multiplied by gamma, exactly, as the sum of two
// bf16 terms (the product has up to 16 bits), and the row's 1/rms (from the squares each wavefront
// sees in its own slices) scales the result.
// One activation row (QKV: also two of up to 1,024 columns) runs a wavefront per output feature or rotary
// pair instead (QKV: at every width), two to four rows of FC a wavefront per two features.
//
// Measured (FC + QKV, weights from memory; one plain-ALU wavefront per feature before): hidden 2,560, 40/8 heads of 64,
// six rows 141 + 67 -> 8.5 + 7.7 us, one row 56 + 22 -> 8.1 + 6.2; hidden 5,120, 40/8 heads of 128, 16 rows 823 + 447 ->
// 38.1 + 34.7 us; hidden 1,024, 16/4 heads of 64, six rows 36 + 21 -> 5.3 + 6.3.
#include <algorithm>

#include "common.hpp"
#include "hsr_input.hpp"

namespace sparrow {

namespace {

constexpr int kSlice = 512;               // k elements per wavefront slice (1 KB of bf16)

constexpr int kMaxWaves = 8;              // wavefronts of a workgroup (16 KB of staging each)
constexpr unsigned int kPastEnd = 0x80000000u;   // a buffer offset that reads as zero

__device__ __forceinline__ __amdgpu_buffer_rsrc_t weight_rows(const bf16_t *first) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)first, (short)0, (int)0x7fffffff, 0x00027000);
}

// An activation times its gamma, u, is the sum of two bf16 terms: hi, its leading 8 bits (cut off), and this, the other 8.
// Where they are zero, 2^-40 of u with its sign: an infinite weight then gives an infinity, and no 0 * inf.  (u - hi is
// zero or larger than u * 2^-40 in magnitude, so the one in the middle is meant; of an infinite u both terms are
// infinite, where u - hi is NaN and the smaller of the other two is taken.)  Against 2^-40 added to u - hi, which was
// NaN there: two to sixteen rows of 256 to 5,120 columns 0.5 to 2 % slower.
__device__ __forceinline__ float low_term(float u, float hi) { return __builtin_amdgcn_fmed3f(u - hi, u * 0x1p-40f, u); }

// ---------------------------------------------------------------------------------------------
// shared main loop over a tile of 16 weight rows.  Wavefront 0 gets D[4*c4 + i][n] = sum over K of
// W[wrow(4*c4 + i)][k] * x[row0 + n][k], lane = n + 16*c4, and (kNorm) the sum of x[row0 + n][k]^2, and
// runs epi(D, sum).  xload(m, k, ok): 8 consecutive bf16 of activation row m at column k (k % 8 == 0),
// zeros if !ok.  With the norm folded in, the activations of a slice are taken in two halves of 256
// columns: their two terms fill 64 registers per half beside the 64 of the weights in flight.
// kFew (norm folded in, at most 8 rows): lanes n and n ^ 8 share row n & 7 and hold one half of a slice's columns each, so
// that a whole slice takes 64 registers and half the arithmetic.  A matrix instruction's 16 columns then meet weights of
// one half: columns below 8 are right where they are the first half's, the others where they are the second half's; two
// sums, added at the end.  The registers left allow a slice's activations to be asked for before its weights (behind them,
// in two halves one after the other, came a second round trip).  Their arithmetic, half of what it was, still runs after
// the wait for the weights: nothing keeps the compiler from moving it there, to its first use.  Before / now, us: 2,560
// columns, 40/8 heads of 64, six rows 10.8 / 9.4; 5,120, 40/8 of 128, two rows 31.9 / 24.5, eight 32.4 / 26.7; 1,536, 24/4
// of 64, five 7.55 / 6.95; 256, 4/1 of 64, three 6.1 / 5.2.
// ---------------------------------------------------------------------------------------------
template <bool kNorm, bool kFew, class WRow, class XLoad, class Epi>
__device__ __forceinline__ void skinny_gemm(const bf16_t *W, int K, WRow wrow, XLoad xload, const bf16_t *gamma,
                                            int row0, int M, unsigned char *smem, Epi epi) {
  constexpr int kPart = kNorm ? 8 : 16;                      // k-steps of 32 fetched together
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = (int)blockDim.x >> 6;
  const int n = lane & 15, c4 = lane >> 4;
  const int n_slices = (K + kSlice - 1) / kSlice;
  unsigned char *stg = smem + w * 16384;
  f32x4 *red = reinterpret_cast<f32x4 *>(smem + nw * 16384);                        // [nw][64]
  float *ssq_lds = reinterpret_cast<float *>(smem + nw * 16384 + nw * 1024);        // [nw][16]

  u32x4 buf[16];
  auto issue = [&](int s) {
    const int first = wrow(0);
    const __amdgpu_buffer_rsrc_t rs = weight_rows(W + (int64_t)first * K);
    const int k = kSlice * s + 8 * lane;
    const unsigned int off = k < K ? (unsigned int)k * 2u : kPastEnd;
#pragma unroll
    for (int r = 0; r < 16; ++r)
      buf[r] = __builtin_amdgcn_raw_buffer_load_b128(rs, off, (wrow(r) - first) * K * 2, 2);
  };
  static_assert(kNorm || !kFew, "the plain product has no registers to save");
  const int m = row0 + (kFew ? n & 7 : n);
  const bool m_ok = m < M;
  const __amdgpu_buffer_rsrc_t rs_g = weight_rows(gamma);
  float ssq = 0.f;
  u32x4 xr[kPart], gr[kNorm ? kPart : 1];
  auto load_x = [&](int k0, u32x4 *xr, u32x4 *gr) {
#pragma unroll
    for (int ks = 0; ks < kPart; ++ks) {
      const int k = k0 + 32 * ks + 8 * c4 + (kFew ? 256 * (n >> 3) : 0);
      xr[ks] = xload(m, k, m_ok && k < K);
      if (kNorm) gr[ks] = __builtin_amdgcn_raw_buffer_load_b128(rs_g, k < K ? (unsigned int)k * 2u : kPastEnd, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // activations times gamma, in place: xr the leading terms, gr the others
  auto convert = [&]() {
#pragma unroll
    for (int ks = 0; ks < kPart; ++ks) {
      float xf[8], gf[8], lo[8];
      unsigned int hb[8];
      Elem<bf16_t>::unpack(xr[ks], xf);
      Elem<bf16_t>::unpack(gr[kNorm ? ks : 0], gf);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        ssq = fmaf(xf[e], xf[e], ssq);
        const float u = xf[e] * gf[e];
        hb[e] = __float_as_uint(u) & 0xffff0000u;
        lo[e] = low_term(u, __uint_as_float(hb[e]));
      }
      xr[ks] = (u32x4){(hb[0] >> 16) | hb[1], (hb[2] >> 16) | hb[3], (hb[4] >> 16) | hb[5], (hb[6] >> 16) | hb[7]};
      gr[kNorm ? ks : 0] = (u32x4){pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]),
                                   pack_bf16x2(lo[4], lo[5]), pack_bf16x2(lo[6], lo[7])};
      // one k-step at a time: unpacked, all of them would need as many registers as the kernel has
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  const int a_base = n * 1024;            // A read: tile row n, 16-byte chunk 4*ks + c4
  auto mul = [&](int part) {
#pragma unroll
    for (int kh = 0; kh < kPart; kh += 2) {
      const int ch0 = 4 * (part * kPart + kh) + c4, ch1 = ch0 + 4;
      const bf16x8 a0 = *reinterpret_cast<const bf16x8 *>(stg + a_base + (((ch0 & ~15) | ((ch0 & 15) ^ n)) << 4));
      const bf16x8 a1 = *reinterpret_cast<const bf16x8 *>(stg + a_base + (((ch1 & ~15) | ((ch1 & 15) ^ n)) << 4));
      acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, __builtin_bit_cast(bf16x8, xr[kh]), acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, __builtin_bit_cast(bf16x8, xr[kh + 1]), acc[1], 0, 0, 0);
      if (kNorm) {
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, __builtin_bit_cast(bf16x8, gr[kNorm ? kh : 0]), acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, __builtin_bit_cast(bf16x8, gr[kNorm ? kh + 1 : 0]), acc[1], 0, 0, 0);
      }
    }
  };

  // lane l of load r holds chunk l of row r; stored at chunk (l & ~15) | ((l & 15) ^ r) so that
  // the A reads (16 rows, same chunk) spread over all banks
  auto stash = [&]() {
#pragma unroll
    for (int r = 0; r < 16; ++r)
      *reinterpret_cast<u32x4 *>(stg + r * 1024 + (((lane & ~15) | ((lane & 15) ^ r)) << 4)) = buf[r];
  };
  if constexpr (kFew) {
    u32x4 xn[kPart], gn[kPart];
    load_x(kSlice * w, xr, gr);
    issue(w);
    for (int s = w; s < n_slices; s += nw) {
      convert();
      stash();
      if (s + nw < n_slices) {
        load_x(kSlice * (s + nw), xn, gn);
        issue(s + nw);
      }
#pragma unroll
      for (int kh = 0; kh < kPart; ++kh) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {                        // the weights of columns 256 h + 32 kh ...
          const int ch = 4 * (8 * h + kh) + c4;
          const bf16x8 a = *reinterpret_cast<const bf16x8 *>(stg + a_base + (((ch & ~15) | ((ch & 15) ^ n)) << 4));
          acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, xr[kh]), acc[h], 0, 0, 0);
          acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, gr[kh]), acc[h], 0, 0, 0);
        }
      }
#pragma unroll
      for (int ks = 0; ks < kPart; ++ks) { xr[ks] = xn[ks]; gr[ks] = gn[ks]; }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[1][e] = lane_xor<8>(acc[1][e], lane);
    ssq += lane_xor<8>(ssq, lane);
  } else {
    issue(w);                             // (nw <= n_slices: every wavefront has a slice)
    for (int s = w; s < n_slices; s += nw) {
      load_x(kSlice * s, xr, gr);
      stash();
      if (s + nw < n_slices) issue(s + nw);
      if (kNorm) convert();
      mul(0);
      if (kNorm) {
        load_x(kSlice * s + 256, xr, gr);
        convert();
        mul(1);
      }
    }
  }
  red[w * 64 + lane] = acc[0] + acc[1];
  if (kNorm) {
    ssq += lane_xor<16>(ssq, lane);
    ssq += lane_xor<32>(ssq, lane);       // all four k-chunk lanes of row n now hold the slices' sum
    if (c4 == 0) ssq_lds[w * 16 + n] = ssq;
  }
  __syncthreads();
  if (w == 0) {
    float s2 = 0.f;
    if (kNorm)
      for (int ww = 0; ww < nw; ++ww) s2 += ssq_lds[ww * 16 + n];
    f32x4 sum = red[lane];
    for (int ww = 1; ww < nw; ++ww) sum += red[ww * 64 + lane];
    epi(sum, s2);
  }
}

constexpr int skinny_lds_bytes(int nw) { return nw * 16384 + nw * 1024 + nw * 64; }

// ---------------------------------------------------------------------------------------------
// Eq. 1: z = FC(e (+) h)
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kMaxWaves * 64)
hsr_fc_any_kernel(HsrFcArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tile = blockIdx.x, row0 = blockIdx.y * 16;
  const int H = a.H;
  const bf16_t *E = (const bf16_t *)a.embed, *Hp = (const bf16_t *)a.h_prev;
  const int lane = threadIdx.x & 63, n = lane & 15, c4 = lane >> 4;
  // the token id of this lane's activation row (clamped into the table)
  const int m = row0 + n;
  int tok = m < a.M ? a.token_ids[m] : 0;
  tok = min(max(tok, 0), a.vocab - 1);
  auto wrow = [&](int r) { return min(tile * 16 + r, H - 1); };    // (the last tile may be half empty)
  // eight columns lie entirely in one half of the concatenation (H is a multiple of 8)
  auto xload = [&](int mm, int k, bool ok) -> u32x4 {
    const int kk = ok ? k : 0, mr = ok ? mm : 0;
    const u32x4 v = *(const u32x4 *)(kk < H ? E + (int64_t)tok * H + kk : Hp + (int64_t)mr * H + (kk - H));
    return ok ? v : (u32x4){0u, 0u, 0u, 0u};
  };
  const int f = tile * 16 + 4 * c4;
  u32x2 bw = {0u, 0u};                    // fetched ahead of the weight stream
  if (a.bias != nullptr && f < H) bw = *(const u32x2 *)((const bf16_t *)a.bias + f);
  auto epi = [&](f32x4 r, float) {
    if (m >= a.M || f >= H) return;
    const u32x2 o = {pack_bf16x2(r[0] + bf16lo_to_f32(bw.x), r[1] + bf16hi_to_f32(bw.x)),
                     pack_bf16x2(r[2] + bf16lo_to_f32(bw.y), r[3] + bf16hi_to_f32(bw.y))};
    *(u32x2 *)((bf16_t *)a.z + (int64_t)m * H + f) = o;
  };
  skinny_gemm<false, false>((const bf16_t *)a.w, 2 * H, wrow, xload, nullptr, row0, a.M, smem, epi);
}

// ---------------------------------------------------------------------------------------------
// draft layer input: RMSNorm, QKV, rotary embedding, scatter
// ---------------------------------------------------------------------------------------------
template <bool kFew>
__global__ void __launch_bounds__(kMaxWaves * 64)
draft_qkv_any_kernel(DraftQkvArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int row0 = blockIdx.y * 16;
  const int H = a.H, d = a.d, half = d >> 1;
  const int tiles_per_head = d >> 4;
  const int lane = threadIdx.x & 63, n = lane & 15, c4 = lane >> 4;
  const int m = row0 + n;
  const bool m_ok = m < a.M;
  // tile -> (head, group j of 8 features); tile row r: feature 8j + (r & 7) of the head's first
  // half for r < 8, its rotary partner (+ d/2) for r >= 8
  const int hd = (int)blockIdx.x / tiles_per_head, j = (int)blockIdx.x - hd * tiles_per_head;
  auto wrow = [&](int r) { return hd * d + 8 * j + (r & 7) + (r >> 3) * half; };
  const __amdgpu_buffer_rsrc_t rs_z = weight_rows((const bf16_t *)a.z);       // at most 64 rows
  auto xload = [&](int mm, int k, bool ok) -> u32x4 {
    return __builtin_amdgcn_raw_buffer_load_b128(rs_z, ok ? (unsigned int)(mm * H + k) * 2u : kPastEnd, 0, 0);
  };
  // lane (n, c4), entry i of a tile's result: tile row 4*c4 + i -> feature f0 + i of half `hi`
  const int hi = c4 >> 1;
  // epilogue operands, fetched ahead of the weight stream: bias, the token's rotary row, its
  // cache row (the table is a kernel argument, read with uniform indices)
  const int f0 = 8 * j + 4 * (c4 & 1);
  u32x2 bw = {0u, 0u};
  if (a.bias != nullptr) bw = *(const u32x2 *)((const bf16_t *)a.bias + hd * d + hi * half + f0);
  const f32x4 cs = *(const f32x4 *)(a.rope_cos + (int64_t)(m_ok ? m : 0) * half + f0);
  const f32x4 sn = *(const f32x4 *)(a.rope_sin + (int64_t)(m_ok ? m : 0) * half + f0);
  int kv_row = 0;
#pragma unroll
  for (int mm = 0; mm < 16; ++mm) {
    const int r = a.kv_rows[min(row0 + mm, kHsrMaxRows - 1)];
    if (n == mm) kv_row = r;
  }
  auto epi = [&](f32x4 res, float ssq) {
    const float rstd = 1.0f / sqrtf(ssq / (float)H + a.eps);
    const float b[4] = {bf16lo_to_f32(bw.x), bf16hi_to_f32(bw.x),
                        bf16lo_to_f32(bw.y), bf16hi_to_f32(bw.y)};
    const bool is_v = hd >= a.Hq + a.Hkv;
    float o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float y = fmaf(res[i], rstd, b[i]);
      const float partner = lane_xor<32>(y, lane);      // the other half of the rotary pair
      o[i] = y;
      if (!is_v) o[i] = hi ? fmaf(partner, sn[i], y * cs[i]) : fmaf(-partner, sn[i], y * cs[i]);
    }
    if (!m_ok) return;
    const u32x2 ow = {pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
    const int feat = hi * half + f0;
    if (hd < a.Hq) {
      *(u32x2 *)((bf16_t *)a.q_out + ((int64_t)m * a.Hq + hd) * d + feat) = ow;
    } else {
      const int c = is_v ? hd - a.Hq - a.Hkv : hd - a.Hq;
      bf16_t *base = (bf16_t *)(is_v ? a.v_cache : a.k_cache);
      *(u32x2 *)(base + (int64_t)kv_row * a.stride_tok + (int64_t)c * a.stride_head + feat) = ow;
    }
  };
  skinny_gemm<true, kFew>((const bf16_t *)a.w, H, wrow, xload, (const bf16_t *)a.gamma, row0, a.M, smem, epi);
}

// ---------------------------------------------------------------------------------------------
// Few activation rows (at most 8) whose weights are all on their way at once: a wavefront per slice of kCols columns, one
// slice each, and as many weight rows per workgroup (at most 16) as give every compute unit the same number.  skinny_gemm
// brings the slices in rounds (10 of 5,120 columns by 5 wavefronts), deals whole tiles of 16 rows (160 workgroups for 2,560
// features, 320 in two rounds for 5,120) and, for QKV, makes the activations' terms behind the weights, on five wavefronts of
// which two share a SIMD; slices of 256 columns halve what a wavefront makes, and the empty statements keep it under the
// weights' flight.  us, skinny_gemm / here: FC of 6 rows, 2,560 columns 10.0 / 8.5, 5 of 1,536 6.75 / 5.7, 8 of 2,048 8.55 /
// 7.6, 5 of 3,072 11.7 / 10.05; QKV of 6 rows, 2,560 columns, 40/8 heads of 64 9.25 / 7.7, 2 of it 9.2 / 7.6, 5 of 3,072,
// 24/8 of 128 17.1 / 12.9, 3 of 256, 4/1 of 64 5.6 / 4.4.  QKV with slices of 512: 9.0 (223 registers).
// ---------------------------------------------------------------------------------------------
constexpr int kOnceWaves = 16;

// Rows per workgroup for n rows (or pairs), at most `most`: a whole number of workgroups per compute unit, all of one size.
inline int even_rows(int n, int most) {
  const int per_cu = (n + 256 * most - 1) / (256 * most);
  return (n + 256 * per_cu - 1) / (256 * per_cu);
}
constexpr int once_lds_bytes(int nw, int rows, int cols) { return nw * rows * cols * 2 + nw * 1024 + nw * 64; }

// Wavefront 0 runs epi(D, sum): as skinny_gemm's, lane n + 16 c4 with n < 8 has the results of activation row n and weight rows
// 4 c4 + i.  rows: how many are fetched (the others of 16 read as zero and cost no memory), stg_rows: at least that;
// at(r): element offset of fetched row r (uniform); staged(x): the fetched row that is row x of the product (any row in range
// where the result is not used).  The activations of a slice of kCols columns are shared out as in skinny_gemm's kFew.
// Operands of the end come in by more(), called when the weights have been asked for.
template <bool kNorm, int kCols, class At, class Staged, class XLoad, class More, class Epi>
__device__ __forceinline__ void skinny_once(const bf16_t *W, int K, int rows, int stg_rows, At at, Staged staged, XLoad xload,
                                            const bf16_t *gamma, int M, unsigned char *smem, More more, Epi epi) {
  constexpr int kPerLoad = 512 / kCols, kLoads = 16 / kPerLoad, kLanes = 64 / kPerLoad;      // rows of a load, loads, lanes of a row
  constexpr int kX = kCols / 64, kBytes = 2 * kCols;                                         // activation k-steps of a lane
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = (int)blockDim.x >> 6;
  const int n = lane & 15, c4 = lane >> 4;
  unsigned char *stg = smem + w * stg_rows * kBytes;
  f32x4 *red = reinterpret_cast<f32x4 *>(smem + nw * stg_rows * kBytes);                     // [nw][64]
  float *ssq_lds = reinterpret_cast<float *>(smem + nw * stg_rows * kBytes + nw * 1024);     // [nw][16]
  const int m = n & 7;
  const bool m_ok = m < M;
  u32x4 buf[kLoads], xr[kX], gr[kNorm ? kX : 1];
  const int sub = lane / kLanes, ld_ch = lane % kLanes;    // row of a load, 16-byte chunk of it
  auto issue = [&]() __attribute__((always_inline)) {
    const int64_t first = at(0);
    const __amdgpu_buffer_rsrc_t rs = weight_rows(W + first);
    const int k = kCols * w + 8 * ld_ch;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int r0 = i * kPerLoad, r1 = r0 + kPerLoad - 1;
      const unsigned int o0 = r0 < rows ? (unsigned int)((at(r0) - first) * 2) : kPastEnd;
      const unsigned int o1 = r1 < rows ? (unsigned int)((at(r1) - first) * 2) : kPastEnd;
      const unsigned int o = sub ? o1 : o0;
      buf[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, k < K && o != kPastEnd ? o + (unsigned int)k * 2u : kPastEnd, 0, 2);
    }
  };
  auto load_x = [&]() __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs_g = weight_rows(gamma);
#pragma unroll
    for (int ks = 0; ks < kX; ++ks) {
      const int k = kCols * w + 32 * ks + 8 * c4 + kCols / 2 * (n >> 3);
      xr[ks] = xload(m, k, m_ok && k < K);
      if (kNorm) gr[ks] = __builtin_amdgcn_raw_buffer_load_b128(rs_g, k < K ? (unsigned int)k * 2u : kPastEnd, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  float ssq = 0.f;
  if (kNorm) {                            // activations first: their terms are made under the weights' flight
    load_x();
    issue();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < kX; ++ks) {
      float xf[8], gf[8], lo[8];
      unsigned int hb[8];
      Elem<bf16_t>::unpack(xr[ks], xf);
      Elem<bf16_t>::unpack(gr[kNorm ? ks : 0], gf);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        ssq = fmaf(xf[e], xf[e], ssq);
        const float u = xf[e] * gf[e];
        hb[e] = __float_as_uint(u) & 0xffff0000u;
        lo[e] = low_term(u, __uint_as_float(hb[e]));
      }
      xr[ks] = (u32x4){(hb[0] >> 16) | hb[1], (hb[2] >> 16) | hb[3], (hb[4] >> 16) | hb[5], (hb[6] >> 16) | hb[7]};
      gr[kNorm ? ks : 0] = (u32x4){pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]), pack_bf16x2(lo[4], lo[5]), pack_bf16x2(lo[6], lo[7])};
      asm volatile("" : "+v"(xr[ks]), "+v"(gr[kNorm ? ks : 0]));     // here, and not where it is used, behind the weights
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {                                // weights first: the activations' addresses wait for the token ids
    issue();
    __builtin_amdgcn_sched_barrier(0);
    load_x();
  }
  if (w == 0) more();
#pragma unroll
  for (int i = 0; i < kLoads; ++i) {
    const int r = i * kPerLoad + sub;
    if (r < rows) *reinterpret_cast<u32x4 *>(stg + r * kBytes + (((ld_ch & ~15) | ((ld_ch & 15) ^ r)) << 4)) = buf[i];
  }
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  const int nr = staged(n);
#pragma unroll
  for (int kh = 0; kh < kX; ++kh)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int ch = 4 * (kX * h + kh) + c4;
      const bf16x8 a = *reinterpret_cast<const bf16x8 *>(stg + nr * kBytes + (((ch & ~15) | ((ch & 15) ^ nr)) << 4));
      acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, xr[kh]), acc[h], 0, 0, 0);
      if (kNorm) acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, gr[kNorm ? kh : 0]), acc[h], 0, 0, 0);
    }
#pragma unroll
  for (int e = 0; e < 4; ++e) acc[1][e] = lane_xor<8>(acc[1][e], lane);
  red[w * 64 + lane] = acc[0] + acc[1];
  if (kNorm) {
    ssq += lane_xor<8>(ssq, lane);
    ssq += lane_xor<16>(ssq, lane);
    ssq += lane_xor<32>(ssq, lane);
    if (c4 == 0) ssq_lds[w * 16 + n] = ssq;
  }
  __syncthreads();
  if (w != 0) return;
  float s2 = 0.f;
  if (kNorm)
    for (int ww = 0; ww < nw; ++ww) s2 += ssq_lds[ww * 16 + n];
  f32x4 sum = red[lane];
  for (int ww = 1; ww < nw; ++ww) sum += red[ww * 64 + lane];
  epi(sum, s2);
}

// Eq. 1, five to eight rows
__global__ void __launch_bounds__(kOnceWaves * 64)
hsr_fc_once_kernel(HsrFcArgs a, int rows) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int H = a.H, f_tile = (int)blockIdx.x * rows;
  const bf16_t *E = (const bf16_t *)a.embed, *Hp = (const bf16_t *)a.h_prev;
  const int lane = threadIdx.x & 63, n = lane & 15, c4 = lane >> 4;
  int tok = (n & 7) < a.M ? a.token_ids[n & 7] : 0;
  tok = min(max(tok, 0), a.vocab - 1);
  auto at = [&](int r) { return (int64_t)(f_tile + r) * (2 * H); };
  auto xload = [&](int mm, int k, bool ok) -> u32x4 {          // eight columns lie in one half of the concatenation
    const int kk = ok ? k : 0, mr = ok ? mm : 0;
    const u32x4 v = *(const u32x4 *)(kk < H ? E + (int64_t)tok * H + kk : Hp + (int64_t)mr * H + (kk - H));
    return ok ? v : (u32x4){0u, 0u, 0u, 0u};
  };
  const int left = min(rows, H - f_tile);                      // rows of this workgroup (even, as H and rows are)
  unsigned int bw[2] = {0u, 0u};
  auto more = [&]() {
    if (a.bias == nullptr) return;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (4 * c4 + 2 * i < left) bw[i] = *(const unsigned int *)((const bf16_t *)a.bias + f_tile + 4 * c4 + 2 * i);
  };
  auto epi = [&](f32x4 r, float) {
    if (n >= a.M) return;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (4 * c4 + 2 * i < left)
        *(unsigned int *)((bf16_t *)a.z + (int64_t)n * H + f_tile + 4 * c4 + 2 * i) =
            pack_bf16x2(r[2 * i] + bf16lo_to_f32(bw[i]), r[2 * i + 1] + bf16hi_to_f32(bw[i]));
  };
  auto staged = [&](int x) { return min(x, left - 1); };
  skinny_once<false, 512>((const bf16_t *)a.w, 2 * H, left, rows, at, staged, xload, nullptr, a.M, smem, more, epi);
}

// Draft layer input, two to eight rows: `pairs` rotary pairs per workgroup, numbered through the heads; weight row j of a tile
// is pair j's first feature, row 8 + j its second, so that both sit in lanes l and l ^ 32 of the result.
__global__ void __launch_bounds__(kOnceWaves * 64)
draft_qkv_once_kernel(DraftQkvArgs a, int pairs) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int H = a.H, d = a.d, half = d >> 1, sh = d == 128 ? 6 : 5;
  const int n_pairs = (a.Hq + 2 * a.Hkv) * half, p_tile = (int)blockIdx.x * pairs;
  const int lane = threadIdx.x & 63, n = lane & 15, c4 = lane >> 4, hi = c4 >> 1;
  const int left = min(pairs, n_pairs - p_tile);
  auto at = [&](int r) {
    const int second = r >= pairs, p = p_tile + min(r - (second ? pairs : 0), left - 1);
    return (int64_t)((p >> sh) * d + (p & (half - 1)) + (second ? half : 0)) * H;
  };
  auto staged = [&](int x) { return (x >> 3) * pairs + min(x & 7, pairs - 1); };
  const __amdgpu_buffer_rsrc_t rs_z = weight_rows((const bf16_t *)a.z);
  auto xload = [&](int mm, int k, bool ok) -> u32x4 {
    return __builtin_amdgcn_raw_buffer_load_b128(rs_z, ok ? (unsigned int)(mm * H + k) * 2u : kPastEnd, 0, 0);
  };
  const bool m_ok = n < a.M;
  bf16_t b[4] = {0, 0, 0, 0};
  float cs[4], sn[4];
  auto more = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = p_tile + min(4 * (c4 & 1) + i, left - 1), f = p & (half - 1);
      if (a.bias != nullptr) b[i] = ((const bf16_t *)a.bias)[(p >> sh) * d + hi * half + f];
      cs[i] = a.rope_cos[(m_ok ? n : 0) * half + f];
      sn[i] = a.rope_sin[(m_ok ? n : 0) * half + f];
    }
  };
  auto epi = [&](f32x4 res, float ssq) {
    const float rstd = 1.0f / sqrtf(ssq / (float)H + a.eps);
    int kv_row = 0;
#pragma unroll
    for (int mm = 0; mm < 8; ++mm) {
      const int r = a.kv_rows[mm];
      if (n == mm) kv_row = r;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = 4 * (c4 & 1) + i, p = p_tile + min(j, left - 1), hd = p >> sh, feat = hi * half + (p & (half - 1));
      const float y = fmaf(res[i], rstd, bf16_to_f32(b[i]));
      const float partner = lane_xor<32>(y, lane);      // the other half of the rotary pair
      const bool is_v = hd >= a.Hq + a.Hkv;
      const float o = is_v ? y : hi ? fmaf(partner, sn[i], y * cs[i]) : fmaf(-partner, sn[i], y * cs[i]);
      if (!m_ok || j >= left) continue;
      if (hd < a.Hq) {
        ((bf16_t *)a.q_out)[((int64_t)n * a.Hq + hd) * d + feat] = f32_to_bf16(o);
      } else {
        const int c = is_v ? hd - a.Hq - a.Hkv : hd - a.Hq;
        ((bf16_t *)(is_v ? a.v_cache : a.k_cache))[(int64_t)kv_row * a.stride_tok + (int64_t)c * a.stride_head + feat] = f32_to_bf16(o);
      }
    }
  };
  skinny_once<true, 256>((const bf16_t *)a.w, H, 2 * pairs, 2 * pairs, at, staged, xload, (const bf16_t *)a.gamma, a.M, smem, more, epi);
}

// ---------------------------------------------------------------------------------------------
// FC, one activation row: a wavefront owns one output feature, as in the kernel of whole slices.  It issues
// the loads of its weight row KS slices at a time, then fetches the activation row (shared by all wavefronts
// through L2), multiplies and reduces across its lanes on the vector ALU.
// ---------------------------------------------------------------------------------------------
template <int KS>             // slices in flight: at least K / 512 (K = 2H), or 16
__global__ void __launch_bounds__(256)
hsr_fc_any_gemv_kernel(HsrFcArgs a) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  const int lane = threadIdx.x & 63;
  const int nfeat = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int H = a.H;
  if (nfeat >= H) return;
  const int K = 2 * H;
  const __amdgpu_buffer_rsrc_t rs = weight_rows((const bf16_t *)a.w + (int64_t)__builtin_amdgcn_readfirstlane(nfeat) * K);
  const int tok = min(max(a.token_ids[0], 0), a.vocab - 1);
  const bf16_t *E = (const bf16_t *)a.embed + (int64_t)tok * H;
  const bf16_t *Hp = (const bf16_t *)a.h_prev;
  float acc = 0.f;
  for (int s0 = 0; s0 < K; s0 += KS * kSlice) {
    u32x4 wv[KS], xv[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int k = s0 + kSlice * s + 8 * lane;
      wv[s] = __builtin_amdgcn_raw_buffer_load_b128(rs, k < K ? (unsigned int)k * 2u : kPastEnd, 0, 2);
    }
    __builtin_amdgcn_sched_barrier(0);   // all of the row on its way before anything else
#pragma unroll
    for (int s = 0; s < KS; ++s) {     // columns below H meet the embedding, the rest the hidden state
      const int k = min(s0 + kSlice * s + 8 * lane, K - 8);
      xv[s] = *(const u32x4 *)(k < H ? E + k : Hp + (k - H));
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s0 + kSlice * s + 8 * lane >= K) xv[s] = (u32x4){0u, 0u, 0u, 0u};
      const unsigned int w4[4] = {wv[s].x, wv[s].y, wv[s].z, wv[s].w};
      const unsigned int x4[4] = {xv[s].x, xv[s].y, xv[s].z, xv[s].w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w4[e]), __builtin_bit_cast(bf16x2, x4[e]),
                                              acc, false);
    }
  }
  acc = wave_sum_valu(acc);
  if (lane == 0) {
    const float b = a.bias != nullptr ? bf16_to_f32(((const bf16_t *)a.bias)[nfeat]) : 0.f;
    ((bf16_t *)a.z)[nfeat] = f32_to_bf16(acc + b);
  }
}

// FC, two to four activation rows: a wavefront owns two output features.  The activations of KS slices (of the
// embeddings, then of the hidden states: a slice lies in one of them) go to LDS without passing through registers, once
// per workgroup, ahead of the weights; a weight row's slices are all on their way at once, and every 16 bytes of
// activations read from LDS meet both features.  The activations do not flow: the token ids are read by a load that the
// compiler waits for in every trip of the loop, and its wait takes in the trip's load before, which it does not count.  A
// wavefront thus makes MM * KS / nw round trips one after the other, 8 at four rows of 2,560, before its weights.  The
// staged kernel brings each wavefront's slices in two or three rounds and leaves compute units without a tile.  Staged /
// here, us: 2,048 columns, two rows 7.8 / 5.7; 640, two 4.3 / 3.1; 2,560, four 10.0 / 8.8; 5,120, two 28.2 / 23.5, four
// 28.6 / 25.9; 1,536, four 6.8 / 5.7; 256, three 3.8 / 3.5.  Above four rows, and at 3,584 and 4,096 columns (where the
// kernels of whole slices are as fast at two rows and faster at four, 12.3 / 14.5), this form is the slower one: 2,560, eight
// rows 10.7 / 12.75, 4,096, seven 16.4 / 21.4.
constexpr int kFewWaves = 8;

template <int MM, int KS>     // rows (the last ones may be empty), slices in flight
__global__ void __launch_bounds__(kFewWaves * 64)
hsr_fc_few_kernel(HsrFcArgs a) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];             // [MM][KS] slices
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = (int)blockDim.x >> 6;
  const int H = a.H, K = 2 * H, half_slices = (H + kSlice - 1) / kSlice, n_slices = 2 * half_slices;
  const int f = 2 * min((int)blockIdx.x * nw + w, H / 2 - 1);                      // features f, f + 1
  const __amdgpu_buffer_rsrc_t rs = weight_rows((const bf16_t *)a.w + (int64_t)f * K);
  const __amdgpu_buffer_rsrc_t rs_b = weight_rows((const bf16_t *)a.bias);
  const unsigned int bias =
      __builtin_amdgcn_raw_buffer_load_b32(rs_b, a.bias != nullptr ? (unsigned int)f * 2u : kPastEnd, 0, 0);
  const int toks = a.token_ids[min(lane, a.M - 1)];          // lane r: row r
  float acc[2][MM];
#pragma unroll
  for (int r = 0; r < MM; ++r) acc[0][r] = acc[1][r] = 0.f;
  for (int c0 = 0; c0 < n_slices; c0 += KS) {
    if (c0 > 0) __syncthreads();                             // the last slices have been read
    for (int x = w; x < MM * KS; x += nw) {
      const int r = x / KS, s = c0 + x - r * KS;
      const bool of_hidden = s >= half_slices;
      const int at = (s - (of_hidden ? half_slices : 0)) * kSlice + 8 * lane;      // column of its half
      const int m = min(r, a.M - 1);
      const int tok = min(max(__builtin_amdgcn_readlane(toks, m), 0), a.vocab - 1);
      const bf16_t *row = of_hidden ? (const bf16_t *)a.h_prev + (int64_t)m * H : (const bf16_t *)a.embed + (int64_t)tok * H;
      const bool some = r < a.M && s < n_slices;
      load_to_lds<false>(buffer_words(row, some ? (unsigned int)H * 2u : 0u), (unsigned int)at * 2u,
                         lds_offset(smem) + (unsigned int)x * 1024u);
    }
    u32x4 w0[KS], w1[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const bool of_hidden = c0 + s >= half_slices;
      const int at = (c0 + s - (of_hidden ? half_slices : 0)) * kSlice + 8 * lane;
      const unsigned int off = at < H ? (unsigned int)((of_hidden ? H : 0) + at) * 2u : kPastEnd;
      w0[s] = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 2);
      w1[s] = __builtin_amdgcn_raw_buffer_load_b128(rs, off, K * 2, 2);
    }
    __builtin_amdgcn_sched_barrier(0);
    wait_loads<2 * KS>();                                    // the activations are in LDS; the weights on their way
    __syncthreads();
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const unsigned int a0[4] = {w0[s].x, w0[s].y, w0[s].z, w0[s].w}, a1[4] = {w1[s].x, w1[s].y, w1[s].z, w1[s].w};
#pragma unroll
      for (int r = 0; r < MM; ++r) {
        const u32x4 xv = *reinterpret_cast<const u32x4 *>(smem + (r * KS + s) * 1024 + lane * 16);
        const unsigned int x4[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bf16x2 x = __builtin_bit_cast(bf16x2, x4[e]);
          acc[0][r] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a0[e]), x, acc[0][r], false);
          acc[1][r] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a1[e]), x, acc[1][r], false);
        }
      }
    }
  }
  float z0 = 0.f, z1 = 0.f;                                  // lane r: row r
#pragma unroll
  for (int r = 0; r < MM; ++r) {
    const float y0 = wave_sum_valu(acc[0][r]), y1 = wave_sum_valu(acc[1][r]);
    if (lane == r) { z0 = y0; z1 = y1; }
  }
  if (lane < a.M && (int)blockIdx.x * nw + w < H / 2)
    *(unsigned int *)((bf16_t *)a.z + (int64_t)lane * H + f) = pack_bf16x2(z0 + bf16lo_to_f32(bias), z1 + bf16hi_to_f32(bias));
}

// QKV, one activation row per blockIdx.y: a wavefront owns one rotary pair.  The activations times gamma, as two bf16
// terms that add up to the whole product (see skinny_gemm), are made once per workgroup and kept in LDS while the weights
// are on their way: two dot-product instructions per two weights, no unpacking.  Made by every
// wavefront, in fp32 with all weights unpacked (448 vector instructions a wavefront against 112 dot products), the
// arithmetic came to 1.7 us a compute unit behind the last weights.  Before / now, us: 3,584 columns, 28/4 heads of 128
// 9.9 / 8.4; 5,120, 40/8 of 128 21.4 / 17.1; 4,096, 32/8 of 128 12.0 / 11.0; 1,024, 16/4 of 64 4.3 / 4.0; two rows of
// 640, 8/2 of 64 4.15 / 3.8.
constexpr int kGemvMinWaves = 4, kGemvMaxWaves = 16;

template <int KS>             // slices in flight: at least H / 512, or 8
__global__ void __launch_bounds__(kGemvMaxWaves * 64)
draft_qkv_gemv_kernel(DraftQkvArgs a) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  // (one slice: a lane's own columns, made by every wavefront for itself, without the barrier; 256 columns 3.3 -> 3.1 us)
  constexpr bool kOwn = KS == 1;
  __shared__ u32x4 uh[KS * 64], ul[KS * 64];                 // leading and other terms, 8 columns each
  __shared__ float ssq_lds[kGemvMaxWaves];
  const int tid = threadIdx.x, lane = tid & 63, m = blockIdx.y;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), nw = (int)blockDim.x >> 6;
  const int half = a.d >> 1;
  const int n_pairs = (a.Hq + 2 * a.Hkv) * half;
  const int pair = min((int)blockIdx.x * nw + w, n_pairs - 1);          // (head, feature of the first half)
  const int hd = pair / half, f = pair - hd * half;
  const int H = a.H;
  const __amdgpu_buffer_rsrc_t rs =
      weight_rows((const bf16_t *)a.w + (int64_t)__builtin_amdgcn_readfirstlane(hd * a.d + f) * H);
  const unsigned int pair_off = (unsigned int)half * (unsigned int)H * 2u;
  const __amdgpu_buffer_rsrc_t rs_z = weight_rows((const bf16_t *)a.z + (int64_t)m * H);
  const __amdgpu_buffer_rsrc_t rs_g = weight_rows((const bf16_t *)a.gamma);
  // the activations of this thread: 8 columns, twice where KS * 64 threads are more than the workgroup has
  constexpr int kChunks = KS * 64;
  static_assert(kChunks <= 2 * 64 * kGemvMinWaves, "two chunks of activations per thread");
  float s0 = 0.f, s1 = 0.f, ssq = 0.f;
  // operands of the end, first of all: in order, they would wait for the weights
  const bool is_v = hd >= a.Hq + a.Hkv;
  const __amdgpu_buffer_rsrc_t rs_b = weight_rows((const bf16_t *)a.bias);
  const unsigned int off_b = a.bias != nullptr ? (unsigned int)(hd * a.d + f) * 2u : kPastEnd;
  const bf16_t b0 = __builtin_amdgcn_raw_buffer_load_b16(rs_b, off_b, 0, 0);
  const bf16_t b1 = __builtin_amdgcn_raw_buffer_load_b16(rs_b, off_b, a.bias != nullptr ? a.d : 0, 0);
  const float cs = a.rope_cos[m * half + f], sn = a.rope_sin[m * half + f];
  for (int k0 = 0; k0 < H; k0 += KS * kSlice) {
    if (k0 > 0) __syncthreads();                             // the last slices' terms have been read
    u32x4 x[2], g[2];
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const int c = kOwn ? lane + 64 * y : tid + y * (int)blockDim.x, k = k0 + 8 * c;
      const unsigned int off = c < kChunks && k < H ? (unsigned int)k * 2u : kPastEnd;
      x[y] = __builtin_amdgcn_raw_buffer_load_b128(rs_z, off, 0, 0);
      g[y] = __builtin_amdgcn_raw_buffer_load_b128(rs_g, off, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);                       // ahead of the weights, whose arrival the terms do not wait for
    u32x4 w0[KS], w1[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int k = k0 + kSlice * s + 8 * lane;
      const unsigned int off = k < H ? (unsigned int)k * 2u : kPastEnd;
      w0[s] = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 2);
      w1[s] = __builtin_amdgcn_raw_buffer_load_b128(rs, off, pair_off, 2);
    }
    __builtin_amdgcn_sched_barrier(0);
    u32x4 h_own, l_own;
    auto terms = [&](const u32x4 &xc, const u32x4 &gc, u32x4 &hi8, u32x4 &lo8) __attribute__((always_inline)) {
      float xf[8], gf[8], lo[8];
      unsigned int hb[8];
      Elem<bf16_t>::unpack(xc, xf);
      Elem<bf16_t>::unpack(gc, gf);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        ssq = fmaf(xf[e], xf[e], ssq);
        const float u = xf[e] * gf[e];
        hb[e] = __float_as_uint(u) & 0xffff0000u;
        lo[e] = low_term(u, __uint_as_float(hb[e]));
      }
      hi8 = (u32x4){(hb[0] >> 16) | hb[1], (hb[2] >> 16) | hb[3], (hb[4] >> 16) | hb[5], (hb[6] >> 16) | hb[7]};
      lo8 = (u32x4){pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]), pack_bf16x2(lo[4], lo[5]), pack_bf16x2(lo[6], lo[7])};
    };
    if constexpr (kOwn) {
      terms(x[0], g[0], h_own, l_own);
    } else {
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        const int c = tid + y * (int)blockDim.x;
        if (c >= kChunks) break;
        u32x4 hv, lv;
        terms(x[y], g[y], hv, lv);
        uh[c] = hv;
        ul[c] = lv;
      }
      __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const u32x4 hv = kOwn ? h_own : uh[64 * s + lane], lv = kOwn ? l_own : ul[64 * s + lane];
      const unsigned int h4[4] = {hv.x, hv.y, hv.z, hv.w}, l4[4] = {lv.x, lv.y, lv.z, lv.w};
      const unsigned int a4[4] = {w0[s].x, w0[s].y, w0[s].z, w0[s].w}, c4[4] = {w1[s].x, w1[s].y, w1[s].z, w1[s].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bf16x2 p0 = __builtin_bit_cast(bf16x2, a4[e]), p1 = __builtin_bit_cast(bf16x2, c4[e]);
        const bf16x2 h = __builtin_bit_cast(bf16x2, h4[e]), l = __builtin_bit_cast(bf16x2, l4[e]);
        s0 = __builtin_amdgcn_fdot2_f32_bf16(p0, l, s0, false);
        s1 = __builtin_amdgcn_fdot2_f32_bf16(p1, l, s1, false);
        s0 = __builtin_amdgcn_fdot2_f32_bf16(p0, h, s0, false);
        s1 = __builtin_amdgcn_fdot2_f32_bf16(p1, h, s1, false);
      }
    }
  }
  ssq = wave_sum_valu(ssq);
  s0 = wave_sum_valu(s0); s1 = wave_sum_valu(s1);
  if constexpr (!kOwn) {
    if (lane == 0) ssq_lds[w] = ssq;
    __syncthreads();
    ssq = 0.f;
    for (int ww = 0; ww < nw; ++ww) ssq += ssq_lds[ww];
  }
  if (lane != 0 || (int)blockIdx.x * nw + w >= n_pairs) return;
  const float rstd = __builtin_amdgcn_rsqf(ssq / (float)H + a.eps);
  const float y0 = fmaf(s0, rstd, bf16_to_f32(b0)), y1 = fmaf(s1, rstd, bf16_to_f32(b1));
  float o0 = y0, o1 = y1;
  if (!is_v) {
    o0 = y0 * cs - y1 * sn;
    o1 = y1 * cs + y0 * sn;
  }
  bf16_t *dst;
  if (hd < a.Hq) {
    dst = (bf16_t *)a.q_out + ((int64_t)m * a.Hq + hd) * a.d;
  } else {
    const int c = is_v ? hd - a.Hq - a.Hkv : hd - a.Hq;
    dst = (bf16_t *)(is_v ? a.v_cache : a.k_cache) + (int64_t)a.kv_rows[m] * a.stride_tok +
          (int64_t)c * a.stride_head;
  }
  dst[f] = f32_to_bf16(o0);
  dst[f + half] = f32_to_bf16(o1);
}

template <auto kKern, class Args>
hipError_t launch_skinny(int nw, dim3 grid, const Args &a, hipStream_t st) {
  // more than 64 KB of dynamic LDS has to be allowed once per kernel
  static const hipError_t attr = hipFuncSetAttribute((const void *)kKern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     skinny_lds_bytes(kMaxWaves));
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kKern, grid, dim3(nw * 64), skinny_lds_bytes(nw), st, a);
  return hipGetLastError();
}

template <int MM, int KS>
hipError_t launch_few(const HsrFcArgs &a, hipStream_t st) {
  static const hipError_t attr = hipFuncSetAttribute((const void *)hsr_fc_few_kernel<MM, KS>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, MM * KS * 1024);
  if (attr != hipSuccess) return attr;
  // as many wavefronts per workgroup as put one workgroup on every compute unit
  const int pairs = a.H / 2, nw = std::min(std::max((pairs + 255) / 256, 4), kFewWaves);
  hipLaunchKernelGGL((hsr_fc_few_kernel<MM, KS>), dim3((pairs + nw - 1) / nw), dim3(nw * 64), MM * KS * 1024, st, a);
  return hipGetLastError();
}

// Wavefronts for rows of K elements: as few rounds of slices as eight wavefronts allow, dealt evenly.
int skinny_waves(int K) {
  const int slices = (K + kSlice - 1) / kSlice;
  const int rounds = (slices + kMaxWaves - 1) / kMaxWaves;
  return (slices + rounds - 1) / rounds;
}

}  // namespace

hipError_t launch_hsr_fc_any(const HsrFcArgs &a, hipStream_t st) {
  const int K = 2 * a.H, slices = (K + kSlice - 1) / kSlice;
  if (a.M == 1) {               // one row: a wavefront per output feature
    const dim3 grid((a.H + 3) / 4);
    if (slices <= 4) hipLaunchKernelGGL(hsr_fc_any_gemv_kernel<4>, grid, dim3(256), 0, st, a);
    else if (slices <= 8) hipLaunchKernelGGL(hsr_fc_any_gemv_kernel<8>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(hsr_fc_any_gemv_kernel<16>, grid, dim3(256), 0, st, a);
    return hipGetLastError();
  }
  if (a.M <= 4) {
    if (slices <= 4) return a.M <= 2 ? launch_few<2, 4>(a, st) : launch_few<4, 4>(a, st);
    return a.M <= 2 ? launch_few<2, 10>(a, st) : launch_few<4, 10>(a, st);
  }
  // five to eight rows: at once, where the slices' wavefronts fit a workgroup and their rows its 160 KB (up to 3,072 columns)
  if (a.M <= 8 && slices <= kOnceWaves) {
    const int rows = (even_rows(a.H, 16) + 1) / 2 * 2;
    if (once_lds_bytes(slices, rows, kSlice) <= 160 * 1024) {
      static const hipError_t attr = hipFuncSetAttribute((const void *)hsr_fc_once_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      if (attr != hipSuccess) return attr;
      hipLaunchKernelGGL(hsr_fc_once_kernel, dim3((a.H + rows - 1) / rows), dim3(slices * 64), once_lds_bytes(slices, rows, kSlice), st, a, rows);
      return hipGetLastError();
    }
  }
  return launch_skinny<hsr_fc_any_kernel>(skinny_waves(K), dim3((a.H + 15) / 16, (a.M + 15) / 16), a, st);
}

hipError_t launch_draft_qkv_any(const DraftQkvArgs &a, hipStream_t st) {
  const int n_heads = a.Hq + 2 * a.Hkv, slices = (a.H + kSlice - 1) / kSlice;
  // One row: a wavefront per rotary pair.  Two rows as well up to 1,024 columns, where both rows' weights come
  // from the caches and the staged kernel's latency shows (256 columns 2.9 us; staged 6.0, plain ALU 4.6).
  if (a.M == 1 || (a.M == 2 && a.H <= 1024)) {
    // as many wavefronts per workgroup as put one workgroup on every compute unit
    const int pairs = n_heads * (a.d / 2), nw = std::min(std::max((pairs * a.M + 255) / 256, kGemvMinWaves), kGemvMaxWaves);
    const dim3 grid((pairs + nw - 1) / nw, a.M), block(nw * 64);
    if (slices <= 1) hipLaunchKernelGGL(draft_qkv_gemv_kernel<1>, grid, block, 0, st, a);
    else if (slices <= 4) hipLaunchKernelGGL(draft_qkv_gemv_kernel<4>, grid, block, 0, st, a);
    else if (slices <= 7) hipLaunchKernelGGL(draft_qkv_gemv_kernel<7>, grid, block, 0, st, a);
    else hipLaunchKernelGGL(draft_qkv_gemv_kernel<8>, grid, block, 0, st, a);
    return hipGetLastError();
  }
  const int nw = (a.H + 255) / 256;          // two to eight rows, up to 4,096 columns: at once
  if (a.M <= 8 && nw <= kOnceWaves) {
    const int n_pairs = n_heads * (a.d / 2), pairs = even_rows(n_pairs, 8);
    static const hipError_t attr = hipFuncSetAttribute((const void *)draft_qkv_once_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(draft_qkv_once_kernel, dim3((n_pairs + pairs - 1) / pairs), dim3(nw * 64), once_lds_bytes(nw, 2 * pairs, 256), st, a, pairs);
    return hipGetLastError();
  }
  const dim3 grid(n_heads * (a.d / 16), (a.M + 15) / 16);
  return a.M <= 8 ? launch_skinny<draft_qkv_any_kernel<true>>(skinny_waves(a.H), grid, a, st)
                  : launch_skinny<draft_qkv_any_kernel<false>>(skinny_waves(a.H), grid, a, st);
}

}  // namespace sparrow
