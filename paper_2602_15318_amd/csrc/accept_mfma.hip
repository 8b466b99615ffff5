// Greedy acceptance, matrix-core lm_head pass: bf16 and fp32, gfx950.
//
// logits[r, v] = sum_x hidden[r, x] * W[v, x] for the B*(n_q+1) verified rows r against the whole
// vocabulary; 1.09 GB of weights for Qwen2.5-VL-7B, read exactly once per pass, so the pass is bound
// by HBM and organised around the weight stream.  Logits never leave the registers unless the
// caller needs them (sampling, top-k): every lane keeps the best (value, lowest index) of the
// vocabulary rows it has seen for its column; one candidate per (workgroup, row) is written at the
// end and reduced by the finalize kernel.
#include <algorithm>
#include <type_traits>

#include "accept.hpp"
#include "common.hpp"

namespace sparrow {

namespace {

constexpr int kNumCU = 256;
constexpr int kKsSlice = 512;             // k elements of a wavefront's slice of a row (1 KB)
constexpr int kKsGroup = 4;               // vocabulary tiles (of 16 rows) per group
constexpr int kKsWaves = 8;               // most wavefronts of a workgroup

// A lane's four consecutive logits of a row, tokens v .. v+3, those past V left out.  One 16-byte store (rows of odd
// vocabularies start at any multiple of 4 bytes; the type asks for no more): a store instruction is worked off line by
// line, and with one per value the 64 of a wavefront's tile showed.  Tiled kernel, us, four stores / one: 174 rows of
// 3,584 x 152,064 393 / 367, 156 of 512 x 16,724 26.3 / 21.6, 315 of 1,408 x 6,828 31.8 / 27.3, 36 of 2,048 x 64,003
// 60.0 / 57.9; the k-split kernel, which waits for its weights, is the same.
typedef f32x4 __attribute__((aligned(4))) f32x4u;
__device__ __forceinline__ void store_logits(float *row, int v, int V, const f32x4 &lg) {
  if (v + 3 < V) {
    *reinterpret_cast<f32x4u *>(row + v) = lg;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (v + i < V) row[v + i] = lg[i];
  }
}

// k-split kernel: any hidden size up to 8,192 that is a multiple of 8.
//
// A row is cut into slices of 512 elements (the last one may be short: its missing columns are read
// as zeros by the bounds check of the buffer loads); the nw wavefronts of a workgroup own one slice
// each (SPW = 2: two, w and w + nw).  The wavefront's slice of the 16 hidden rows lives in registers
// for the whole pass (16 B operands), and every load instruction of the wavefront reads 1 KB that is
// contiguous in memory (the slice of one weight row), so the workgroup sweeps W front to back.  The
// 16-row tile goes registers -> LDS (private 16 KB per wavefront, XOR swizzled) -> A operands.  The
// wavefronts' partial logits of a group of tiles are summed through LDS; wavefront g then owns the
// argmax bookkeeping of tile g of the group.
//
// nw = ceil(H / 512) (half of it above 4,096); as many workgroups per compute unit as their 20 KB of
// LDS per wavefront allow, so that 80 to 128 KB of weights are in flight per compute unit whatever
// H is.
//
// NB = blocks of 16 hidden rows handled in one pass over W (1 or 2); the vocabulary group is
// kKsGroup / NB tiles so that the partial logits in LDS stay at 4 KB per wavefront.
// A matrix instruction rounds its sums at the size they have reached, so a chain over a whole slice loses
// more than the products deserve: pairs of instructions (64 products) start from zero and are added up in
// fp64, and so are the wavefronts' shares.  Error of a logit 0.55e-7 of its size whatever H is (chains
// over the slice in fp32: 0.65e-7 at H = 256, 1.35e-7 at 5,120; a plain-ALU sum 0.55 to 0.9e-7).
// Measured: 152,064 x 3584 at 9 rows 165 us with the finalize pass (6.6 TB/s); 64,003 x 2048 at 9
// rows 49 us, 32 rows 54 us; 151,936 x 2560 118 us.
template <int SPW, int NB>
__global__ void __launch_bounds__(kKsWaves * 64)
lm_head_ksplit_kernel(AcceptArgs a) {
  const int row0 = 16 * NB * (int)blockIdx.y;     // row blocks side by side
  const int wg = (int)blockIdx.x, n_wg = (int)gridDim.x;      // streams of vocabulary tiles
  constexpr int G = kKsGroup / NB;          // vocabulary tiles per group
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // [nw][16 KB] staging, then [NB][nw][G][64] f32x4 partial logits
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = (int)blockDim.x >> 6;
  const int n = lane & 15, c4 = lane >> 4;
  const int H = a.H, V = a.V;
  const unsigned int row_bytes = (unsigned int)H * 2u;
  unsigned char *stg = smem + w * 16384;
  f32x4 *red = reinterpret_cast<f32x4 *>(smem + nw * 16384);

  // Vocabulary tiles (16 rows) are dealt round-robin to the workgroups one by one, so that the
  // workgroups' shares differ by at most one tile (9,504 tiles over 256 workgroups: 38 against a
  // mean of 37.1; dealt in groups of four tiles it was 40 against 37.1, and the kernel ends with
  // its slowest workgroup); a workgroup still reduces its tiles in groups of G, the last group
  // possibly short.
  const int n_vt = (V + 15) / 16;
  const int n_tiles = n_vt > wg ? (n_vt - wg + n_wg - 1) / n_wg : 0;

  // tile t of this workgroup -> first vocabulary row
  auto tile_row0 = [&](int t) { return (wg + t * n_wg) * 16; };
  // 16 loads of 1 KB: load r = the k-slice of row r of the tile (rows clamped to the last row), as
  // buffer loads from the tile's first row: columns past H get an offset past the buffer's end and
  // read as zero.  Issued unconditionally (tile index clamped) so that the number of loads in
  // flight is static.  One tile (16 KB per wavefront) in flight: the weight stream already
  // saturates HBM with that, a second tile in flight measured 2 us slower at H = 3584.
  constexpr unsigned int kPastEnd = 0x80000000u;
  unsigned int col_off[SPW];
#pragma unroll
  for (int sl = 0; sl < SPW; ++sl) {
    const int k = kKsSlice * (w + sl * nw) + 8 * lane;
    col_off[sl] = k < H ? (unsigned int)k * 2u : kPastEnd;
  }
  u32x4 buf[16];
  auto issue = [&](int t, int sl) {
    const int v0 = tile_row0(min(t, max(n_tiles - 1, 0)));
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const unsigned char *)a.lm_head + (int64_t)min(v0, V - 1) * row_bytes), (short)0, (int)0x7fffffff, 0x00027000);
#pragma unroll
    for (int r = 0; r < 16; ++r)
      buf[r] = __builtin_amdgcn_raw_buffer_load_b128(rs, col_off[sl], max(min(r, V - 1 - v0), 0) * row_bytes, 2);
  };
  issue(0, 0);

  // B operands: lane (n, c4) holds hidden[row0 + 16 nb + n][slice + 32 ks + 8 c4 .. +8], ks = 0..15
  bf16x8 hreg[NB][SPW][16];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int row = row0 + 16 * nb + n;
    const bool ok = row < a.M;
    // rows past M (padding of the last block) take the data of valid rows: never stored
    const bf16_t *hp = (const bf16_t *)a.hidden + (int64_t)(ok ? row : row % a.M) * H;
#pragma unroll
    for (int sl = 0; sl < SPW; ++sl)
#pragma unroll
      for (int ks = 0; ks < 16; ++ks) {
        const int k = kKsSlice * (w + sl * nw) + 32 * ks + 8 * c4;
        u32x4 h = {0u, 0u, 0u, 0u};
        if (k < H) h = *(const u32x4 *)(hp + k);
        hreg[nb][sl][ks] = __builtin_bit_cast(bf16x8, h);
      }
  }

  // staging: lane i of load r holds chunk i (16 bytes) of row r; stored at chunk position
  // (i & ~15) | ((i & 15) ^ r) so that the A-operand reads (16 rows, same chunk) hit all banks
  const int a_base = n * 1024;      // A read: row n, chunk 4 ks + c4
  float best[NB];
  int best_i[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) { best[nb] = -INFINITY; best_i[nb] = 0x7fffffff; }
  for (int t = 0; t < n_tiles; ++t) {
    double acc[NB][4];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[nb][i] = 0.0;
#pragma unroll
    for (int sl = 0; sl < SPW; ++sl) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        *reinterpret_cast<u32x4 *>(stg + r * 1024 + (((lane & ~15) | ((lane & 15) ^ r)) << 4)) = buf[r];
      issue(sl + 1 < SPW ? t : t + 1, sl + 1 < SPW ? sl + 1 : 0);
#pragma unroll
      for (int ks = 0; ks < 16; ks += 2) {
        if (NB > 1 && ks % 8 == 0) __builtin_amdgcn_sched_barrier(0);     // operands read further ahead spill registers
        const int ch0 = 4 * ks + c4, ch1 = ch0 + 4;
        const bf16x8 a0 = *reinterpret_cast<const bf16x8 *>(stg + a_base + (((ch0 & ~15) | ((ch0 & 15) ^ n)) << 4));
        const bf16x8 a1 = *reinterpret_cast<const bf16x8 *>(stg + a_base + (((ch1 & ~15) | ((ch1 & 15) ^ n)) << 4));
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          f32x4 p = {0.f, 0.f, 0.f, 0.f};
          p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, hreg[nb][sl][ks], p, 0, 0, 0);
          p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, hreg[nb][sl][ks + 1], p, 0, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[nb][i] += (double)p[i];
        }
      }
    }
    const int g = t % G;
    // the tile's partial logits go to LDS at once ([row block][wavefront][tile of the group]: G * NB
    // = 4 slots per wavefront whatever NB), not into registers held for the whole group
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      red[((nb * nw + w) * G + g) * 64 + lane] = (f32x4){(float)acc[nb][0], (float)acc[nb][1], (float)acc[nb][2], (float)acc[nb][3]};
    if (g == G - 1 || t == n_tiles - 1) {     // uniform over the workgroup
      // sum the group's partial logits over the wavefronts; the tiles of the group (the last group
      // may hold fewer than G) are dealt to the wavefronts
      __syncthreads();
      for (int tg = w; tg <= g; tg += nw) {
        const int vbase = tile_row0(t - g + tg) + 4 * c4;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          double sum64[4] = {0.0, 0.0, 0.0, 0.0};
          for (int ww = 0; ww < nw; ++ww) {
            const f32x4 part = red[((nb * nw + ww) * G + tg) * 64 + lane];
#pragma unroll
            for (int i = 0; i < 4; ++i) sum64[i] += (double)part[i];
          }
          const f32x4 sum = {(float)sum64[0], (float)sum64[1], (float)sum64[2], (float)sum64[3]};
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (vbase + i < V && sum[i] > best[nb]) { best[nb] = sum[i]; best_i[nb] = vbase + i; }
          if (a.logits != nullptr) {
            const int row = row0 + 16 * nb + n;
            if (row < a.M) store_logits(a.logits + (int64_t)row * V, vbase, V, sum);
          }
        }
      }
      __syncthreads();   // reads done before the next partials are written
    }
  }

  // one candidate per (workgroup, row): best over the four lanes of a column, then over the
  // wavefronts through LDS (all partial logits have been read: the loop ends with a barrier)
  float *cv = reinterpret_cast<float *>(red);                     // [nw][NB][16]
  int *ci = reinterpret_cast<int *>(cv + nw * NB * 16);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    float bv = best[nb];
    int bi = best_i[nb];
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const float ov = __shfl_xor(bv, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    }
    if (c4 == 0) { cv[(w * NB + nb) * 16 + n] = bv; ci[(w * NB + nb) * 16 + n] = bi; }
  }
  __syncthreads();
  if (tid < 16 * NB && row0 + tid < a.M) {
    float bv = cv[tid];
    int bi = ci[tid];
    for (int ww = 1; ww < nw; ++ww) {
      const float ov = cv[ww * NB * 16 + tid];
      const int oi = ci[ww * NB * 16 + tid];
      if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    }
    a.cand_val[(int64_t)(row0 + tid) * a.n_cand + blockIdx.x] = bv;
    a.cand_idx[(int64_t)(row0 + tid) * a.n_cand + blockIdx.x] = bi;
  }
}

int ksplit_waves(int H) {
  const int slices = (H + kKsSlice - 1) / kKsSlice;
  return slices <= kKsWaves ? slices : (slices + 1) / 2;
}
int ksplit_lds(int nw) { return nw * (16384 + kKsGroup * 64 * 16); }

// Workgroups of a row block = candidates per row: as many as fit the compute units (160 KB of LDS, eight
// wavefronts each), shared by the row blocks, and no more than there are vocabulary tiles.
int ksplit_slots(int H) {
  const int nw = ksplit_waves(H);
  return kNumCU * std::min(160 * 1024 / ksplit_lds(nw), kKsWaves / nw);
}
// (a multiple of 8 where several blocks stream the same tiles: one XCD, whose L2 serves all but the first)
int ksplit_grid(int H, int V, int blocks) {
  return std::min(blocks > 1 ? std::max(ksplit_slots(H) / blocks / 8 * 8, 8) : ksplit_slots(H), (V + 15) / 16);
}
// Hidden rows of a workgroup: 32, or 16 above 4,096 columns, where the hidden rows of a wavefront's two slices
// fill its registers.
bool ksplit_wide(int H) { return H > kKsWaves * kKsSlice; }
int ksplit_rows(int H) { return ksplit_wide(H) ? 16 : 32; }
int ksplit_blocks(int M, int H) { return (M + ksplit_rows(H) - 1) / ksplit_rows(H); }

template <int SPW, int NB>
hipError_t launch_ksplit(const AcceptArgs &a, int blocks, hipStream_t st) {
  static const hipError_t attr = hipFuncSetAttribute((const void *)lm_head_ksplit_kernel<SPW, NB>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, ksplit_lds(kKsWaves));
  if (attr != hipSuccess) return attr;
  const int nw = ksplit_waves(a.H);
  hipLaunchKernelGGL((lm_head_ksplit_kernel<SPW, NB>), dim3(a.n_cand, blocks), dim3(nw * 64), ksplit_lds(nw), st, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Tiled kernel for the rows that the k-split kernel does not take (bf16: more than 32, more than 16 above 4,096
// columns) and for fp32: one pass over W whatever the number of rows up to 256 (fp32: 128), row blocks side by
// side above.
//
// A persistent workgroup owns tiles of VT vocabulary rows x BM hidden rows and walks the hidden size in steps of
// kRow bytes of a row; its wavefronts form a WV x WM grid.  16-byte chunks lie XOR-swizzled in LDS as in the
// attention kernel.  fp32: 4 wavefronts; both operands of a step travel memory -> registers (requested one step
// ahead) -> LDS -> MFMA operands; the workgroups that share a compute unit have one LDS tile each and one's MFMAs
// run under the other's loads and LDS traffic.  bf16: 8 wavefronts; the loads fill three LDS tiles directly, two
// steps ahead.  Rows past V or M and columns past H come back as zeros from the bounds check of the buffer loads,
// so no size has to be a multiple of anything.
// What bounds it at 248 rows: MFMAs (530 ns of a step at the clock they run at), fp64 additions (600 ns) and
// operand reads from LDS, which overlap only in part with two wavefronts per SIMD; without any load a step takes
// 1.05 us, with them 1.5.  152,064 x 3584 at 248 / 372 rows, us, step by step: through registers, two LDS tiles
// 458 / 880; straight to LDS 440 / 850; barrier before the last row of tiles 430 / 800; additions of a row of tiles
// beside the next one's MFMAs 415 / 750.  (The two wavefronts of a SIMD half a step apart, with two barriers per
// step, 495 / 960.)
// bf16 tiles, 4 wavefronts through registers (256 rows: 8, two LDS tiles) / as here, time ratio over drawn sizes,
// median and range: 64 x 64 1.07 (0.97 to 1.59), 128 x 64 1.02 (0.93 to 1.16), 64 x 128 1.23 (1.10 to 1.63), 128 x
// 128 1.11 (0.99 to 1.24), 64 x 256 1.02 (0.94 to 1.14), 128 x 256 1.11 (0.99 to 1.46), the gains of other tile
// heights included; with the logits stored 1.02, 1.00, 1.09, 1.03, 1.01, 1.06 (0.93 to 1.49).  128 x 64 is slower
// where all tiles fit the chip at once and rows are short (33 rows of 584 x 45,097 22.9 / 24.6 us), 64 x 256 with
// more than 400 rows of 3,000 columns and more (429 rows of 4,560 x 5,977 87.5 / 92.5), 128 x 128 where the store of
// the logits has no second workgroup to hide behind (103 rows of 2,720 x 65,136 125 / 134).
// Sums: a matrix instruction rounds at the size its sums have reached (about four times per 32 bf16
// products, once per fp32 product), so chains of two bf16 instructions or four fp32 ones start from zero
// and are added up in fp64.  Error of a logit, against one fp32 chain over H (bf16) or over a step (fp32)
// and against the plain-ALU kernels: bf16 0.5e-7 of its size at every width (0.86e-7 at H = 256, 3.7e-7 at
// 3,584, 4.5e-7 at 5,120; 0.55 to 1.05e-7), fp32 0.8e-7 (1.2 to 2.7e-7; 0.78 to 1.9e-7).  The sums take
// 8 registers per 16 x 16 tile and the additions two vector instructions per value: wavefront tiles are
// 64 x 64 at most, and 256 rows take one workgroup of 8 wavefronts per compute unit.
// 152,064 x 3584 with the finalize pass, us (through registers): 40 rows 178 (188), 62 rows 186 (191), 96 rows 230
// (276), 124 rows 253 (281), 248 rows 399 (446), 372 rows 746 (874).
// fp32 (v_mfma_f32_16x16x4: fp32 products at 157 TFLOP/s; in brackets the plain-ALU kernel): 9 rows 335 (1678), 64
// rows 735 (7324), 248 rows 3124 (29370); 32,000 x 1024 at 9 rows 32 (137).
template <int kRow> __device__ __forceinline__ int gm_swz(int row) {
  return kRow == 256 ? (row & 7) << 1 : ((row >> 1) & 3) << 1;
}

// LDS tiles: three for a workgroup of 8 wavefronts (144 KiB at 128 x 256, two workgroups of 72 KiB at 128 x 64)
constexpr int tiled_buffers(int waves) { return waves == 8 ? 3 : 1; }

template <class T, int VT, int BM, int kWaves, int WV, int kRow>      // kRow: bytes of a row that a step covers
__global__ void __launch_bounds__(kWaves * 64, kWaves == 8 && BM <= 64 ? 4 : 2)
lm_head_tiled_kernel(AcceptArgs a, int blocks_m) {
  constexpr int WM = kWaves / WV;
  constexpr int NV = VT / WV / 16, NM = BM / WM / 16;      // 16-row tiles of a wavefront
  constexpr bool kF32 = std::is_same<T, float>::value;
  constexpr int kPer = Elem<T>::kPer16B, kChunks = kRow / 16, BK = kChunks * kPer;
  constexpr int kLdRows = kWaves * 64 / kChunks;           // rows that one load of the workgroup covers
  constexpr int kLdV = VT / kLdRows, kLdM = BM / kLdRows;  // loads of a thread per step
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wv = w / WM, wm = w % WM;
  const int n = lane & 15, c4 = lane >> 4;
  const int H = a.H, V = a.V;
  const unsigned int row_bytes = (unsigned int)H * (unsigned int)sizeof(T);
  // workgroups of one vocabulary stream (the row blocks) sit 8 indices apart: one XCD, one time
  const int mb = __builtin_amdgcn_readfirstlane(((int)blockIdx.x >> 3) % blocks_m);
  const int stream = __builtin_amdgcn_readfirstlane(((int)blockIdx.x >> 3) / blocks_m * 8 + ((int)blockIdx.x & 7));
  const int n_streams = __builtin_amdgcn_readfirstlane((int)gridDim.x / blocks_m);
  const int row0 = mb * BM;
  const int n_vt = (V + VT - 1) / VT;
  const int n_tiles = __builtin_amdgcn_readfirstlane(n_vt > stream ? (n_vt - stream + n_streams - 1) / n_streams : 0);
  const int nk = (H + BK - 1) / BK;
  const int n_steps = n_tiles * nk;

  // loader: thread -> rows tid / kChunks + kLdRows j, one 16-byte chunk of the step's part of a row
  const int ld_row = tid / kChunks, ld_pos = tid % kChunks;
  constexpr int kTileBytes = (VT + BM) * kRow;
  constexpr int kLd = kLdV + kLdM;
  // straight to LDS: the 64 lanes of a load fill 1 KB in their order, so that the swizzle is a choice of which
  // chunk a lane fetches (kLdRows is a multiple of 16: the same one for every j)
  constexpr bool kDirect = tiled_buffers(kWaves) > 1;
  static_assert(!kDirect || (kLdRows % 16 == 0 && kRow == 128), "a wavefront's load covers whole rows");
  const int ld_ch = kDirect ? ld_pos ^ gm_swz<kRow>(ld_row) : ld_pos;
  const unsigned int ld_off = (unsigned int)ld_row * row_bytes + (unsigned int)ld_ch * 16u;
  const unsigned char *const hid0 = (const unsigned char *)a.hidden + (int64_t)row0 * row_bytes;
  const unsigned int hid_bytes = (unsigned int)min(BM, a.M - row0) * row_bytes;
  u32x4 sg[kLd];
  // Rows of about a multiple of 4 KB, up to 64 hidden rows: the workgroups of an XCD start three steps apart and walk the
  // hidden size round.  All of them at one column of such rows meet in a few of the memory channels; at other widths the
  // columns of a step lie spread and this changes nothing (0.98 to 1.02).  us with the finalize pass, together / apart:
  // 36 rows of 2,048 x 64,003 61 / 52, 64 rows 60 / 52, 48 of 4,096 x 64,000 112 / 91, 24 of 6,144 x 32,000 83 / 77.  One
  // step apart 56, two 54, five 53 at the first.  With 128 rows 72 / 70 (100 of 2,048), 137 / 134 (128 of 4,096), but the
  // scalar work of it costs the other widths (124 of 3,584 x 152,064 273 / 281); 256 rows wait for their sums.
  constexpr bool kApart = kDirect && BM <= 64;
  const bool apart = kApart && ((row_bytes + 256u) & 4095u) <= 512u;
  const int k_first = apart ? __builtin_amdgcn_readfirstlane(3 * (stream >> 3) % nk) : 0;
  int is_tile = 0, is_k = k_first;                                 // the step the next issue() fetches
  auto issue = [&](int buf) {
    const int v0 = (stream + min(is_tile, max(n_tiles - 1, 0)) * n_streams) * VT;
    const int rows = min(VT, max(V - v0, 0));
    const unsigned char *const w0 = (const unsigned char *)a.lm_head + (int64_t)min(v0, V - 1) * row_bytes;
    const int k = is_k * BK + ld_ch * kPer;
    const unsigned int off = k < H ? ld_off + (unsigned int)(is_k * kRow) : 0x80000000u;
    if constexpr (kDirect) {
      const u32x4 rs_v = buffer_words(w0, (unsigned int)rows * row_bytes), rs_m = buffer_words(hid0, hid_bytes);
      const unsigned int dst = lds_offset(smem) + (unsigned int)(buf * kTileBytes + w * 1024);
#pragma unroll
      for (int j = 0; j < kLd; ++j)
        if (j < kLdV) load_to_lds<true>(rs_v, off + (unsigned int)(kLdRows * j) * row_bytes, dst + j * kLdRows * kRow);
        else load_to_lds<false>(rs_m, off + (unsigned int)(kLdRows * (j - kLdV)) * row_bytes, dst + j * kLdRows * kRow);
    } else {
      const __amdgpu_buffer_rsrc_t rs_v =
          __builtin_amdgcn_make_buffer_rsrc((void *)w0, (short)0, (int)(rows * row_bytes), 0x00027000);
      const __amdgpu_buffer_rsrc_t rs_m =
          __builtin_amdgcn_make_buffer_rsrc((void *)hid0, (short)0, (int)hid_bytes, 0x00027000);
#pragma unroll
      for (int j = 0; j < kLdV; ++j)
        sg[j] = __builtin_amdgcn_raw_buffer_load_b128(rs_v, off + (unsigned int)(kLdRows * j) * row_bytes, 0, 2);
#pragma unroll
      for (int j = 0; j < kLdM; ++j)
        sg[kLdV + j] = __builtin_amdgcn_raw_buffer_load_b128(rs_m, off + (unsigned int)(kLdRows * j) * row_bytes, 0, 0);
    }
    if (++is_k == nk) is_k = 0;
    if (is_k == k_first) ++is_tile;
  };
  auto stash = [&]() {
    unsigned char *p = smem + ld_row * kRow + ((ld_pos ^ gm_swz<kRow>(ld_row)) << 4);
#pragma unroll
    for (int j = 0; j < kLd; ++j) *reinterpret_cast<u32x4 *>(p + kLdRows * j * kRow) = sg[j];
  };

  double acc[NV][NM][4];
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int j = 0; j < NM; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.0;
  float best[NM];
  int best_i[NM];
#pragma unroll
  for (int j = 0; j < NM; ++j) { best[j] = -INFINITY; best_i[j] = 0x7fffffff; }
  const int m_wave = row0 + wm * (NM * 16);                  // first hidden row of the wavefront
  const bool live = m_wave < a.M;                            // a wavefront of padding rows only loads
  const int rd_row = n * kRow, rd_swz = gm_swz<kRow>(n);

  int cp_tile = 0, cp_k = 0;
  // Operands out of LDS, chains of kChain 16-byte chunks from zero (64 bf16 products, 16 fp32 ones), each added to the
  // tile's running sums in fp64
  constexpr int kChain = kF32 ? 1 : 2;
  u32x4 bm[kChain][NM];
  // Straight to LDS: the products of a row of tiles are added while the matrix cores form the next one's, over
  // the barrier and into the next step
  f32x4 pend[NM];
  if constexpr (kDirect) {
#pragma unroll
    for (int j = 0; j < NM; ++j) pend[j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  auto chunk = [&](int ks) { return ((4 * ks + c4) ^ rd_swz) << 4; };
  auto read_m = [&](int buf, int ks) {
    const unsigned char *pm = smem + buf * kTileBytes + (VT + wm * (NM * 16)) * kRow + rd_row;
#pragma unroll
    for (int x = 0; x < kChain; ++x)
#pragma unroll
      for (int j = 0; j < NM; ++j) bm[x][j] = *reinterpret_cast<const u32x4 *>(pm + j * 16 * kRow + chunk(ks + x));
  };
  auto read_v = [&](u32x4 *av, int buf, int ks, int i) {
    const unsigned char *pv = smem + buf * kTileBytes + wv * (NV * 16 * kRow) + rd_row;
#pragma unroll
    for (int x = 0; x < kChain; ++x) av[x] = *reinterpret_cast<const u32x4 *>(pv + i * 16 * kRow + chunk(ks + x));
  };
  auto products = [&](const u32x4 *av, int i) {              // row i of the wavefront's tiles
    f32x4 p[NM];
#pragma unroll
    for (int x = 0; x < (kF32 ? 4 : kChain); ++x)
#pragma unroll
      for (int j = 0; j < NM; ++j) {
        if (x == 0) p[j] = (f32x4){0.f, 0.f, 0.f, 0.f};
        if constexpr (kF32)       // element x of the four lanes' chunks is one k-step of 4 (same columns on both sides)
          p[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(av[0][x]), __uint_as_float(bm[0][j][x]), p[j], 0, 0, 0);
        else
          p[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[x]),
                                                         __builtin_bit_cast(bf16x8, bm[x][j]), p[j], 0, 0, 0);
      }
    const int to = kDirect ? (i + NV - 1) % NV : i;
#pragma unroll
    for (int j = 0; j < NM; ++j) {
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[to][j][e] += (double)(kDirect ? pend[j][e] : p[j][e]);
      if constexpr (kDirect) pend[j] = p[j];
    }
  };
  auto end_step = [&]() {
    if (++cp_k == nk) {                                      // tile finished
      if (live) {
        if constexpr (kDirect) {
#pragma unroll
          for (int j = 0; j < NM; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              acc[NV - 1][j][e] += (double)pend[j][e];
              pend[j][e] = 0.f;
            }
        }
        const int v0 = (stream + cp_tile * n_streams) * VT + wv * (NV * 16) + 4 * c4;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          const int vbase = v0 + 16 * i;
#pragma unroll
          for (int j = 0; j < NM; ++j) {
            const int row = m_wave + 16 * j + n;
            f32x4 lg;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              lg[e] = (float)acc[i][j][e];
              if (vbase + e < V && lg[e] > best[j]) { best[j] = lg[e]; best_i[j] = vbase + e; }   // ascending: lowest wins
              acc[i][j][e] = 0.0;
            }
            if (a.logits != nullptr && row < a.M) store_logits(a.logits + (int64_t)row * V, vbase, V, lg);
          }
        }
      }
      if (kDirect && a.logits != nullptr) wait_loads<0>();   // its stores share the loads' counter
      cp_k = 0;
      ++cp_tile;
    }
  };

  if constexpr (kDirect) {
    // One barrier per step, before the last row of tiles: behind it tile s + 1 is complete in LDS and tile s read
    // for the last time (that row's operands are in registers), so that the step goes on with the hidden rows of
    // tile s + 1 and step s + 1 begins by filling tile s's buffer.  Every load has a step and a half to arrive.
    static_assert(kRow / 64 == kChain, "one chain per step");
    issue(0);
    issue(1);
    wait_loads<kLd>();
    __syncthreads();
    read_m(0, 0);
    int rd = 0, wr = 2;
    for (int s = 0; s < n_steps; ++s) {
      u32x4 av[kChain];
      issue(wr);
      if (live) {
#pragma unroll
        for (int i = 0; i < NV - 1; ++i) {
          read_v(av, rd, 0, i);
          products(av, i);
        }
        read_v(av, rd, 0, NV - 1);
      }
      wait_loads<kLd>();
      __syncthreads();
      rd = rd == 2 ? 0 : rd + 1;
      wr = wr == 2 ? 0 : wr + 1;
      if (live) {
        products(av, NV - 1);
        read_m(rd, 0);
      }
      end_step();
    }
    wait_loads<0>();                                         // the two tiles requested past the end
  } else {
    issue(0);
    for (int s = 0; s < n_steps; ++s) {
      stash();
      __syncthreads();
      issue(0);
      if (live) {
#pragma unroll
        for (int ks = 0; ks < kRow / 64; ks += kChain) {
          read_m(0, ks);
#pragma unroll
          for (int i = 0; i < NV; ++i) {
            u32x4 av[kChain];
            read_v(av, 0, ks, i);
            products(av, i);
          }
        }
      }
      end_step();
      __syncthreads();
    }
  }

  // one candidate per (workgroup, row): the four lanes of a column, then the WV wavefronts of a row
  __syncthreads();
  float *cv = reinterpret_cast<float *>(smem);               // [WV][BM]
  int *ci = reinterpret_cast<int *>(smem + WV * BM * 4);
#pragma unroll
  for (int j = 0; j < NM; ++j) {
    float bv = best[j];
    int bi = best_i[j];
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const float ov = __shfl_xor(bv, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    }
    if (c4 == 0) { cv[wv * BM + wm * (NM * 16) + 16 * j + n] = bv; ci[wv * BM + wm * (NM * 16) + 16 * j + n] = bi; }
  }
  __syncthreads();
  for (int r = tid; r < blocks_m * BM && r < a.M; r += kWaves * 64) {
    float bv = -INFINITY;                                    // rows of the other block: a neutral candidate
    int bi = 0x7fffffff;
    if (r >= row0 && r < row0 + BM) {
      for (int x = 0; x < WV; ++x) {
        const float ov = cv[x * BM + r - row0];
        const int oi = ci[x * BM + r - row0];
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
      }
    }
    a.cand_val[(int64_t)r * a.n_cand + blockIdx.x] = bv;
    a.cand_idx[(int64_t)r * a.n_cand + blockIdx.x] = bi;
  }
}

template <class T, int VT, int BM, int kWaves, int WV, int kRow>
hipError_t launch_tiled_vt(const AcceptArgs &a, hipStream_t st) {
  constexpr int lds = tiled_buffers(kWaves) * (VT + BM) * kRow;
  if (lds > 64 * 1024) {      // has to be allowed once per kernel
    static const hipError_t attr = hipFuncSetAttribute((const void *)lm_head_tiled_kernel<T, VT, BM, kWaves, WV, kRow>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
  }
  hipLaunchKernelGGL((lm_head_tiled_kernel<T, VT, BM, kWaves, WV, kRow>), dim3(a.n_cand), dim3(kWaves * 64), lds, st, a,
                     (a.M + BM - 1) / BM);
  return hipGetLastError();
}

// Workgroups of the tiled kernel on a compute unit.  bf16: one of 8 wavefronts, two up to 64 rows, as registers and
// LDS tiles allow (64 x 128 with 102 registers and 72 KiB would fit twice and runs once, as 128 x 128 does); fp32:
// workgroups of 4, two at 128 rows, three at 64, four below.
int tiled_per_cu(bool f32, int bm) { return f32 ? (bm > 64 ? 2 : bm > 32 ? 3 : 4) : bm > 64 ? 1 : 2; }

// Rows of a vocabulary tile: 128, or 64.  bf16: 64 where all tiles of 64 then fit the chip at once; a second round
// of them takes longer than one of 128 (2,560 x 32,000 at 100 rows, one workgroup per compute unit either way, 57 us
// against 43, 5,120 x 32,000 at 200 rows 147 against 118; 2,048 x 16,384 at 100 rows, 256 tiles of 64, 26).  fp32:
// where tiles of 128 would leave compute units without one (9 rows 56 us).
int tiled_rows(bool f32, int M, int V, int bm) {
  const int blocks_m = (M + bm - 1) / bm;
  if (f32) return (V + 127) / 128 * blocks_m < kNumCU ? 64 : 128;
  return (V + 63) / 64 * blocks_m <= kNumCU * tiled_per_cu(f32, bm) ? 64 : 128;
}

template <class T, int BM, int kWaves, int WV, int kRow>
hipError_t launch_tiled(const AcceptArgs &a, hipStream_t st) {
  return tiled_rows(std::is_same<T, float>::value, a.M, a.V, BM) == 64
             ? launch_tiled_vt<T, 64, BM, kWaves, WV, kRow>(a, st)
             : launch_tiled_vt<T, 128, BM, kWaves, WV, kRow>(a, st);
}

// Workgroups for row blocks of bm: as many as the chip holds, fewer if there are fewer tiles; a multiple of 8 per
// row block.
int tiled_grid(bool f32, int M, int V, int bm) {
  const int blocks_m = (M + bm - 1) / bm, vt = tiled_rows(f32, M, V, bm);
  const int tiles = (V + vt - 1) / vt;
  const int per_block = kNumCU * tiled_per_cu(f32, bm) / (8 * blocks_m) * 8;
  return std::min(per_block, (tiles + 7) / 8 * 8) * blocks_m;
}
int f32_block(int M) { return M <= 16 ? 16 : M <= 32 ? 32 : M <= 64 ? 64 : 128; }

// Up to here the k-split kernel, whose hidden rows sit in registers: one row block.  Against the tiled kernel at 32
// rows, us: 152,064 x 3584 171 / 167, 64,003 x 2048 53 / 57, 40,003 x 1024 26.7 / 23.5, 32,000 x 2560 38 / 34: either
// way by width and vocabulary up to 4,096 columns; above, where 17 rows need a second pass over W, 32,000 x 5120
// 112 / 60.
//
// Above that line the k-split kernel, all its row blocks side by side, where the vocabulary is too small to fill
// the chip with tiles of the whole hidden size: the tiled kernel then lasts some 0.6 us per 64 columns, one step
// after the other, a k-split workgroup 4 us per 16-row tile (6 with two slices per wavefront), whatever the width.
// The rule's 0.8 us are those of the tiled kernel through registers: it estimates today's a third too high, the
// k-split kernel 5 per cent.  180 drawn shapes that it gives to the k-split kernel, k-split / tiled in us with the
// finalize pass: 1,221 x 6,280 at 155 rows 26 / 91, 1,476 x 8,120 at 62 rows 23 / 66, 11,134 x 3,080 at 56 rows 31 /
// 33; 1.49 times as fast in the median, and for ten of them slower, by up to a sixth, where the two estimates are
// close (6,229 x 768 at 43 rows 14.8 / 12.3, 14,547 x 7,464 at 34 rows 82 / 72).
bool ksplit_small(int M, int H, int V) {
  if (M <= ksplit_rows(H) || H > 2 * kKsWaves * kKsSlice) return false;
  const int blocks = ksplit_blocks(M, H), grid = ksplit_grid(H, V, blocks);
  const int rounds = ((V + 15) / 16 + grid - 1) / grid * ((blocks * grid + ksplit_slots(H) - 1) / ksplit_slots(H));
  return (ksplit_wide(H) ? 6 : 4) * rounds + 8 < 6 + H / 80;
}

}  // namespace

bool lm_head_mfma_supported(int dtype, int M, int H, int V) {
  (void)M; (void)V;
  if (dtype == SPARROW_F32) return H % 4 == 0 && H <= (1 << 20);
  return dtype == SPARROW_BF16 && H % 8 == 0 && H <= 2 * kKsWaves * kKsSlice;     // two slices per wavefront
}

int accept_num_candidates(int dtype, int M, int H, int V) {
  if (dtype == SPARROW_F32) return tiled_grid(true, M, V, f32_block(M));
  if (ksplit_small(M, H, V)) return ksplit_grid(H, V, ksplit_blocks(M, H));
  return M > ksplit_rows(H) ? tiled_grid(false, M, V, M > 128 ? 256 : M > 64 ? 128 : 64) : ksplit_grid(H, V, 1);
}

hipError_t launch_lm_head_mfma(int dtype, const AcceptArgs &a, hipStream_t st) {
  if (dtype == SPARROW_F32) {
    switch (f32_block(a.M)) {
      case 16: return launch_tiled<float, 16, 4, 4, 256>(a, st);
      case 32: return launch_tiled<float, 32, 4, 4, 256>(a, st);
      case 64: return launch_tiled<float, 64, 4, 2, 128>(a, st);
      default: return launch_tiled<float, 128, 4, 2, 128>(a, st);
    }
  }
  const bool wide = ksplit_wide(a.H);
  if (ksplit_small(a.M, a.H, a.V)) {
    const int blocks = ksplit_blocks(a.M, a.H);
    return wide ? launch_ksplit<2, 1>(a, blocks, st) : launch_ksplit<1, 2>(a, blocks, st);
  }
  if (a.M > 128) return launch_tiled<bf16_t, 256, 8, 2, 128>(a, st);
  if (a.M > 64) return launch_tiled<bf16_t, 128, 8, 2, 128>(a, st);
  if (a.M > ksplit_rows(a.H)) return launch_tiled<bf16_t, 64, 8, 2, 128>(a, st);
  if (wide) return launch_ksplit<2, 1>(a, 1, st);
  return a.M > 16 ? launch_ksplit<1, 2>(a, 1, st) : launch_ksplit<1, 1>(a, 1, st);
}

}  // namespace sparrow
