// Verification attention, matrix-core partial pass: bf16, head_dim 128 or 64, gfx950.
//
// One workgroup (8 wavefronts) owns one (context split, KV head, block of 64, 128 or 192 rows); a row is a
// (draft row, query head of the group) pair, so all rows of a block share the K/V stream.
// The workgroup runs two token streams (wavefronts 0-3 and 4-7) that take alternate 32-token
// tiles; within a stream wavefront w owns rows 16w..16w+15 of each 64 of the block, so rows are never merged
// between wavefronts and the two streams are merged once, through LDS, at the end.
// K/V tiles travel HBM -> registers (coalesced 16-byte loads, several tiles in flight) -> LDS
// (XOR-swizzled 16-byte chunks, double buffered per stream) and are read by the four wavefronts
// of the stream.
//
// Per tile and wavefront, with v_mfma_f32_16x16x32_bf16 (A: 16 x 32, lane = row + 16*kchunk;
// B: 32 x 16, lane = column + 16*kchunk; D: 16 x 16, lane = column + 16*(row/4), 4 rows each):
//   S^T = K Q^T   A = K rows from LDS (ds_read_b128), B = Q^T kept in registers.
//                 A lane then holds, for its query row, the scores of tokens 4c+0..3 (c = lane/16)
//                 of each 16-token sub-tile: the row max needs two cross-lane steps only.
//   O^T += V^T P^T  B = P^T straight from the score registers (k index = the lane's own eight
//                 tokens), A = V^T through the transposing LDS read ds_read_b64_tr_b16.
// The online-softmax state (m, l) and the rescale factor are per lane (= per query row).
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "verify_attn.hpp"

namespace sparrow {

namespace {

constexpr int kTile = 32;                 // tokens per tile
constexpr int kRowsPerWG = 64;
constexpr int kStreams = 2;
constexpr float kSlack = 8.0f;            // log2 units a score may exceed a row's reference point

// Swizzle of the 16-byte chunk index by the token row: chunk c of row r is stored at chunk position
// c ^ ((r & 7) << 1).  Measured with the bank-conflict counter on the three access patterns of this
// kernel (16-byte writes of whole rows, 16-byte reads of 16 rows at one chunk, transposing 8-byte
// reads of 16 rows x 32 bytes): no conflict cycle on any of them.  Variants that also fold bit 3
// of the row in (so that rows r and r + 8 land on different chunks) doubled the cycles of the
// 16-byte operand reads -- two thirds of the kernel's LDS cycles were bank conflicts with it.
// With 128-byte rows (head_dim 64) two consecutive rows share the 256 bytes of one bank line, so the
// parity of the row picks the half line and the next two bits the swizzle: the eight rows r .. r+7
// land on eight different 16-byte columns, as they do with 256-byte rows.
template <int kD> __device__ __forceinline__ int swz(int row) {
  return kD == 128 ? (row & 7) << 1 : ((row >> 1) & 3) << 1;
}

__device__ __forceinline__ bf16x8 lds_read_b128(const unsigned char *p) {
  return *reinterpret_cast<const bf16x8 *>(p);
}

__device__ __forceinline__ bf16x4 lds_read_tr(const unsigned char *p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4 *)p);
}

// max / sum over the four lanes l, l^16, l^32, l^48 (the four k-chunk lanes of one query row),
// with the gfx950 row-swap instructions (no LDS round trip).
__device__ __forceinline__ float quad_max(float v) {
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

// kQT = 16-row tiles per wavefront: 1 serves up to 64 rows per workgroup (chains), 2 and 3 serve
// 128 and 192 (draft trees): the K and V^T operands read from LDS then feed every row tile, and a
// tree of R rows needs a half or a third as many passes over the K/V stream.  Three tiles take
// all 256 registers with one step in flight.
// kPrefetch = steps in flight in registers.  The whole split of a workgroup is only a handful of
// steps at decode-time sizes (7 at 26k context on 256 compute units), so a deep look-ahead turns
// the kernel into "load most of it, then compute": depth 3-4 is slower there, depth 2 wins from
// about four steps on, depth 1 for the shortest splits.
// Per-sequence split length in tokens (split_len of the sequence), worked out by the host so that
// the kernel's way to its first load holds no integer division.
struct PieceTable {
  int32_t piece[SPARROW_MAX_BATCH];
};

// What `shape` of the partial pass holds beside the row blocks (from bit 3 up)
constexpr int kShapeFlat = 1, kShapeDirect = 2, kShapeTable = 4, kShapeBits = 3;

// Heads of 64 keep the intermediate state of an attention row in 32 bits (as the plain-ALU kernel
// does): probabilities enter the output MFMA as three bf16 terms that add up to their 24 bits, row
// sums are added up on the vector ALU, split partials are stored in fp32.  Heads of 128 round
// probabilities to bf16 and partials to fp16.  The second and third output MFMA of a tile are mostly
// hidden: with 64-wide heads a token brings half the bytes and the same number of scores, and the kernel
// waits for memory or for the softmax.  Against two terms (16 bits of a probability): four ragged
// sequences of 6,001, 16/4 heads, chain of 8, 14.0 -> 14.5 us a call; 60-node tree at 26k 36.4 -> 39 to 41.
template <int kD> constexpr bool kWideState = kD == 64;

// kPing (two row tiles, several row blocks, long splits) runs its two streams half a step apart: while one stream's
// wavefronts issue the MFMAs of a step (scores of the next tile, output of this one), the other stream's, which
// share the SIMDs with them, are in their softmax.  In step, the phases of all wavefronts add up: matrix
// cores, vector ALU and LDS were busy 27, 31 and 42 per cent of the time.  The LDS reads of V^T, the LDS
// writes and the requests of later tiles are issued between the MFMAs; independent sums alternate.
// In step / half a step apart, us a call with the combine pass, in an unbroken row of calls, on two cards: 60-node
// tree over 26,112 tokens (28/4 heads) 38.5 / 35.8 and 40.2 / 39.4, two of 64 nodes over 30,000 (64/8 heads) 147 /
// 135 (930 TFLOP/s) and 158 / 144.  Three row tiles and the fp32 state of heads of 64 do not leave the registers
// for it (the latter 42 -> 67 us with spills); which calls take it: half_step_pays below.

// kTilesOfRows = 0 (heads of 64, at most 32 rows per KV head): two of a stream's four wavefronts would have no row.  All
// four have rows 0..31 between them twice, and of the two tiles of a step each pair takes one, so that scores and
// exponentials, which set the pace with two wavefronts, take half as long; four states of a row meet at the end instead
// of two.  One step in flight: two are slower here (124 registers against 99).  us a call with the combine pass, two
// wavefronts / all: four ragged sequences of 6,001, 16/4 heads, chain of 8 12.9 / 12.3, eight of 3,000, 32/8, 8 19.6 /
// 16.7, sixteen of 3,000, 16/4, one row 19.35 / 16.1, six of 9,000, 32/4, 4 20.0 / 16.8, one of 26,000, 14/2, 2 12.9 /
// 12.2, of 24,004, 16/4, 8 13.5 / 13.0; with two steps in flight 12.9, 17.1, 16.9, 17.4, 12.9, 13.6.  In one piece of up to two
// steps, without a combine pass: one of 60, 4/2, 4 4.1 / 3.9, four of 200, 16/4, 4 6.0 / 5.2, sixteen of 250, 8/8, 16 7.5 / 6.8.
// kD = head size.  A step of a stream stages 8 KB of K and 8 KB of V at either size: one tile of 32
// tokens at kD = 128, two at 64, so the loads in flight and the barriers per byte are the same.
// LDS of a workgroup: two buffers of K and V tiles a stream.  After the main loop the first part is reused for the merge: 1 KB
// a d-tile that one wavefront sends another (kPairs: three by each of eight; else as many as a row has, by each of four pairs),
// then 8 bytes a lane of (m, l).
template <int kD> constexpr int kLdsBytes = kStreams * 2 * 2 * (128 / kD) * kTile * kD * 2;
template <int kD, bool kPairs> constexpr int kMergeTiles = (kPairs ? 24 : 4 * (kD / 16)) * 1024;
template <int kD, bool kPairs> constexpr int kMergeBytes = kMergeTiles<kD, kPairs> + 4 * kStreams * 64 * 8;
template <int kD, int kPrefetch, int kTilesOfRows, bool kPing>
__global__ void __launch_bounds__(256 * kStreams)
verify_partial_mfma_kernel(const void *k_base, const void *v_base, int64_t stride_head, int stride_tok, int cl0_one,
                           int len_one, int ns_one, int piece_one, int n_slots, int shape, VerifyArgs a, SeqTable tab,
                           PieceTable pt) {
  constexpr bool kPairs = kTilesOfRows == 0;
  constexpr int kQT = kPairs ? 1 : kTilesOfRows;
  constexpr int kSub = 128 / kD;                           // 32-token tiles per stream per step
  constexpr int kRowBytes = 2 * kD;                        // one K or V row of a head
  constexpr int kChunks = kD / 8;                          // 16-byte chunks of a row
  constexpr int kLdRows = 256 / kChunks;                   // token rows that one load of a stream covers
  constexpr int kSubW = kPairs ? 1 : kSub;                 // 32-token tiles of a wavefront per step
  constexpr int kSlabs = 2 * kSubW;                        // 16-token slabs of a wavefront per step
  static_assert(!kPairs || (kSub == 2 && kQT == 1 && !kPing), "two tiles a step, rows for two wavefronts");
  constexpr int kKS = kD / 32, kMT = kD / 16;              // MFMA k-steps of a score, 16-wide d-tiles
  constexpr bool kWide = kWideState<kD>;
  constexpr bool kShare = !kPing;                          // both streams merge and store
  // [stream][buf][K,V][kSub tiles]; the merge takes 36 KB of it (heads of 64: 20, kPairs 28)
  static_assert(kMergeBytes<kD, kPairs> <= kLdsBytes<kD>, "the merge reuses the tiles' LDS");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  constexpr int kStepBytes = kSub * kTile * kRowBytes;     // K (or V) rows of one stream step
  static_assert(kLdsBytes<kD> == kStreams * 2 * 2 * kStepBytes, "");
  auto lds_at = [&](int strm_, int buf, int kv) {
    return lds + ((strm_ * 2 + buf) * 2 + kv) * kStepBytes;
  };

  // wavefront-uniform indices as scalars, so that everything derived from them (which rows are
  // live, whether a step touches the split end) is decided by scalar branches
  const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int strm = wave_id >> 2, w = wave_id & 3;
  const int tid = threadIdx.x & 255, lane = threadIdx.x & 63;
  const int n = lane & 15, c4 = lane >> 4;
  const int wr = kPairs ? w & 1 : w, u0 = kPairs ? w >> 1 : 0;      // rows 16 wr .. of each 64; first tile of a step
  const int part = kPairs ? strm * 2 + u0 : strm;         // of the wavefronts that hold a row
  // Workgroup -> (sequence, KV head, split of the sequence, row block).  Workgroups are handed to
  // the 8 XCDs round-robin by their linear index and gridDim.x is a multiple of 8, so x & 7 is
  // the XCD; the row blocks of one split stream the same K/V and get x values that are equal
  // modulo 8 and adjacent in that XCD's order: they run at the same time on one XCD and all but
  // the first fetch of a tile hit its L2.  (Only the speed depends on the round-robin placement.)
  // Two grid shapes:
  //  - (x, KV head, sequence): x is sized for the sequence with the most splits; the XCD of a split is rotated by
  //    its global number, so that the splits of all heads and sequences together are dealt evenly to the XCDs.
  //  - flat (x only; for ragged batches, where the first shape would launch mostly padding):
  //    x enumerates (global split, KV head) and the sequence is searched in the split table.
  // At decode-time sizes the whole kernel lasts 6 to 13 us and every dependent round trip before the first load
  // shows.  The arguments that it needs are leading scalars, which reach the registers with the launch: one sequence, or
  // several of one length, read nothing before it.  Sequences that differ read their table entries, a line of the arguments
  // or two, 0.4 us; the flat grid the table and then the entries.  (One round of loads of all arguments before: chain of 5
  // over 8,192 tokens 11.5 us a call, now 11.3, both with the combine pass of that time.)
  const int xj = blockIdx.x >> 3, xcd = blockIdx.x & 7;
  const int rbs = shape >> kShapeBits;
  const bool flat = (shape & kShapeFlat) != 0, direct = (shape & kShapeDirect) != 0;
  int rb = 0, sq = xj;
  if (rbs > 1) { rb = xj % rbs; sq = xj / rbs; }
  int b = 0, c, s_loc, cl0 = cl0_one, len = len_one, cs0 = 0, ns = ns_one, piece = piece_one;
  if (flat) {
    const int grp = sq * 8 + xcd;                          // global split + n_slots * KV head
    if (grp >= len_one) return;                            // padding of the last round of 8
    const QuotRest cg = div_uniform(grp, n_slots);
    const int gslot = cg.rest;
    c = cg.quot;
    // (an empty statement that takes these as scalar-register inputs: their lines come with the ends that the search reads,
    // and the entries of the sequence found are then at hand)
    asm volatile("" ::"s"(tab.cu_len[0]), "s"(tab.cu_len[16]), "s"(pt.piece[0]), "s"(pt.piece[15]), "s"(tab.cu_split[0]),
                 "s"(tab.cu_split[1]), "s"(tab.cu_split[16]));
    b = seq_of_slot(tab, gslot);
    cl0 = tab.cu_len[b]; len = tab.cu_len[b + 1] - cl0;
    cs0 = tab.cu_split[b]; ns = tab.cu_split[b + 1] - cs0;
    piece = pt.piece[b];
    s_loc = gslot - cs0;
  } else {
    c = blockIdx.y;
    b = blockIdx.z;
    if (!(shape & kShapeTable)) {                          // sequences of one length (or one sequence): no table is read
      cl0 += b * len;
      cs0 = b * ns;
    } else {
      cl0 = tab.cu_len[b]; len = tab.cu_len[b + 1] - cl0;
      cs0 = tab.cu_split[b]; ns = tab.cu_split[b + 1] - cs0;
      piece = pt.piece[b];
      // an empty statement that takes these values as scalar-register inputs: the compiler has to have all of them
      // loaded here, which makes it issue their loads together, instead of one round per use
      asm volatile("" ::"s"(cl0), "s"(len), "s"(cs0), "s"(ns), "s"(piece));
    }
    s_loc = sq * 8 + ((xcd - (cs0 + n_slots * c)) & 7);    // split within the sequence
    if (s_loc >= ns) return;                               // padding of the grid (uniform)
  }
  const int slot = cs0 + s_loc;
  const int t0 = min(len, s_loc * piece);
  const int t1 = min(len, t0 + piece);
  const int n_tiles = (t1 - t0 + kTile - 1) / kTile;                    // of the workgroup
  const int n_steps = (n_tiles + kStreams * kSub - 1) / (kStreams * kSub);   // loop trips
  // K/V of this sequence and head; a token row is addressed by a 32-bit byte offset from here
  // (the host checks that a sequence's K/V spans less than 2 GB)
  const int64_t seq_off = (int64_t)cl0 * stride_tok + (int64_t)c * stride_head;
  const unsigned char *Kg = (const unsigned char *)((const bf16_t *)k_base + seq_off);
  const unsigned char *Vg = (const unsigned char *)((const bf16_t *)v_base + seq_off);
  const unsigned int row_bytes = (unsigned int)stride_tok * 2u;

  // ---- loader: in step `st` stream `strm` owns tiles (st*kStreams + strm)*kSub .. +kSub, i.e.
  // 32*kSub consecutive tokens; thread -> rows tid/kChunks + kLdRows j, 16-byte chunk tid%kChunks.  Rows past
  // the end of the split are clamped to its last token (their probability is zero), so every load is
  // unconditional and the number of loads in flight is a compile-time constant at every wait.
  const int ld_row = tid / kChunks, ld_ch = tid % kChunks;
  constexpr int kLd = kSub * kTile / kLdRows;         // loads per step (per K and per V)
  // (A request far past the end of the split may wrap around 2^32 where rows are megabytes apart: it still lies
  // between the sequence's first row and ld_last, and no step of the split reads what it brings.)
  const unsigned int ld_first = (unsigned int)(t0 + ld_row) * row_bytes + (unsigned int)ld_ch * 16u;
  const unsigned int ld_last = (unsigned int)(t1 - 1) * row_bytes + (unsigned int)ld_ch * 16u;
  auto issue1 = [&](const unsigned char *src, int st, int j, u32x4 *sg) __attribute__((always_inline)) {
    const unsigned int to = (unsigned int)((st * kStreams + strm) * kSub * kTile + kLdRows * j) * row_bytes;
    sg[j] = __builtin_nontemporal_load((const u32x4 *)(src + min(ld_first + to, ld_last)));
  };
  auto issue = [&](const unsigned char *src, int st, u32x4 *sg) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < kLd; ++j) issue1(src, st, j, sg);
  };
  // row r of the step lands at byte r*kRowBytes + ((chunk ^ swz(r)) * 16); swz depends on r mod 8 only
  const int st_off = ld_row * kRowBytes + ((ld_ch ^ swz<kD>(ld_row)) << 4);
  auto stash1 = [&](int buf, int kv, int st, int j, u32x4 *sg) __attribute__((always_inline)) {
    if (kPing && kv == 1) {                                // values past the end of the split: zero
      const int left = t1 - (t0 + (st * kStreams + strm) * kSub * kTile);
      if (left < kSub * kTile && ld_row + kLdRows * j >= left) sg[j] = (u32x4){0u, 0u, 0u, 0u};
    }
    *reinterpret_cast<u32x4 *>(lds_at(strm, buf, kv) + st_off + kLdRows * j * kRowBytes) = sg[j];
  };
  auto stash = [&](int buf, int kv, int st, u32x4 *sg) __attribute__((always_inline)) {
    if (kWide && kv == 1) {
      // values past the end of the split are zero, as in the plain-ALU kernel: a duplicate of an
      // infinite last row would give 0 * inf.  One test per step, uniform over the wavefront (tested load by
      // load: 0.2 us a call)
      const int left = t1 - (t0 + (st * kStreams + strm) * kSub * kTile);
      if (left < kSub * kTile) {
#pragma unroll
        for (int j = 0; j < kLd; ++j)
          if (ld_row + kLdRows * j >= left) sg[j] = (u32x4){0u, 0u, 0u, 0u};
      }
    }
#pragma unroll
    for (int j = 0; j < kLd; ++j) stash1(buf, kv, st, j, sg);
  };
  // kPing: K runs one step ahead of V, so K of the second step is asked for with the first
  u32x4 kst[kPrefetch][kLd], vst[kPrefetch][kLd];
  u32x4 k_next[kLd];

  // ---- first step, then Q^T (B operand of the score MFMA: lane (n, c4) holds
  // Q[row][32*ks + 8*c4 .. +8]), then the rest of the look-ahead.
  issue(Kg, 0, kst[0]);
  issue(Vg, 0, vst[0]);
  if (kPing) issue(Kg, 1, k_next);
  __builtin_amdgcn_sched_barrier(0);      // the first step is on its way before anything else is worked out

  const int L = len - a.n_q;
  const int g = a.g;
  const int R = a.n_q * g;
  // ---- this lane's query rows: one per row tile
  bool row_ok[kQT];
  int i_row[kQT], h[kQT];                         // h: within the KV head's group
  int n_act = 0;                                  // row tiles of this wavefront that hold rows
#pragma unroll
  for (int qt = 0; qt < kQT; ++qt) {
    const int rho = (rb * kQT + qt) * kRowsPerWG + 16 * wr + n;
    row_ok[qt] = rho < R;
    if ((rb * kQT + qt) * kRowsPerWG + 16 * wr < R) n_act = qt + 1;
    // rows past R take the data of row 0 (in bounds); what comes of them is not used
    const QuotRest rh = row_and_head(rho, g, a.inv_g);
    i_row[qt] = row_ok[qt] ? rh.quot : 0;
    h[qt] = row_ok[qt] ? rh.rest : 0;
  }
  const int64_t q_row0 = (int64_t)b * a.n_q * a.Hq + (int64_t)c * g;     // of the call: row (b, 0), first head of the group

  u32x4 qv[kQT][kKS];
#pragma unroll
  for (int qt = 0; qt < kQT; ++qt) {
    const int64_t at = (int64_t)(i_row[qt] * a.Hq + h[qt]) * (2 * kD) + 16 * c4;      // (64 rows of 266,305 heads pass 4 GiB)
    const unsigned char *qp = (const unsigned char *)a.q + q_row0 * (2 * kD) + at;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) qv[qt][ks] = *(const u32x4 *)(qp + 64 * ks);
  }
  // The memory pipeline of a compute unit serves requests in issue order and a wavefront
  // issues all its loads back to back: without this barrier the look-ahead of the wavefronts
  // that issue first would queue ahead of the FIRST step of the others (measured: 3 us of
  // skew between the two streams).
  if (kPrefetch > 1) __syncthreads();
#pragma unroll
  for (int p = 1; p < kPrefetch; ++p) {
    issue(Vg, p, vst[p]);
    issue(Kg, kPing ? p + 1 : p, kst[p]);
  }
  // Loads retire in order: Q (and the first step before it) have landed once at most the
  // loads issued after Q are outstanding (other counters untouched).
  constexpr int kAfterQ = (kPrefetch - 1) * 2 * kLd;
  static_assert(kAfterQ < 64, "vmcnt is a 6-bit counter");
  bf16x8 qreg[kQT][kKS];
  auto take_q = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0x0F70 | (kAfterQ & 15) | ((kAfterQ >> 4) << 14));
#pragma unroll
    for (int qt = 0; qt < kQT; ++qt)
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks) qreg[qt][ks] = __builtin_bit_cast(bf16x8, qv[qt][ks]);
  };
  if (kQT > 1) take_q();                          // (what follows has no registers to wait in)
  // draft rows a row may attend (bit j <=> draft row j); only needed if the split reaches them
  unsigned long long anc[kQT];
#pragma unroll
  for (int qt = 0; qt < kQT; ++qt) {
    anc[qt] = 0ull;
    if (t1 > L) {                                            // uniform over the workgroup
      anc[qt] = ancestor_mask_wave(a.parent ? a.parent + (int64_t)b * a.parent_stride : nullptr, a.n_q,
                                   i_row[qt], lane);
      if (!row_ok[qt]) anc[qt] = 0ull;
    }
  }

  // LDS read offsets
  const int k_off = n * kRowBytes;                 // + 16-row slab, chunk (4*ks + c4) ^ swz(n)
  const int k_swz = swz<kD>(n);
  const int s16 = lane & 15;                       // source lane index within the 16-lane group
  const int v_row = 4 * c4 + (s16 >> 2);           // token within a 16-token slab
  // (o_acc[.][i] is d-tile i ^ (the first of the wavefront's own), chosen by the chunks that it reads)
  const int v_swz = swz<kD>(v_row) ^ (kPairs ? 2 * part : kShare ? kMT * strm : 0);
  const int v_off = v_row * kRowBytes + ((s16 & 1) << 3);   // + chunk (2*mt + ((s16>>1)&1)) ^ swz
  const int v_chb = (s16 >> 1) & 1;

  float m_run[kQT];
  f32x4 l_acc[kQT];       // running sum of a row's exponentials, the same value in all 4 entries
  f32x4 o_acc[kQT][kMT];
  constexpr bool kMfmaRowSum = !kWide;
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int qt = 0; qt < kQT; ++qt) {
      m_run[qt] = kNegBig;
      l_acc[qt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int mt = 0; mt < kMT; ++mt) {
        o_acc[qt][mt] = (f32x4){0.f, 0.f, 0.f, 0.f};
        if (kQT == 1) asm volatile("" : "+v"(o_acc[qt][mt]));     // now, and not behind the wait
      }
    }
  };
  if (kQT == 1) clear();                          // (several row tiles have no registers to spare for it)
  if (kQT == 1) take_q();
  if (kQT > 1) clear();

  f32x4 s[kQT][kSlabs];                           // scores of a step, S^T
  bf16x8 pb[kQT][kSubW];                          // its probabilities, P^T
  bf16x8 pm[kWide ? kQT : 1][kSubW], pl[kWide ? kQT : 1][kSubW];   // kWide: what pb leaves of the probability
  bf16x8 ka[kSlabs][kKS];                         // K operands of a step
  auto read_k = [&](int buf, int j) __attribute__((always_inline)) {
    const unsigned char *Ks = lds_at(strm, buf, 0);
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks)
      ka[j][ks] = lds_read_b128(Ks + (2 * u0 + j) * 16 * kRowBytes + k_off + (((4 * ks + c4) ^ k_swz) << 4));
  };
  auto scores = [&](int j) __attribute__((always_inline)) {
#pragma unroll
    for (int qt = 0; qt < kQT; ++qt) s[qt][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
      for (int qt = 0; qt < kQT; ++qt)
        s[qt][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[j][ks], qreg[qt][ks], s[qt][j], 0, 0, 0);
  };
  // One joint softmax update of a step (a single running-max / rescale for its 32*kSub tokens).
  auto softmax = [&](int st) __attribute__((always_inline)) {
    const int tb = t0 + ((st * kStreams + strm) * kSub + u0) * kTile;
    // mask, online softmax (per lane = per query row).  Scores stay unscaled until the exponent:
    // exp2(s * scale_log2 - m) is one fused multiply-add per score (scale_log2 > 0, so the
    // maximum can be taken before scaling).
    const bool edge = tb + kSubW * kTile > min(t1, L);   // uniform: split end or draft rows in reach
#pragma unroll
    for (int qt = 0; qt < kQT; ++qt) {
      float sc[4 * kSlabs];       // (as elements of s the maxima cost an instruction more per score)
#pragma unroll
      for (int e = 0; e < 4 * kSlabs; ++e) sc[e] = s[qt][e >> 2][e & 3];
      if (edge) {
        // (an opaque copy of the step's first token: without it the compiler works the token
        // numbers, their distances to L and the shift counts out on EVERY step, ahead of the
        // branch -- some 20 vector instructions per row tile that all but one step throw away)
        int tb_e = tb;
        asm volatile("" : "+v"(tb_e));
#pragma unroll
        for (int j = 0; j < kSlabs; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int tok = tb_e + 16 * j + 4 * c4 + i;
            const int dj = tok - L;
            const bool vis = (dj < 0) | (((anc[qt] >> (dj & 63)) & 1ull) != 0ull);
            sc[4 * j + i] = ((tok < t1) & vis) ? sc[4 * j + i] : -INFINITY;
          }
      }
      float mx = sc[0];
#pragma unroll
      for (int e = 1; e < 4 * kSlabs; ++e) mx = fmaxf(mx, sc[e]);
      mx *= a.scale_log2;
      // The reference point m of a row moves only when some score of the wavefront's tile lies
      // more than kSlack above it (exponentials then stay below 2^kSlack, far from overflow, and
      // softmax does not depend on the reference point): the cross-lane maximum, the rescale
      // factor and the 32 accumulator multiplies are skipped for almost every tile.
      if (__builtin_amdgcn_ballot_w64(mx > m_run[qt] + kSlack) != 0ull) {
        const float m_new = fmaxf(m_run[qt], quad_max(mx));
        const float alpha = fast_exp2(m_run[qt] - m_new);
        m_run[qt] = m_new;
        if (st > 0) {                                        // (of the first step nothing has been added up)
          if (kMfmaRowSum) l_acc[qt] *= alpha; else l_acc[qt][0] *= alpha;
#pragma unroll
          for (int mt = 0; mt < kMT; ++mt) o_acc[qt][mt] *= alpha;
        }
      }
#pragma unroll
      for (int u = 0; u < kSubW; ++u) {
        float psum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float p = fast_exp2(fmaf(sc[8 * u + e], a.scale_log2, -m_run[qt]));
          if (!kMfmaRowSum) psum += p;
          if (kWide) {
            // p = hi + mid + lo: the leading 8 bits (cut off, so that the rest has p's sign), the
            // next 8, the last 8.  Where hi is not zero the others are at least 2^-126 (the median:
            // rest < hi), far below p, so that an infinite V gives an infinity here and no 0 * inf.
            const float hi = __uint_as_float(__float_as_uint(p) & 0xffff0000u);
            const float rest = __builtin_amdgcn_fmed3f(p - hi, 0x1p-126f, hi);
            const float mid = __uint_as_float(__float_as_uint(rest) & 0xffff0000u);
            pb[qt][u][e] = (__bf16)hi;
            pm[qt][u][e] = (__bf16)mid;
            pl[qt][u][e] = (__bf16)__builtin_amdgcn_fmed3f(rest - mid, 0x1p-126f, mid);
          } else {
            pb[qt][u][e] = (__bf16)p;
          }
        }
        if (!kMfmaRowSum) l_acc[qt][0] += psum;   // (merged across the four lanes at the end)
      }
    }
  };
  auto read_v = [&](const unsigned char *Vs, int mt, int u) __attribute__((always_inline)) {   // V^T operand
    const unsigned char *at = Vs + v_off + (((2 * mt + v_chb) ^ v_swz) << 4);
    const bf16x4 va = lds_read_tr(at + (2 * (u0 + u)) * 16 * kRowBytes);
    const bf16x4 vb = lds_read_tr(at + (2 * (u0 + u) + 1) * 16 * kRowBytes);
    return (bf16x8)__builtin_shufflevector(va, vb, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  // row sums on the matrix cores: every row of ones . P^T is the sum over the 32 tokens
  auto row_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int qt = 0; qt < kQT; ++qt)
#pragma unroll
      for (int u = 0; u < kSubW; ++u)
        l_acc[qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[qt][u], l_acc[qt], 0, 0, 0);
  };
  auto output = [&](int buf) __attribute__((always_inline)) {
    const unsigned char *Vs = lds_at(strm, buf, 1);
    if (kMfmaRowSum) row_sums();
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt) {
      if (kQT > 1 && mt == 4) __builtin_amdgcn_sched_barrier(0);    // at most 4 d-tiles of V^T in flight
#pragma unroll
      for (int u = 0; u < kSubW; ++u) {
        const bf16x8 vt = read_v(Vs, mt, u);
#pragma unroll
        for (int qt = 0; qt < kQT; ++qt) {
          o_acc[qt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt, pb[qt][u], o_acc[qt][mt], 0, 0, 0);
          if (kWide) {
            o_acc[qt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt, pm[qt][u], o_acc[qt][mt], 0, 0, 0);
            o_acc[qt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt, pl[qt][u], o_acc[qt][mt], 0, 0, 0);
          }
        }
      }
    }
  };

  // A wavefront with a partly filled set of row tiles computes all of them (the empty ones on a zero
  // query): a second, one-tile instance of the step in the same kernel costs more registers than
  // the kernel has.
  // Steps of this stream that hold tokens (none for a wavefront without rows)
  const int my_steps = n_act > 0 ? (n_tiles - strm * kSub - u0 + kStreams * kSub - 1) / (kStreams * kSub) : 0;
  if constexpr (kPing) {
    // Step st of a stream: vector phase (K operands of step st + 1 out of LDS, softmax of st), barrier,
    // matrix phase (scores of st + 1, output of st; V of st + 1 and K of st + 2 into LDS, their successors
    // requested), barrier.  Steps past the stream's last tile run on masked scores and zero values.
    static_assert(!kWide && kSub == 1 && kPrefetch == 2, "the instance that runs this");
    stash(0, 0, 0, kst[0]);
    stash(0, 1, 0, vst[0]);
    stash(1, 0, 1, k_next);
    issue(Vg, 2, vst[0]);
    issue(Kg, 3, kst[0]);
    __syncthreads();
    if (strm == 1) __syncthreads();                        // half a step behind
    if (n_act > 0) {
#pragma unroll
      for (int j = 0; j < kSlabs; ++j) { read_k(0, j); scores(j); }
    }
    __syncthreads();
    auto fetch1 = [&](int st, int p, int x) __attribute__((always_inline)) {   // p = st & 1; x: V's loads, then K's
      if (x < kLd) {
        stash1(p ^ 1, 1, st + 1, x, vst[p ^ 1]);
        issue1(Vg, st + 3, x, vst[p ^ 1]);
      } else {
        stash1(p, 0, st + 2, x - kLd, kst[p ^ 1]);
        issue1(Kg, st + 4, x - kLd, kst[p ^ 1]);
      }
    };
    auto step = [&](int st, auto parity) __attribute__((always_inline)) {
      constexpr int p = decltype(parity)::value;           // st & 1
#pragma unroll
      for (int j = 0; j < kSlabs; ++j) read_k(p ^ 1, j);
      softmax(st);
      __syncthreads();
      __builtin_amdgcn_s_setprio(1);
      const unsigned char *Vs = lds_at(strm, p, 1);
      bf16x8 vt[kMT];
#pragma unroll
      for (int qt = 0; qt < kQT; ++qt)
#pragma unroll
        for (int j = 0; j < kSlabs; ++j) s[qt][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < kMT; ++i) {                    // four independent sums alternate
        const int j = i % kSlabs, ks = i / kSlabs;
        vt[i] = read_v(Vs, i, 0);
#pragma unroll
        for (int qt = 0; qt < kQT; ++qt)
          s[qt][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[j][ks], qreg[qt][ks], s[qt][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int mt = 0; mt < kMT; ++mt) {
#pragma unroll
        for (int qt = 0; qt < kQT; ++qt)
          o_acc[qt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[mt], pb[qt][0], o_acc[qt][mt], 0, 0, 0);
        if (mt < 2 * kLd) fetch1(st, p, mt);
        __builtin_amdgcn_sched_barrier(0);
      }
      row_sums();
      __builtin_amdgcn_s_setprio(0);
      __syncthreads();
    };
    auto idle_step = [&](int st, auto parity) __attribute__((always_inline)) {   // a wavefront without rows only loads
      __syncthreads();
#pragma unroll
      for (int x = 0; x < 2 * kLd; ++x) fetch1(st, decltype(parity)::value, x);
      __syncthreads();
    };
    // (Pairs of steps and a remainder, not one loop with two exits, and a loop of its own for idle wavefronts: the
    // compiler then knows which loads are under way at every wait.)
    auto all_steps = [&](auto &one) __attribute__((always_inline)) {
      int st = 0;
      for (; st + 2 <= n_steps; st += 2) {
        one(st, std::integral_constant<int, 0>{});
        one(st + 1, std::integral_constant<int, 1>{});
      }
      if (st < n_steps) one(st, std::integral_constant<int, 0>{});
    };
    if (n_act > 0) all_steps(step);
    else all_steps(idle_step);
    if (strm == 0) __syncthreads();
  } else {
    auto run = [&](int st, int buf) __attribute__((always_inline)) {
      if (st >= my_steps) return;
      // Instances for several row tiles raise the wavefront's priority for their MFMA phases: the other
      // wavefront of the SIMD is then in its softmax, and the matrix pipe stays fed (-3 % on the 60-node tree).
      constexpr bool kPrio = kQT > 1;
      if (kPrio) __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int j = 0; j < kSlabs; ++j) { read_k(buf, j); scores(j); }
      if (kPrio) __builtin_amdgcn_s_setprio(0);
      if (kPrio) __builtin_amdgcn_sched_barrier(0);        // keep the V^T reads below the softmax
      softmax(st);
      if (kPrio) __builtin_amdgcn_sched_barrier(0);
      if (kPrio) __builtin_amdgcn_s_setprio(1);
      output(buf);
      if (kPrio) __builtin_amdgcn_s_setprio(0);
    };
    // ---- main loop, unrolled by the prefetch depth so that the staging registers are static.
    // Look-ahead loads past the end of the split are clamped duplicates of its last rows.
    int base = 0;
    for (; base + kPrefetch <= n_steps; base += kPrefetch) {
#pragma unroll
      for (int p = 0; p < kPrefetch; ++p) {
        const int st = base + p;
        const int buf = st & 1;
        stash(buf, 0, st, kst[p]);
        stash(buf, 1, st, vst[p]);
        issue(Kg, st + kPrefetch, kst[p]);
        issue(Vg, st + kPrefetch, vst[p]);
        __syncthreads();
        run(st, buf);
      }
    }
    // remainder (n_steps % kPrefetch trips): everything it needs is already in flight
#pragma unroll
    for (int p = 0; p < kPrefetch - 1; ++p) {
      const int st = base + p;
      if (st < n_steps) {                    // uniform over the workgroup
        const int buf = st & 1;
        stash(buf, 0, st, kst[p]);
        stash(buf, 1, st, vst[p]);
        __syncthreads();
        run(st, buf);
      }
    }
  }

  // ---- merge the states of a row and write the split's partials in register layout: [slot][kv head][row block]
  // [wavefront][pair of d-tiles][lane] x 8 halves, so that every store instruction writes 1 KB of contiguous memory.
  // The d-tiles are shared out over the wavefronts that hold a row (o_acc[.][i] is d-tile i of the wavefront's own
  // order, the first ones its own): each sends the others theirs through LDS and normalises and stores its own.
  if constexpr (kPairs) {
    // four wavefronts hold a row (two streams, two tiles of a step) and a d-tile each: o_acc[0][i] is tile part ^ i
    static_assert(kMT == 4, "a d-tile per wavefront");
    f32x4 *po4 = reinterpret_cast<f32x4 *>(lds) + lane;                        // [part][i - 1][wr][lane]
    float *pm4 = reinterpret_cast<float *>(lds + kMergeTiles<kD, kPairs>) + 2 * lane;        // [part][wr][lane][m, l]
    const float l_mine = quad_sum(l_acc[0][0]);
    __syncthreads();
#pragma unroll
    for (int i = 1; i < 4; ++i) po4[(((part ^ i) * 3 + i - 1) * 2 + wr) * 64] = o_acc[0][i];
    pm4[(part * 2 + wr) * 128] = m_run[0];
    pm4[(part * 2 + wr) * 128 + 1] = l_mine;
    __syncthreads();
    if (n_act == 0) return;
    float m_x[3], m_new = m_run[0];
#pragma unroll
    for (int i = 1; i < 4; ++i) {
      m_x[i - 1] = pm4[((part ^ i) * 2 + wr) * 128];
      m_new = fmaxf(m_new, m_x[i - 1]);
    }
    const float a0 = fast_exp2(m_run[0] - m_new);
    float ax[3], l_tot = l_mine * a0;
#pragma unroll
    for (int i = 1; i < 4; ++i) {
      ax[i - 1] = fast_exp2(m_x[i - 1] - m_new);
      l_tot += pm4[((part ^ i) * 2 + wr) * 128 + 1] * ax[i - 1];
    }
    // each state by its share of the sum, before they meet: values near the end of the range would leave it added up
    const float inv_l = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    f32x4 r = o_acc[0][0] * (a0 * inv_l);
#pragma unroll
    for (int i = 1; i < 4; ++i) r += po4[((part * 3 + i - 1) * 2 + wr) * 64] * (ax[i - 1] * inv_l);
    if (direct) {
      if (!row_ok[0]) return;
      const int64_t orow = q_row0 + i_row[0] * a.Hq + h[0];
      *reinterpret_cast<u32x2 *>((bf16_t *)a.out + orow * kD + 16 * part + 4 * c4) =
          (u32x2){pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3])};
      if (a.lse != nullptr && part == 0 && c4 == 0) a.lse[orow] = lse_of<kWide>(m_new, l_tot);
      return;
    }
    const int64_t unit = ((int64_t)slot * a.Hkv + c) * ((R + kRowsPerWG - 1) / kRowsPerWG) + rb;
    f32x4 *po = reinterpret_cast<f32x4 *>(a.part_o) + (unit * 4 + wr) * (kMT * 64) + lane;
    __builtin_nontemporal_store(r, &po[part * 64]);
    if (part == 0 && c4 == 0) {
      float *pml = a.part_ml + (unit * kRowsPerWG + 16 * wr + n) * kMlFloats;
      __builtin_nontemporal_store(m_new, &pml[0]);
      __builtin_nontemporal_store(l_tot, &pml[1]);
    }
    return;
  }
  constexpr int kOwn = kShare ? kMT / 2 : kMT;                                 // d-tiles of a stream: strm * kOwn ..
  f32x4 *mo = reinterpret_cast<f32x4 *>(lds) + w * kOwn * 64 + lane;           // [stream][w][own tile][lane]
  float *mm = reinterpret_cast<float *>(lds + kMergeTiles<kD, kPairs>) + (w * 64 + lane) * 2;     // [stream][w][lane][m,l]
#pragma unroll
  for (int qt = 0; qt < kQT; ++qt) {
    const float l_mine = kMfmaRowSum ? l_acc[qt][0] : quad_sum(l_acc[qt][0]);
    __syncthreads();                    // all tile reads (and the previous merge) done: LDS is free
    if (kShare || strm == 1) {
#pragma unroll
      for (int i = 0; i < kOwn; ++i) mo[((strm ^ 1) * 4 * kOwn + i) * 64] = o_acc[qt][kMT - kOwn + i];
    }
    mm[strm * 512] = m_run[qt];
    mm[strm * 512 + 1] = l_mine;
    __syncthreads();
    if (qt < n_act && (kShare || strm == 0)) {
      const float m1 = mm[(strm ^ 1) * 512], l1 = mm[(strm ^ 1) * 512 + 1];
      const float m_new = fmaxf(m_run[qt], m1);
      const float a0 = fast_exp2(m_run[qt] - m_new), a1 = fast_exp2(m1 - m_new);
      // unit = (split, KV head, block of 64 rows).  The split's output is stored normalised
      // (o / l: a convex combination of V rows, of the magnitude of V) in fp16, two d-tiles per
      // 16-byte store; m and l in fp32, and a power-of-two scale c per half of the row, two bf16.  c is 1 unless
      // the half's largest |o / l| would leave the fp16 range (|V| beyond 16384), then o / (l c) is stored.
      const int64_t unit = ((int64_t)slot * a.Hkv + c) * ((R + kRowsPerWG - 1) / kRowsPerWG) + rb * kQT + qt;
      const float l_tot = l_mine * a0 + l1 * a1;
      const float inv_l = l_tot > 0.f ? 1.0f / l_tot : 0.f;
      const float s0 = a0 * inv_l, s1 = a1 * inv_l;
      f32x4 r[kOwn];
#pragma unroll
      for (int i = 0; i < kOwn; ++i) r[i] = o_acc[qt][i] * s0 + mo[(strm * 4 * kOwn + i) * 64] * s1;
      if (direct) {
        // the split is the whole sequence: the merged streams are the result (the rows and columns
        // of a lane as in the combine pass)
        if (row_ok[qt]) {
          const int64_t orow = q_row0 + i_row[qt] * a.Hq + h[qt];
          bf16_t *out = (bf16_t *)a.out + orow * kD + 16 * kOwn * strm + 4 * c4;
#pragma unroll
          for (int i = 0; i < kOwn; ++i)
            *reinterpret_cast<u32x2 *>(out + 16 * i) = (u32x2){pack_bf16x2(r[i][0], r[i][1]), pack_bf16x2(r[i][2], r[i][3])};
          if (a.lse != nullptr && strm == 0 && c4 == 0) a.lse[orow] = lse_of<kWide>(m_new, l_tot);
        }
        continue;
      }
      float *pml = a.part_ml + (unit * kRowsPerWG + 16 * w + n) * kMlFloats;
      if (strm == 0 && c4 == 0) {
        __builtin_nontemporal_store(m_new, &pml[0]);
        __builtin_nontemporal_store(l_tot, &pml[1]);
      }
      if (kWide) {
        // fp32 partials: [unit][wavefront][d-tile][lane] x 4 floats
        f32x4 *po = reinterpret_cast<f32x4 *>(a.part_o) + (unit * 4 + w) * (kMT * 64) + strm * kOwn * 64 + lane;
#pragma unroll
        for (int i = 0; i < kOwn; ++i) __builtin_nontemporal_store(r[i], &po[i * 64]);
        continue;
      }
      float amax = 0.f;
#pragma unroll
      for (int i = 0; i < kOwn; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) amax = fmaxf(amax, fabsf(r[i][e]));
      amax = quad_max(amax);                       // over half of the row's kD values
      unsigned int cbits = 0x3f80u;                // 1 as bf16
      if (__builtin_amdgcn_ballot_w64(amax > 16384.f) != 0ull) {
        const int e = amax > 16384.f ? (int)((__float_as_uint(amax) >> 23) & 0xff) - 127 - 13 : 0;   // of amax / 16384, up
        cbits = (unsigned int)(127 + e) << 7;
        const float inv_c = __uint_as_float((unsigned int)(127 - e) << 23);
#pragma unroll
        for (int i = 0; i < kOwn; ++i) r[i] *= inv_c;
      }
      u32x4 *po = reinterpret_cast<u32x4 *>(a.part_o) + (unit * 4 + w) * (kMT / 2 * 64) + strm * (kOwn / 2) * 64 + lane;
#pragma unroll
      for (int pr = 0; pr < kOwn / 2; ++pr) {
        const f32x4 x = r[2 * pr], y = r[2 * pr + 1];
        __builtin_nontemporal_store((u32x4){pack_f16x2(x[0], x[1]), pack_f16x2(x[2], x[3]),
                                            pack_f16x2(y[0], y[1]), pack_f16x2(y[2], y[3])}, &po[pr * 64]);
      }
      if (kShare && c4 == 0) __builtin_nontemporal_store((bf16_t)cbits, reinterpret_cast<bf16_t *>(&pml[2]) + strm);
      if (!kShare && c4 == 0) __builtin_nontemporal_store(__uint_as_float(cbits << 16 | cbits), &pml[2]);
    }
  }
}

// Combine for the tiled partial layout above.  What bounds these kernels is not bytes (4 MB a call) but how many load
// instructions a compute unit has to issue (16 cycles each, whatever their width) and the instructions around them, one
// wavefront per SIMD; then a round trip to memory and the end of a launch.  So the addresses are scalar offsets of buffer
// loads, a split's (m, l, c) is fetched and turned into a weight by one of the four lanes that need it and handed to the
// others across lanes, and the arguments that the first load needs arrive in registers (leading scalars of the kernel).
//
// Up to 16 splits: one workgroup per (sequence, KV head, 16-row tile, kTiles d-tiles of 16); wavefront ws merges splits ws,
// ws + kWaves, ..., four of them at a time, and the wavefronts' states meet in LDS.
// kWaves = 1 and 2 (at most four and eight splits: batches, thousands of output tiles): two d-tiles each, as the number of
// wavefronts sets the pace.  12 trees of 30 nodes over 4,099 tokens, 32/8 heads: 54.0 us a call with four wavefronts of one
// d-tile, 49.2 with one of two (both with the partial pass); 12 of 2 over 700, 16/8 14.9 / 12.9.
// kWaves = 4 (9 to 16 splits): two d-tiles, one with fp32 partials, whose loads are twice as wide; us a call, loads of every
// lane's own (m, l, c) with 64-bit addresses / here: 60 nodes over 12,000 25.1 / 24.2.
typedef __attribute__((ext_vector_type(3))) unsigned int u32x3;

// KV head and row block of a unit (for rows' numbers in it: a combine workgroup without rows leaves before it loads).
__device__ __forceinline__ QuotRest head_and_block(int unit, int rbs) { return rbs == 1 ? QuotRest{unit, 0} : div_uniform(unit, rbs); }

struct CombineArgs {                               // what a combine kernel's scalar arguments say, in its own terms
  const unsigned char *part_o, *part_ml;
  void *res;
  float *lse;
  int ns_one, units, Hq, g, n_q, shape;
};

template <class T, int kD, int kWaves>
__device__ __forceinline__ void combine_rows16(const CombineArgs &a, const SeqTable &tab) {
  const unsigned char *part_o = a.part_o, *part_ml = a.part_ml;
  const int ns_one = a.ns_one, units = a.units, Hq = a.Hq, g = a.g, n_q = a.n_q, shape = a.shape;
  constexpr int kInFlight = 4;
  constexpr int kTiles = kWaves > 2 && (kWideState<kD> || std::is_same<T, float>::value) ? 1 : 2;
  constexpr bool kWide = kWideState<kD> || std::is_same<T, float>::value;    // fp32 partials
  static_assert(kInFlight == 4, "the four lanes of a row load (m, l, c) of a round's splits, one each");
  constexpr int kQuarter = kWide ? 64 * kD : 4096; // bytes of 16 rows of a unit: a wavefront of the partial pass
  constexpr int kLoad = !kWide && kTiles == 1 ? 8 : 16;
  __shared__ f32x4 xo[kWaves][kTiles][64];
  __shared__ float xm[kWaves][16], xl[kWaves][16];
  const int wq = blockIdx.x & 3, unit = blockIdx.x >> 2;       // 16 rows of unit KV head * rbs + row block
  const QuotRest cr = head_and_block(unit, shape >> 1);
  const int c = cr.quot, rho0 = cr.rest * kRowsPerWG + 16 * wq;
  if (rho0 >= n_q * g) return;                     // tile without rows (uniform)
  const int b = blockIdx.z;
  int s0 = b * ns_one, ns = ns_one;
  if (shape & 1) {                                 // sequences that differ
    s0 = tab.cu_split[b]; ns = tab.cu_split[b + 1] - s0;
  }
  const int mt = blockIdx.y * kTiles;              // first d-tile: half (mt & 1) of the stored pair mt >> 1
  const int ws = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int n = lane & 15, c4 = lane >> 4;
  // This wavefront's splits are ws, ws + kWaves, ... of the sequence's, at 32-bit offsets from its first one
  // (verify_mfma_max_splits).
  const int64_t first = ((int64_t)s0 * units + unit) * 4 + wq;
  const __amdgpu_buffer_rsrc_t rs_o = __builtin_amdgcn_make_buffer_rsrc((void *)(part_o + first * kQuarter), (short)0, (int)0x7fffffff, 0x00027000);
  const __amdgpu_buffer_rsrc_t rs_ml = __builtin_amdgcn_make_buffer_rsrc((void *)(part_ml + first * (16 * 4 * kMlFloats)), (short)0, (int)0x7fffffff, 0x00027000);
  const unsigned int step_o = (unsigned int)units * (4 * kQuarter), step_ml = (unsigned int)units * (64 * 4 * kMlFloats);
  const unsigned int at_o = (unsigned int)lane * 16u + (kLoad == 8 ? 8u * (mt & 1) : 0u);
  const unsigned int tile_o = (unsigned int)(kWide ? mt : mt >> 1) * 1024u;
  f32x4 o[kTiles];
  float m_run = kNegBig, l_run = 0.f;
#pragma unroll
  for (int t = 0; t < kTiles; ++t) o[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (int sb = ws; sb < ns; sb += kWaves * kInFlight) {
    typedef typename std::conditional<kLoad == 8, u32x2, u32x4>::type part_t;
    part_t pa[kInFlight][kWide ? kTiles : 1];
    const int s_own = sb + kWaves * c4;
    const u32x3 ml = __builtin_amdgcn_raw_buffer_load_b96(rs_ml, __umul24(min(s_own, ns - 1), step_ml) + (unsigned int)n * (4 * kMlFloats), 0, 2);
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      const unsigned int so = (unsigned int)min(sb + kWaves * u, ns - 1) * step_o + tile_o;
      if constexpr (kLoad == 8) {
        pa[u][0] = __builtin_amdgcn_raw_buffer_load_b64(rs_o, at_o, so, 2);
      } else {
#pragma unroll
        for (int t = 0; t < (kWide ? kTiles : 1); ++t) pa[u][t] = __builtin_amdgcn_raw_buffer_load_b128(rs_o, at_o, so + 1024u * t, 2);
      }
    }
    const float mx = quad_max(s_own < ns ? fmaxf(m_run, __uint_as_float(ml.x)) : m_run);
    // weight of a split: its share of the softmax denominator (its output is normalised), worked out by one of the four
    // lanes of a row and handed to the others
    const float w_own = s_own < ns ? fast_exp2(__uint_as_float(ml.x) - mx) * __uint_as_float(ml.y) : 0.f;
    const float sc = kWide ? 1.f : __uint_as_float(mt < kD / 32 ? ml.z << 16 : ml.z & 0xffff0000u);
    const unsigned int wc = __float_as_uint(w_own * sc);
    const auto w02 = __builtin_amdgcn_permlane16_swap(wc, wc, false, false);
    const auto w0 = __builtin_amdgcn_permlane32_swap(w02[0], w02[0], false, false);
    const auto w1 = __builtin_amdgcn_permlane32_swap(w02[1], w02[1], false, false);
    const float wgt[kInFlight] = {__uint_as_float(w0[0]), __uint_as_float(w1[0]), __uint_as_float(w0[1]), __uint_as_float(w1[1])};
    const float alpha = fast_exp2(m_run - mx);
    m_run = mx;
    l_run = l_run * alpha + quad_sum(w_own);
#pragma unroll
    for (int t = 0; t < kTiles; ++t) o[t] *= alpha;
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      const bool in = sb + kWaves * u < ns;        // (uniform; past the end no 0 * inf)
#pragma unroll
      for (int t = 0; t < (kWide ? kTiles : 1); ++t) if (!in) pa[u][t] = part_t{};
#pragma unroll
      for (int t = 0; t < kTiles; ++t) {
        f32x4 x;
        if constexpr (kWide) x = __builtin_bit_cast(f32x4, pa[u][t]);
        else if constexpr (kTiles == 1) x = unpack_f16x4(pa[u][0].x, pa[u][0].y);
        else x = t == 0 ? unpack_f16x4(pa[u][0].x, pa[u][0].y) : unpack_f16x4(pa[u][0].z, pa[u][0].w);
        o[t] += x * wgt[u];
      }
    }
  }
  // where this lane's row goes
  const int rho = rho0 + n;
  const QuotRest rh = row_and_head(rho, g, __builtin_amdgcn_rcpf((float)g));
  const bool row_ok = rho < n_q * g;
  const int64_t orow = (int64_t)b * n_q * Hq + c * g + (int64_t)(rh.quot * Hq + rh.rest);
  int t0 = 0;                                      // the d-tiles that this wavefront stores: all, or one
  float m = m_run, l = l_run;
  if constexpr (kWaves > 1) {
#pragma unroll
    for (int t = 0; t < kTiles; ++t) xo[ws][t][lane] = o[t];
    if (c4 == 0) { xm[ws][n] = m_run; xl[ws][n] = l_run; }
    __syncthreads();
    if (ws >= kTiles) return;
    t0 = ws;
    m = xm[0][n];
#pragma unroll
    for (int k = 1; k < kWaves; ++k) m = fmaxf(m, xm[k][n]);
    l = 0.f;
    o[0] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
      const float x = fast_exp2(xm[k][n] - m);
      l = fmaf(xl[k][n], x, l);
      o[0] += xo[k][t0][lane] * x;
    }
  }
  if (!row_ok) return;
  const float inv = 1.0f / l;
#pragma unroll
  for (int t = 0; t < (kWaves > 1 ? 1 : kTiles); ++t) {
    const f32x4 r = o[t] * inv;
    T *out = (T *)a.res + orow * kD + 16 * (mt + t0 + t) + 4 * c4;
    if constexpr (std::is_same<T, float>::value) *reinterpret_cast<f32x4 *>(out) = r;
    else *reinterpret_cast<u32x2 *>(out) = (u32x2){pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3])};
  }
  if (a.lse != nullptr && mt + t0 == 0 && c4 == 0) a.lse[orow] = lse_of<kWide>(m, l);
}

// (two names, so that the few-splits instances can be told apart in traces)
template <class T, int kD, int kWaves>
__global__ void __launch_bounds__(64 * kWaves)
verify_combine_tiled_kernel(const unsigned char *part_o, const unsigned char *part_ml, void *res, float *lse, int ns_one, int units,
                            int Hq, int g, int n_q, int shape, SeqTable tab) {
  combine_rows16<T, kD, kWaves>({part_o, part_ml, res, lse, ns_one, units, Hq, g, n_q, shape}, tab);
}
template <class T, int kD, int kWaves>
__global__ void __launch_bounds__(64 * kWaves)
verify_combine_few_kernel(const unsigned char *part_o, const unsigned char *part_ml, void *res, float *lse, int ns_one, int units,
                          int Hq, int g, int n_q, int shape, SeqTable tab) {
  combine_rows16<T, kD, kWaves>({part_o, part_ml, res, lse, ns_one, units, Hq, g, n_q, shape}, tab);
}

// More splits than that, and 9 to 16 of calls with few row blocks: one workgroup per (sequence, KV head, 4 rows, 32
// columns), so that one sequence's few output rows fill the chip: 224 workgroups that have rows for a chain of 8 with 28/4
// heads (of 256; the others leave), not 128.  Four lanes of a column take four splits side by side, so that a wavefront merges 16 splits with four loads of
// 16 bytes a lane (eight with fp32 partials) and one of (m, l, c).  Combine pass alone, us, 16 wavefronts over 16 rows and one
// d-tile / here: chain of 8 over 26,112 tokens 4.1 / 2.75, of 5 over 8,192 3.8 / 2.5, of 4 over 12,000 4.0 / 2.7; with the
// partial pass, one KV head, chain of 8 over 16,000 (256 splits) 16.8 / 12.6.
// Four rows are 64 bytes of a 128-byte line of the partials: the two workgroups of a line lie eight apart, on one XCD, so
// that it comes to one L2 and not to two.  Neighbours / eight apart, us a call: chain of 8 over 26,112 16.2 / 15.8, of 5 over
// 8,192 10.2 / 9.95, over 3,300 9.05 / 8.6, one KV head over 16,000 12.5 / 11.5, 16 nodes over 5,000 13.2 / 12.2.
// Against wavefronts over 16-row tiles: 17 to 32 splits (eight of them) 30 nodes over 26,112 27.3 / 26.9, two of 30 over up to
// 4,000 16.15 / 15.6, four of 20 over up to 6,000 23.9 / 23.6; 9 to 16 splits (four), 4 to 8 units (KV heads x row blocks of
// 64) a chain of 5 over 600 7.5 / 7.3, of 8 over 900 8.0 / 7.65, four ragged of 8 over 2,000 10.9 / 10.8, but 28 units, 60
// nodes over 5,000 17.5 / 17.7 and over 26,112 39.6 / 40.0.
template <class T, int kD, int kWaves>
__global__ void __launch_bounds__(64 * kWaves)
verify_combine_long_kernel(const unsigned char *part_o, const unsigned char *part_ml, void *res, float *lse, int ns_one, int units,
                       int Hq, int g, int n_q, int shape, SeqTable tab) {
  constexpr bool kWide = kWideState<kD> || std::is_same<T, float>::value;    // fp32 partials
  constexpr int kQuarter = kWide ? 64 * kD : 4096; // bytes of 16 rows of a unit: a wavefront of the partial pass
  constexpr unsigned int kPastEnd = 0x80000000u;   // a buffer offset that reads as zero
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  __shared__ f32x2 xo[kWaves][64], xml[kWaves][4];
  // four rows of unit KV head * rbs + row block
  const int rows4 = (blockIdx.x & 7) * 2 + (blockIdx.x >> 3 & 1), unit = blockIdx.x >> 4;
  const QuotRest cr = head_and_block(unit, shape >> 1);
  const int c = cr.quot, rho0 = cr.rest * kRowsPerWG + 4 * rows4;
  if (rho0 >= n_q * g) return;                     // group without rows (uniform)
  const int b = blockIdx.z;
  int s0 = b * ns_one, ns = ns_one;
  if (shape & 1) {                                 // sequences that differ
    s0 = tab.cu_split[b]; ns = tab.cu_split[b + 1] - s0;
  }
  const int ws = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & 3, c4 = (lane >> 2) & 3, ss = lane >> 4;
  const int64_t first = (int64_t)s0 * units + unit;
  const __amdgpu_buffer_rsrc_t rs_o = __builtin_amdgcn_make_buffer_rsrc((void *)(part_o + first * (4 * kQuarter)), (short)0, (int)0x7fffffff, 0x00027000);
  const __amdgpu_buffer_rsrc_t rs_ml = __builtin_amdgcn_make_buffer_rsrc((void *)(part_ml + first * (64 * 4 * kMlFloats)), (short)0, (int)0x7fffffff, 0x00027000);
  const unsigned int step_o = (unsigned int)units * (4 * kQuarter), step_ml = (unsigned int)units * (64 * 4 * kMlFloats);
  const unsigned int tile = (unsigned int)(rows4 >> 2) * kQuarter + (unsigned int)blockIdx.y * (kWide ? 2048u : 1024u);
  const unsigned int at_o = tile + (unsigned int)(c4 * 16 + 4 * (rows4 & 3) + r) * 16u;
  const unsigned int at_ml = (unsigned int)(4 * rows4 + r) * (4 * kMlFloats);
  float o[8], m_run = kNegBig, l_run = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = 0.f;
  for (int base = 16 * ws; base < ns; base += 16 * kWaves) {
    const int s_own = base + 4 * c4 + ss;
    const u32x3 ml = __builtin_amdgcn_raw_buffer_load_b96(rs_ml, s_own < ns ? (unsigned int)s_own * step_ml + at_ml : kPastEnd, 0, 0);
    u32x4 pa[4][kWide ? 2 : 1];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int s = base + 4 * ((c4 + j) & 3) + ss;
      const unsigned int at = s < ns ? (unsigned int)s * step_o + at_o : kPastEnd;
#pragma unroll
      for (int t = 0; t < (kWide ? 2 : 1); ++t) pa[j][t] = __builtin_amdgcn_raw_buffer_load_b128(rs_o, at, 1024 * t, 2);
    }
    const float m_own = s_own < ns ? __uint_as_float(ml.x) : kNegBig;
    float mx = fmaxf(m_run, m_own);
    mx = fmaxf(mx, dpp_f32<0x128>(mx));
    mx = fmaxf(mx, dpp_f32<0x124>(mx));
    mx = quad_max(mx);
    const float w = fast_exp2(m_own - mx) * __uint_as_float(ml.y);
    const float wc = kWide ? w : w * __uint_as_float(blockIdx.y < kD / 64 ? ml.z << 16 : ml.z & 0xffff0000u);
    const float alpha = fast_exp2(m_run - mx);
    m_run = mx;
    l_run = l_run * alpha + w;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] *= alpha;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float x = j == 0 ? wc : j == 1 ? dpp_f32<0x12C>(wc) : j == 2 ? dpp_f32<0x128>(wc) : dpp_f32<0x124>(wc);
      f32x4 lo, hi;
      if constexpr (kWide) { lo = __builtin_bit_cast(f32x4, pa[j][0]); hi = __builtin_bit_cast(f32x4, pa[j][1]); }
      else { lo = unpack_f16x4(pa[j][0].x, pa[j][0].y); hi = unpack_f16x4(pa[j][0].z, pa[j][0].w); }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[e] = fmaf(lo[e], x, o[e]);
        o[4 + e] = fmaf(hi[e], x, o[4 + e]);
      }
    }
  }
  // sums over the splits of the wavefront's four lanes of a column; two of the eight columns are left to a lane
  float y[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[e]), __float_as_uint(o[4 + e]), false, false);
    y[e] = __uint_as_float(q[0]) + __uint_as_float(q[1]);
  }
  f32x2 z;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(y[e]), __float_as_uint(y[2 + e]), false, false);
    z[e] = __uint_as_float(q[0]) + __uint_as_float(q[1]);
  }
  l_run += dpp_f32<0x128>(l_run);
  l_run += dpp_f32<0x124>(l_run);
  l_run = quad_sum(l_run);
  const int rho = rho0 + r;
  const QuotRest rh = row_and_head(rho, g, __builtin_amdgcn_rcpf((float)g));
  const int64_t orow = (int64_t)b * n_q * Hq + c * g + (int64_t)(rh.quot * Hq + rh.rest);
  float m = m_run, l = l_run;
  if constexpr (kWaves > 1) {
    xo[ws][lane] = z;
    if (lane < 4) xml[ws][r] = (f32x2){m_run, l_run};
    __syncthreads();
    if (ws != 0) return;
    f32x2 q[kWaves];
#pragma unroll
    for (int k = 0; k < kWaves; ++k) { q[k] = xml[k][r]; m = fmaxf(m, q[k][0]); }
    l = 0.f;
    z = (f32x2){0.f, 0.f};
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
      const float x = fast_exp2(q[k][0] - m);
      l = fmaf(q[k][1], x, l);
      z += xo[k][lane] * x;
    }
  }
  if (rho >= n_q * g) return;
  const float inv = 1.0f / l;
  z *= inv;
  T *out = (T *)res + orow * kD + 32 * blockIdx.y + 16 * (ss >> 1) + 4 * c4 + 2 * (ss & 1);
  if constexpr (std::is_same<T, float>::value) *reinterpret_cast<f32x2 *>(out) = z;
  else *reinterpret_cast<unsigned int *>(out) = pack_bf16x2(z[0], z[1]);
  if (lse != nullptr && blockIdx.y == 0 && (lane & ~3) == 0) lse[orow] = lse_of<kWide>(m, l);
}

}  // namespace

// Both head sizes of the boundary.  Measured at d = 64 (16/4 heads, 4 ragged sequences of 6,001 on
// average, chain of 8, 23.5 MB a call): 107 us with the plain-ALU kernels (fp32 multiply-adds and LDS
// reads bound them), 14.5 us here, launched call by call, with the same error against 64 bits (1.7e-3:
// the output's own rounding).
bool verify_partial_mfma_supported(int dtype, int head_dim) {
  return (dtype == SPARROW_BF16 || dtype == SPARROW_F32) && (head_dim == 128 || head_dim == 64);
}

// Floats of workspace per (split, KV head, row block) unit of the tiled partial layout: 64 rows of 128
// halves, or of floats.
int64_t verify_mfma_unit_floats_o(int dtype, int head_dim) { return dtype == SPARROW_F32 ? 64 * head_dim : 4096; }
int64_t verify_mfma_unit_floats_ml() { return kRowsPerWG * kMlFloats; }

// The combine pass addresses the splits of a sequence by 31-bit offsets from the first one, and multiplies 24 bits for those
// of (m, l, c).  A few hundred units as a rule, but the plan gives one KV head eight splits (fp32: 16) however many rows it
// has: from 4,369 units (fp32, heads of 128; 64: 8,739) or 18,725 (bf16) on it gets fewer, where thousands of row blocks fill
// the chip by themselves.
int verify_mfma_max_splits(int dtype, int head_dim, int64_t units) {
  if (units * verify_mfma_unit_floats_ml() * 4 >= 1 << 24) return 1;
  const int64_t unit_o = verify_mfma_unit_floats_o(dtype, head_dim) * 4;
  return (int)std::min<int64_t>(1 + (0x7fffffff - unit_o) / (units * unit_o), INT32_MAX);
}

// Row blocks (workgroups per split and KV head) for R rows: blocks of three 64-row tiles unless
// blocks of two leave fewer empty tiles (7 tiles: 2+2+2+1 beats 3+3+1, measured).
int verify_mfma_row_blocks(int dtype, int R) {
  if (dtype == SPARROW_F32) return verify_f32_row_blocks(R);
  const int tiles = (R + kRowsPerWG - 1) / kRowsPerWG;
  const int rbs3 = (tiles + 2) / 3, rbs2 = (tiles + 1) / 2;
  return rbs3 * 3 - tiles <= rbs2 * 2 - tiles ? rbs3 : rbs2;
}

// The two streams half a step apart: where several row blocks share a stream, from 14 steps on.  Time in step / half a
// step apart, medians on two cards and the whole range, over drawn calls (8 to 64 nodes, 1 to 12 sequences, all
// layouts of K and V):
//   several blocks, 11 to 13 steps 0.99 and 0.98 (0.89 to 1.04), 14 to 18 steps 1.02 and 1.01 (0.92 to 1.08), more
//   1.04 and 1.03 (0.92 to 1.10): the longer start and end of a split have to be earned back;
//   one block of 128 rows 0.97 and 0.97 (0.85 to 1.11): half of the matrix work per byte of K and V, which then set
//   the pace.
static bool half_step_pays(int steps, int rbs) { return rbs > 1 && steps >= 14; }

// All sequences of a call of one length, cut alike: the kernels then work out a sequence's place from its number.  (Table
// entries are 0.3 to 0.4 us ahead of a workgroup's first load: they are in lines of the arguments that nothing else reads.)
static bool equal_sequences(const VerifyArgs &a, const SeqTable &tab) {
  for (int b = 1; b < a.B; ++b)
    if (tab.cu_len[b + 1] - tab.cu_len[b] != tab.cu_len[1] - tab.cu_len[0] || tab.cu_split[b + 1] - tab.cu_split[b] != tab.cu_split[1])
      return false;
  return true;
}

template <int kD>
static hipError_t launch_partial(const VerifyArgs &a, const SeqTable &tab, hipStream_t st) {
  const int R = a.n_q * (a.Hq / a.Hkv);
  const int rbs = verify_mfma_row_blocks(SPARROW_BF16, R);
  PieceTable pt;
  int max_ns = 0;
  for (int b = 0; b < SPARROW_MAX_BATCH; ++b) {
    const int ns = b < a.B ? tab.cu_split[b + 1] - tab.cu_split[b] : 0;
    pt.piece[b] = ns > 0 ? split_len(tab.cu_len[b + 1] - tab.cu_len[b], ns) : 0;
    if (ns > max_ns) max_ns = ns;
  }
  // grid shape: one x range per (KV head, sequence) unless that would launch mostly padding
  const int x3d = (max_ns + 7) / 8 * 8;
  const int flat = (int64_t)a.n_slots * 4 < (int64_t)x3d * a.B * 3;      // fewer than 3/4 of the slots real
  dim3 grid(x3d * rbs, a.Hkv, a.B), block(256 * kStreams);
  if (flat) grid = dim3((a.n_slots * a.Hkv + 7) / 8 * 8 * rbs, 1, 1);
  constexpr int kSub = 128 / kD;
  static_assert(kLdsBytes<kD> <= 64 * 1024, "beyond 64 KB the kernel needs the dynamic-LDS attribute");
  const int shape = rbs << kShapeBits | (flat ? kShapeFlat : 0) | (a.direct ? kShapeDirect : 0) | (equal_sequences(a, tab) ? 0 : kShapeTable);
  const int len0 = flat ? a.n_slots * a.Hkv : tab.cu_len[1] - tab.cu_len[0], ns0 = tab.cu_split[1];
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, block, kLdsBytes<kD>, st, a.k, a.v, a.stride_head, (int)a.stride_tok, (int)tab.cu_len[0], len0, ns0,
                       (int)pt.piece[0], a.n_slots, shape, a, tab, pt);
  };
  const int steps = (a.chunk / kTile + kStreams * kSub - 1) / (kStreams * kSub);   // of a full split
  const int tiles = (R + kRowsPerWG - 1) / kRowsPerWG;
  const int qt = (tiles + rbs - 1) / rbs;
  if (qt == 3)      // a second tile in flight does not fit the registers (and the step is compute-bound)
    go(verify_partial_mfma_kernel<kD, 1, 3, false>);
  else if (qt == 2 && steps <= 10)
    go(verify_partial_mfma_kernel<kD, 1, 2, false>);
  else if (qt == 2 && kD == 128 && half_step_pays(steps, rbs))
    go(verify_partial_mfma_kernel<128, 2, 2, true>);
  else if (qt == 2)
    go(verify_partial_mfma_kernel<kD, 2, 2, false>);
  else if (kD == 64 && R <= 32)
    go(verify_partial_mfma_kernel<64, 1, 0, false>);
  else if (steps <= 3)       // (a second step in flight pays from 4 steps on: -0.15 us at the 7 steps of a 26k chain)
    go(verify_partial_mfma_kernel<kD, 1, 1, false>);
  else
    go(verify_partial_mfma_kernel<kD, 2, 1, false>);
  return hipGetLastError();
}

hipError_t launch_verify_partial_mfma(int dtype, const VerifyArgs &a, const SeqTable &tab, hipStream_t st) {
  if (dtype == SPARROW_F32) return launch_verify_partial_f32(a, tab, st);
  return a.d == 128 ? launch_partial<128>(a, tab, st) : launch_partial<64>(a, tab, st);
}

template <class T, int kD>
static hipError_t launch_combine(const VerifyArgs &a, const SeqTable &tab, hipStream_t st) {
  const int R = a.n_q * (a.Hq / a.Hkv);
  const int rbs = (R + kRowsPerWG - 1) / kRowsPerWG;
  int max_ns = 0;
  for (int b = 0; b < a.B; ++b) max_ns = std::max(max_ns, tab.cu_split[b + 1] - tab.cu_split[b]);
  const int shape = rbs << 1 | !equal_sequences(a, tab), units = a.Hkv * rbs;
  constexpr int kTiles = kWideState<kD> || std::is_same<T, float>::value ? 1 : 2;      // of more than two wavefronts
  auto go = [&](auto kern, int waves, int groups, int tiles) {      // row groups of a unit, d-tiles of a workgroup
    hipLaunchKernelGGL(kern, dim3(units * groups, kD / 16 / tiles, a.B), dim3(64 * waves), 0, st, (const unsigned char *)a.part_o,
                       (const unsigned char *)a.part_ml, a.out, a.lse, (int)tab.cu_split[1], units, a.Hq, a.g, a.n_q, shape, tab);
  };
  if (max_ns > 128) go(verify_combine_long_kernel<T, kD, 16>, 16, 16, 2);
  else if (max_ns > 64) go(verify_combine_long_kernel<T, kD, 8>, 8, 16, 2);
  else if (max_ns > 32) go(verify_combine_long_kernel<T, kD, 4>, 4, 16, 2);
  else if (max_ns > 16) go(verify_combine_long_kernel<T, kD, 2>, 2, 16, 2);
  else if (max_ns > 8 && units <= 8) go(verify_combine_long_kernel<T, kD, 1>, 1, 16, 2);
  else if (max_ns > 8) go(verify_combine_tiled_kernel<T, kD, 4>, 4, 4, kTiles);
  else if (max_ns > 4) go(verify_combine_few_kernel<T, kD, 2>, 2, 4, 2);
  else go(verify_combine_few_kernel<T, kD, 1>, 1, 4, 2);
  return hipGetLastError();
}

hipError_t launch_verify_combine_mfma(int dtype, const VerifyArgs &a, const SeqTable &tab, hipStream_t st) {
  if (dtype == SPARROW_F32) return a.d == 128 ? launch_combine<float, 128>(a, tab, st) : launch_combine<float, 64>(a, tab, st);
  return a.d == 128 ? launch_combine<bf16_t, 128>(a, tab, st) : launch_combine<bf16_t, 64>(a, tab, st);
}

}  // namespace sparrow
