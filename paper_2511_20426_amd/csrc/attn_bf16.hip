// bf16 block-cascaded attention on the gfx950 matrix cores (head_dim 128, 128-token pages).
//
// What it computes: for every in-flight query block, softmax(Q K^T / sqrt(D)) V over the
// pages of the KV blocks that block may see -- the clean cache plus the in-flight blocks,
// all of them (bidirectional cascade, Sec. 3.4) or those not later than itself (block-causal,
// Sec. 3.2 / 4.2).  Visibility is per block pair, so masking is "walk only the visible pages":
// pages of invisible blocks are never loaded.
//
// Shape of the kernel
//   workgroup = 4 waves, one per SIMD; a wave owns 64 query rows, a workgroup 256 rows of one head.
//   K and V pages (32 KB each) stream global -> LDS without passing through registers into two
//   2-page rings shared by the four waves.
//   S^T = K Q^T   : A = K rows from LDS, B = Q (AGPRs).  A lane then holds keys of ONE query per column
//                   tile, so a row reduction is a cross-lane step or two, and only on the rare steps
//                   where the exponent reference moves.
//   O^T += V^T P^T: A = V^T rows from LDS, B = P^T straight from the S^T accumulator
//                   registers (rounded to bf16).  V pages are stored transposed and with the
//                   key order the accumulators hand over, so no data movement is needed
//                   between the two products (see cascade_attn.h for the page format).
//   Softmax is the running-reference form in base 2: p = exp2(s*c - m_ref), c = log2(e)/sqrt(D);
//   m_ref moves (and the accumulators are rescaled) only when the probabilities of a step grow past a limit.
//   The loop exists on two matrix instructions, picked per launch by takes_core16: 32x32x16 (two column tiles
//   of 32 queries; fewer cycles) and 16x16x32 (four tiles of 16; less power).  Row sums are taken in fp32 over the probabilities
//   before their rounding to bf16 in both.  Errors against fp64 over seven shapes and logit scales, flat rows and peaked ones: 2.4066e-3 ..
//   5.3026e-3 with either; rows with one key of weight 0.9 whose V is zero: 1.5e-4 off as a whole, with either.
//   The 256-byte page rows are stored with their 16-byte chunks XOR-swizzled by (row & 15),
//   which makes every ds_read_b128 of an MFMA operand bank-conflict free (K with 16x16x32: two lanes to a bank).
//   Workgroups are numbered so that the eight XCDs each take a contiguous range of
//   (head, row tile) work: workgroups running together on an XCD stream the same head's pages
//   and share them in that XCD's L2.
//   This file holds the set-up and the epilogue; the software-pipelined main loop is the
//   hand-scheduled assembly emitted by gen_attn_core.py and gen_attn_core16.py.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>

#include "ca_internal.hpp"

namespace ca {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

constexpr int kPageBytes = 128 * 128 * 2;       // one K or V page
constexpr int kPairBytes = 2 * kPageBytes;      // K page followed by V page
constexpr int kRowsPerWg = 256;

// Everything a launch needs.  A workgroup starts with nothing but this block's address: the scalars of the first part come
// in three loads issued together (load_head: left to the compiler they were fetched one after the other as they were needed,
// seven trips before the first load of Q), the per-block tables as one dword per lane of
// `lanes` (a lane's entry is picked with v_readlane later), the rotation factors as two vectors per lane.  What a workgroup
// works on is found with scalar instructions alone: divisions by launch constants are a multiplication and a correction.
struct AttnHead {
  const uint16_t* q;                   // [row, head, dim] with the strides below; unrotated for attn_bf16_kernel<true, ..>
  uint16_t* o;
  const uint8_t* pool;
  float* partials;                     // [xcd][split item][chunk][kPartialFloats]
  // Query segments: rows that share one visible prefix (one segment in a bidirectional cascade,
  // one per query block in a block-causal one, longest prefix first); all have tiles_per_seg row
  // tiles.  A "column" is a (head, row tile) pair, a work item a segment of a column.  Counted column by column the items
  // are shared out to the XCDs in eight ranges of one length, so that an XCD's first and last column may be its own in some
  // segments only; an XCD works through its range segment by segment (decode_item).  Workgroups that run together on an XCD then
  // walk KV prefixes of one length, start and finish together, and stay in step on the same pages
  // of the same few heads, which is what keeps those pages in the XCD's L2.
  // With whole columns to an XCD, 60 columns were 8 for seven of them and 4 for the last, 9 columns 2 for four and none for three.  Whole
  // block-causal steps of five blocks, us, whole columns / ranges of items: 12 heads of 4680 tokens 4392 / 3998 (143 items an XCD
  // instead of 145 leave 15 for the last round, which can then be halved), of 1170 323 / 307; 3 heads of 540 58.5 / 42.8; four
  // blocks of 2 heads of 1200 84 / 59.
  // Segment i has rows seg_first - i seg_rows .. and sees the first vis_first - i KV blocks.
  int32_t heads, pages_per_block, last_valid, n_seg;
  int32_t tiles_per_seg, items, work_per_xcd;   // work_per_xcd: of the XCDs with the most, items / 8 rounded up
  // Splitting: the last `split_items` work items of every XCD's range have their KV walk cut
  // into `split` page ranges, one workgroup each; their partial results meet in
  // merge_partials_kernel.
  // With `range` > 0 all items of a launch with walks of several lengths are cut into ranges of that many pages (the last
  // one of a walk is what is left), and a walk of one range is not cut: range_segs has, four bits each, in how many segments
  // walks have a first, second .. range.  A workgroup has a place of its own for its partial result then.
  int32_t split, split_items, full_items;   // per XCD: full_items + split_items == work_per_xcd
  float c;                             // log2(e) / sqrt(head_dim)
  uint32_t per_seg, per_tiles, per_pages, per_split, per_split_items;   // reciprocal() of n_seg and those
  int64_t q_tok_stride, q_head_stride;
  // Rotary embedding of the queries (attn_bf16_kernel<true, ..> only).  Angles are formed in revolutions:
  // pair j turns by pos * freq[j] / 2pi; that factor is split into a 12-bit head and a tail so that
  // pos * head is exact in fp32 for pos < 4096 and only its fractional part meets the hardware
  // sin / cos (measured: cos and sin within 4.2e-7 of fp64 for every pos < 4096 and every pair).
  int32_t pairs_t, pairs_h;            // pairs [0, pairs_t): frame axis, then pairs_h: row axis, rest: column axis
  int32_t plane, grid_h, grid_w, frames_per_block;   // plane = grid_h * grid_w
  uint32_t per_plane, per_grid_w;
  // cos and sin per axis value present in a tile, in LDS, by quads of four pairs as a lane of 16 has them: tab_f frames, then
  // tab_y rows, then grid_w columns, each with the quads that its axis has a pair in; tab_y == 0: a geometry without a table,
  // every lane evaluates its own
  int32_t tab_f, tab_y, tab_quads;     // tab_quads: of the table
  int32_t seg_first, seg_rows, vis_first;
  int32_t range, spare[2];
  uint64_t range_segs;
};
static_assert(sizeof(AttnHead) == 192, "three loads of 64 bytes");

struct AttnArgs : AttnHead {
  int32_t lanes[64];                   // kLane*: first frame per query block; KV slots
  float rev_hi[kMaxPairs], rev_lo[kMaxPairs];
};
constexpr int kLaneFrame = 0, kLaneSlot = 32;
static_assert(kMaxInflight == 8 && kMaxKvBlocks == 32, "AttnArgs::lanes");

constexpr int kMaxSplit = 16;          // page ranges of a walk
constexpr int kPartialsPerXcd = kMaxPartials / 8;   // of launches with `range`

typedef __attribute__((ext_vector_type(16))) uint32_t u32x16;

// the scalars of the launch (AttnArgs is the kernel's one argument)
__device__ __forceinline__ AttnHead load_head() {
  struct Raw { u32x16 x[3]; } raw;
  const uint64_t at = reinterpret_cast<uint64_t>(__builtin_amdgcn_kernarg_segment_ptr());
  asm volatile("s_load_dwordx16 %0, %3, 0x0\n\ts_load_dwordx16 %1, %3, 0x40\n\ts_load_dwordx16 %2, %3, 0x80\n\ts_waitcnt lgkmcnt(0)"
               : "=&s"(raw.x[0]), "=&s"(raw.x[1]), "=&s"(raw.x[2]) : "s"(at));
  return __builtin_bit_cast(AttnHead, raw);
}

// one partial result of a 256-row tile, in the order the accumulators leave the registers: O^T
// contributions [wave][register group][lane] as fp32 x 4 (not normalised), then (exponent
// reference in log2 units, row sum) per row
constexpr int kPartialMl = kRowsPerWg * 128;
constexpr int kPartialFloats = kRowsPerWg * 132;
static_assert(size_t(kMaxPartials) * kPartialFloats * 4 == kAttnScratchBytes, "scratch size");

// n / d and n % d with per = reciprocal(d): floor(n per / 2^32) is the quotient or one less
__host__ constexpr uint32_t reciprocal(int32_t d) { return d > 1 ? uint32_t((uint64_t(1) << 32) / uint32_t(d)) : 0xffffffffu; }
__device__ __forceinline__ int div_by(int n, int d, uint32_t per, int* rem) {
  uint32_t q = __umulhi(uint32_t(n), per), r = uint32_t(n) - q * uint32_t(d);
  const bool more = r >= uint32_t(d);
  *rem = int(more ? r - uint32_t(d) : r);
  return int(more ? q + 1 : q);
}

// n / d with inv = 1 / d to within an ulp, for n < 2^20: half of 1 / d away from the next whole number, the product cannot round to it
__device__ __forceinline__ int div_small(int n, float inv) { return int((float(n) + 0.5f) * inv); }

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

struct WorkItem {
  int h, row0, rows_end, seg;       // h < 0: no such item (an XCD may own one less than another)
};

// An XCD's items: columns from .. to - 1, in the first `to_segs` segments column `to` too, in the first `from_segs` not column
// `from`.
struct Share {
  int from, from_segs, to, to_segs;
  __device__ __forceinline__ int first(int seg) const { return from + (seg < from_segs); }
  __device__ __forceinline__ int end(int seg) const { return to + (seg < to_segs); }
  // items of the first n segments
  __device__ __forceinline__ int count(int n) const { return n * (to - from) + min(n, to_segs) - min(n, from_segs); }
};

template <typename Args>
__device__ __forceinline__ Share share_of(const Args& a, int xcd) {
  Share s;
  s.from = div_by((xcd * a.items) >> 3, a.n_seg, a.per_seg, &s.from_segs);
  s.to = div_by(((xcd + 1) * a.items) >> 3, a.n_seg, a.per_seg, &s.to_segs);
  return s;
}

// Item `item` of an XCD, longest walks first.
template <typename Args>
__device__ __forceinline__ WorkItem decode_item(const Args& a, const Share& share, int item) {
  WorkItem w;
  int t, seg = 0, col = share.first(0) + item, end = share.end(0);
  while (col >= end && ++seg < a.n_seg) {
    col += share.first(seg) - end;
    end = share.end(seg);
  }
  w.seg = seg;
  w.h = div_by(col, a.tiles_per_seg, a.per_tiles, &t);
  const int row0 = a.seg_first - seg * a.seg_rows;
  w.row0 = row0 + t * kRowsPerWg;
  w.rows_end = row0 + a.seg_rows;
  if (seg == a.n_seg) w.h = -1;
  return w;
}

// u a + w b, the product with w rounded: written out, because the compiler joins either product to the sum, not the same in each place
__device__ __forceinline__ float turned(float u, float w, float a, float b) { return __builtin_fmaf(u, a, w * b); }

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  f32x2 f = {lo, hi};
  bf16x2 b = __builtin_convertvector(f, bf16x2);   // v_cvt_pk_bf16_f32, round to nearest even
  return __builtin_bit_cast(uint32_t, b);
}

// value of the partner lane (lane ^ 32)
__device__ __forceinline__ float other_half(float x) { return __shfl_xor(x, 32, 64); }

// what a wave wrote to LDS is there for its other lanes
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

#include "attn_core_clobbers.inc"
#include "attn_core16_clobbers.inc"

// LDS map: K ring (2 pages), V ring (2 pages), token positions of the tile's rows, cos / sin table; the main loop lives
// in attn_core_gfx950.inc (generated by gen_attn_core.py, which also documents the pipeline and the
// register map).  Before the loop the second slots of the two rings hold the tile's Q rows.
constexpr uint32_t kVRing = 2 * kPageBytes;
constexpr uint32_t kPosArea = 4 * kPageBytes;
constexpr uint32_t kTrigArea = kPosArea + kRowsPerWg * 16;
constexpr int kAttnLds = 160 * 1024;
constexpr int kTrigQuads = (kAttnLds - int(kTrigArea)) / 32;

// rows I0 .. I1 - 1 of a lane's 16 (row i is 4 i rows on, `rows` are left), from `at` on in steps of `step` bytes; rows past the end
// re-read the last one.  They stay where they stand between other work.
template <int I0, int I1>
__device__ __forceinline__ void load_q(u32x4 (&v)[16], uint64_t& at, uint64_t end, uint64_t step, int rows) {
#pragma unroll
  for (int i = I0; i < I1; ++i, at += step)
    v[i] = *reinterpret_cast<const __attribute__((address_space(1))) u32x4*>(4 * i < rows ? at : end);
  __builtin_amdgcn_sched_barrier(0);
}

// load i of the wave's 16 of a K page and its V page (at `page`) into the first slots of their rings
__device__ __forceinline__ void load_page_piece(uint32_t lds_wave, uint32_t lane_off, uint64_t page, int i) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds_wave + (i & 7) * 4096 + (i >> 3) * kVRing), "v"(lane_off + (i & 7) * 4096),
                  "s"(page + (i >> 3) * uint64_t(kPageBytes)) : "m0");
}

// What a workgroup spends outside the loop is paid once per item, and one workgroup per CU means that nothing overlaps it.  Cycles
// (timestamps of a probe build; a page of walk is 4300): 31 000 when a thread rotated a whole row, scalars were fetched one by one
// and results left in 8-byte pieces; 23 000 with Q read and the results written as whole 256-byte rows and the
// rotation shared out so that a thread needs the factors of four pairs only; 22 000 with cos and sin from a table in LDS: a
// tile of 256 rows meets few values per axis (1262 at 30 x 52 for 16 384 pairs), filled while Q is on its way; 18 000 now, the
// smallest step 26.9 -> 24.9 us.  What that took: the item found with scalar instructions and the arguments in one go (to the
// first load of Q 2100 -> 1000), the table filled by all threads in turn, Q's loads dealt out between (with positions and Q's loads
// 5600 -> 2700), the reads of the table ahead of the products and beside the page loads (7000 -> 5300), the accumulators cleared and
// K(1) requested beside the first tile's products (3600 -> 3000).  The scale c comes behind the rotation: multiplied into
// the table it would be two instructions less a pair, but rounds otherwise and keeps finite what rope3d_apply takes out of
// range.  The first K and V page are requested when Q has landed, behind loads that the compiler counts: requested
// before, they cost 0.5 us, the waits for Q then include them.  Nothing of this shows at the 14B shape, where an item walks
// 407 pages.
//
// kTails: the loop that walks half of a short last page (gen_attn_core.py), picked by has_tails.
// kCore16: which of the two main loops.  Both walk the same pages the same way; they differ in the matrix
// instruction, and so in where a lane's part of Q, of the accumulators and of a row sum is.
template <bool kRopeQ, bool kCore16, bool kTails>
__global__ __launch_bounds__(256, 1) void attn_bf16_kernel(AttnArgs args) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, hi = lane >> 5, l15 = lane & 15, grp = lane >> 4;
  const int lane_tab = args.lanes[lane];
  const int my_slot = args.lanes[kLaneSlot + (lane & 31)];
  const int c16 = lane & 15, r4 = lane >> 4;               // 16-byte chunk and row (mod 4) of Q / O this lane moves
  const float pair_hi = kRopeQ ? args.rev_hi[lane] : 0.f, pair_lo = kRopeQ ? args.rev_lo[lane] : 0.f;   // of pair `lane`
  const AttnHead a = load_head();

  // ---- which (head, row tile, page range): XCD x takes its own work_per_xcd items; inside an XCD
  // the full items come first, then the split ones, all their first page ranges, then the second ...
  const int xcd = blockIdx.x & 7, nth = blockIdx.x >> 3;
  const Share share = share_of(a, xcd);
  int item = nth, chunk = 0, n_chunks = 1;
  if (a.range > 0) {                                       // all first ranges, then the second ones of the walks that have one ..
    uint64_t segs = a.range_segs;
    for (int n; item >= (n = share.count(int(segs & 15)));) {
      item -= n;
      segs >>= 4;
      ++chunk;
      if (segs == 0) return;
    }
  } else if (nth >= a.full_items) {
    int in_chunk;
    chunk = div_by(nth - a.full_items, a.split_items, a.per_split_items, &in_chunk);
    item = a.full_items + in_chunk;
    n_chunks = a.split;
  }
  const WorkItem wi = decode_item(a, share, item);
  if (wi.h < 0) return;
  const int h = wi.h, row0 = wi.row0, rows_end = wi.rows_end, n_kvb = a.vis_first - wi.seg;
  const int all_pages = n_kvb * a.pages_per_block;
  int page_lo = 0, page_hi = all_pages, in_block, rem;
  if (a.range > 0) {
    page_lo = chunk * a.range;
    page_hi = min(page_lo + a.range, all_pages);
  } else if (n_chunks > 1) {
    page_lo = div_by(all_pages * chunk, n_chunks, a.per_split, &rem);
    page_hi = div_by(all_pages * (chunk + 1), n_chunks, a.per_split, &rem);
  }
  const int kb0 = div_by(page_lo, a.pages_per_block, a.per_pages, &in_block), pg0 = in_block;
  const int n_pages = page_hi - page_lo;

  // ---- Q rows: a wave takes its own 64, 16 lanes to a row (one multiplication per lane and one for the last row, which rows past
  // the end re-read)
  u32x4 v[16];
  const int first = row0 + wave * 64 + r4;
  const uint64_t qp = reinterpret_cast<uint64_t>(a.q) + 2 * (int64_t(h) * a.q_head_stride + c16 * 8);
  const uint64_t q_end = qp + 2 * int64_t(rows_end - 1) * a.q_tok_stride, q_step = 8 * a.q_tok_stride;
  uint64_t q_at = qp + 2 * int64_t(first) * a.q_tok_stride;
  // (a load keeps the unit that forms addresses busy for 16 cycles, those of four waves for 64: with a table to fill they are dealt out)
  load_q<0, kRopeQ ? 4 : 16>(v, q_at, q_end, q_step, rows_end - first);
  uint8_t* const parked = lds + kPageBytes + (wave >> 1) * kPageBytes + wave * 64 * 256;
  uint8_t* park[4];                                        // of this lane's piece of rows r4 + 4 i, i = 0..3; 16 rows on: 4096 bytes
#pragma unroll
  for (int i = 0; i < 4; ++i) park[i] = parked + (r4 + 4 * i) * 256 + ((c16 ^ (r4 + 4 * i)) << 4);
  int4* const pos = reinterpret_cast<int4*>(lds + kPosArea) + wave * 64;
  if (kRopeQ) {
    // ---- while Q is on its way: the rows' positions (without a table) or places in it, and the table
    int in_plane, x0;
    const int frame0 = div_by(row0, a.plane, a.per_plane, &in_plane);    // counted through all query blocks
    const int y0 = div_by(in_plane, a.grid_w, a.per_grid_w, &x0);
    const float inv_w = __builtin_amdgcn_rcpf(float(a.grid_w)), inv_h = __builtin_amdgcn_rcpf(float(a.grid_h));
    const float inv_frames = __builtin_amdgcn_rcpf(float(a.frames_per_block));
    // of row tid of the tile: columns and rows counted on from the first row's
    const int along = x0 + min(tid, rows_end - 1 - row0), down = div_small(along, inv_w), x = along - down * a.grid_w;
    const int frames = div_small(y0 + down, inv_h), y = y0 + down - frames * a.grid_h;
    auto frame_pos = [&](int frame) {
      const int blk = div_small(frame, inv_frames);
      return __shfl(lane_tab, kLaneFrame + blk) + frame - blk * a.frames_per_block;
    };
    if (a.tab_y == 0) {
      pos[lane] = make_int4(frame_pos(frame0 + frames), y, x, 0);
      load_q<4, 16>(v, q_at, q_end, q_step, rows_end - first);
    } else {
      const int last_frame = div_by(rows_end - 1, a.plane, a.per_plane, &in_plane);
      const int to_y = a.pairs_t, to_x = a.pairs_t + a.pairs_h, pairs_w = 64 - to_x;
      // quads of a frame, row and column; where those of frame 0, row y0 and column 0 begin, less the quads before their first
      const int of_t = (to_y + 3) >> 2, of_y = ((to_x + 3) >> 2) - (to_y >> 2), of_x = 16 - (to_x >> 2);
      const int in_y = a.tab_f * of_t - (to_y >> 2), in_x = a.tab_f * of_t + a.tab_y * of_y - (to_x >> 2);
      const int rows_on = y - y0 + (y < y0 ? a.grid_h : 0);
      pos[lane] = make_int4(16 * frames * of_t, 16 * (in_y + rows_on * of_y), 16 * (in_x + x * of_x), 0);
      // The entries, shared out to the threads: pairs of the frames, of the rows, of the columns.  Pairs 0 and 1 of a quad lie in
      // one half of the table, 2 and 3 in the other, so that the 16 lanes of a row read neighbouring 16 bytes.
      uint8_t* const trig = lds + kTrigArea;
      const int n_t = a.tab_f * to_y, n_ty = n_t + a.tab_y * a.pairs_h, n_all = n_ty + a.grid_w * pairs_w;
      const float inv_t = __builtin_amdgcn_rcpf(float(to_y)), inv_p = __builtin_amdgcn_rcpf(float(a.pairs_h)), inv_q = __builtin_amdgcn_rcpf(float(pairs_w));
      // entry e of the table (uniform: the lanes of a wave exchange values)
#define CA_FILL(e0)                                                                                                            \
      {                                                                                                                        \
        const int e = (e0) + tid;                                                                                              \
        const bool on_t = e < n_t, on_y = e < n_ty;                                                                            \
        const int k = e - (on_t ? 0 : (on_y ? n_t : n_ty)), v = div_small(k, on_t ? inv_t : (on_y ? inv_p : inv_q));           \
        const int pair = (on_t ? 0 : (on_y ? to_y : to_x)) + k - v * (on_t ? to_y : (on_y ? a.pairs_h : pairs_w));             \
        const int t_pos = frame_pos(min(frame0 + v, last_frame)), y_pos = y0 + v - (y0 + v >= a.grid_h ? a.grid_h : 0);        \
        const float at = float(on_t ? t_pos : (on_y ? y_pos : v)), k_hi = __shfl(pair_hi, pair), k_lo = __shfl(pair_lo, pair); \
        const float rev = __builtin_amdgcn_fractf(at * k_hi) + at * k_lo;                                                      \
        const int quad = (on_t ? 0 : (on_y ? in_y : in_x)) + v * (on_t ? of_t : (on_y ? of_y : of_x)) + (pair >> 2);           \
        if (e < n_all)                                                                                                         \
          *reinterpret_cast<float2*>(trig + 16 * (quad + ((pair >> 1) & 1 ? a.tab_quads : 0)) + 8 * (pair & 1)) =              \
              make_float2(__builtin_amdgcn_cosf(rev), __builtin_amdgcn_sinf(rev));                                             \
      }
      load_q<4, 8>(v, q_at, q_end, q_step, rows_end - first);
      CA_FILL(0)
      load_q<8, 12>(v, q_at, q_end, q_step, rows_end - first);
      if (n_all > 256) CA_FILL(256)
      load_q<12, 16>(v, q_at, q_end, q_step, rows_end - first);
      for (int e0 = 512; e0 < n_all; e0 += 256) CA_FILL(e0)
#undef CA_FILL
    }
  }
  // Q has landed (and is taken note of as such before other loads are on their way, which the compiler does not count)
#pragma unroll
  for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(v[i]));
  // ---- the first K and V page on their way into the first slots of their rings (beside the rotation where there is one:
  // the 16 loads take the 1000 cycles that their addresses take)
  const uint32_t lane_off = wave * 1024 + lane * 16;   // this lane's 16 bytes inside each 4 KB slice of a page
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  const int slot0 = __builtin_amdgcn_readlane(lane_tab, kLaneSlot + kb0);
  const uint64_t k0 = reinterpret_cast<uint64_t>(a.pool) +
                      ((uint64_t(slot0) * a.pages_per_block + pg0) * a.heads + h) * uint64_t(kPairBytes);
  if (!kRopeQ || a.tab_y == 0)
#pragma unroll
    for (int i = 0; i < 16; ++i) load_page_piece(lds0 + wave * 1024, lane_off, k0, i);
  // ---- rotate, scale by c (scores then leave the matrix pipe in log2 units), round once, park the rows
  // in the second ring slots (rows 0..127 in K's, the others in V's), chunks swizzled as in a page
  int end_again = rows_end;            // (compared anew: 16 masks kept from the loads would not fit the scalar registers)
  asm volatile("" : "+s"(end_again));
  if (kRopeQ) {
    bool on_t[4], on_y[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      on_t[j] = 4 * c16 + j < a.pairs_t;
      on_y[j] = 4 * c16 + j < a.pairs_t + a.pairs_h;
    }
    if (a.tab_y > 0) {
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");       // the table is there (page loads stay in flight)
      // Each of a lane's four pairs has an entry of its own axis.  A lane's first two are of one axis, and so are its last two but
      // in a lane where an axis ends behind the third pair, which has the fourth one read apart, ahead of the others (`ends`).  The
      // reads of a row stand two rows before its products, so that the two run side by side, and a row's share of the page loads
      // behind it.  Cycles of this part: 5200 with all reads first, of which 1700 wait for LDS, 4500 with four reads of 8 bytes.
      const uint8_t* entry[4];
      const int* place[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        entry[j] = lds + kTrigArea + 16 * (c16 + (j >> 1) * a.tab_quads) + 8 * (j & 1);
        place[j] = reinterpret_cast<const int*>(pos + r4) + (on_t[j] ? 0 : (on_y[j] ? 1 : 2));
      }
      auto rotated = [&](int i, const float2 (&t)[4]) {
        const float c = row0 + wave * 64 + r4 + 4 * i < end_again ? a.c : 0.f;       // rows past the end are zeros
        u32x4 out;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t x = v[i][j];
          const float u = __uint_as_float(x << 16), w = __uint_as_float(x & 0xffff0000u);
          out[j] = pack2(turned(u, w, t[j].x, -t[j].y) * c, turned(u, w, t[j].y, t[j].x) * c);
        }
        return out;
      };
      constexpr int kAhead = 2;
      if ((a.pairs_t & 3) != 1 && ((a.pairs_t + a.pairs_h) & 3) != 1) {
        const bool ends = place[3] != place[2];
        int at[16][3];
        float2 fourth[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) at[i][2] = place[3][16 * i], at[i][0] = place[0][16 * i], at[i][1] = place[2][16 * i];
        if (ends) {
#pragma unroll
          for (int i = 0; i < 16; ++i) fourth[i] = *reinterpret_cast<const float2*>(entry[3] + at[i][2]);
        }
        float4 e[kAhead + 1][2];
#pragma unroll
        for (int i = 0; i < 16 + kAhead; ++i) {
          if (i < 16) {
            e[i % (kAhead + 1)][0] = *reinterpret_cast<const float4*>(entry[0] + at[i][0]);
            e[i % (kAhead + 1)][1] = *reinterpret_cast<const float4*>(entry[2] + at[i][1]);
          }
          if (i < kAhead) continue;
          const int k = i - kAhead;
          const float4 lo = e[k % (kAhead + 1)][0], hi4 = e[k % (kAhead + 1)][1];
          const float2 t[4] = {make_float2(lo.x, lo.y), make_float2(lo.z, lo.w), make_float2(hi4.x, hi4.y),
                               make_float2(ends ? fourth[k].x : hi4.z, ends ? fourth[k].y : hi4.w)};
          *reinterpret_cast<u32x4*>(park[k & 3] + (k >> 2) * 4096) = rotated(k, t);
          load_page_piece(lds0 + wave * 1024, lane_off, k0, k);
        }
      } else {                                             // an axis ends behind a lane's first pair: four reads
        float2 e[kAhead + 1][4];
#pragma unroll
        for (int i = 0; i < 16 + kAhead; ++i) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (i < 16) e[i % (kAhead + 1)][j] = *reinterpret_cast<const float2*>(entry[j] + place[j][16 * i]);
          if (i < kAhead) continue;
          const int k = i - kAhead;
          *reinterpret_cast<u32x4*>(park[k & 3] + (k >> 2) * 4096) = rotated(k, e[k % (kAhead + 1)]);
          load_page_piece(lds0 + wave * 1024, lane_off, k0, k);
        }
      }
    } else {
      const float4 hi4 = *reinterpret_cast<const float4*>(args.rev_hi + 4 * c16), lo4 = *reinterpret_cast<const float4*>(args.rev_lo + 4 * c16);
      const float rev_hi[4] = {hi4.x, hi4.y, hi4.z, hi4.w}, rev_lo[4] = {lo4.x, lo4.y, lo4.z, lo4.w};
      wave_lds_fence();
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = r4 + 4 * i;
        const int4 p = pos[r];
        u32x4 out;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float at = float(on_t[j] ? p.x : (on_y[j] ? p.y : p.z));
          const float rev = __builtin_amdgcn_fractf(at * rev_hi[j]) + at * rev_lo[j];
          const float cs = __builtin_amdgcn_cosf(rev), sn = __builtin_amdgcn_sinf(rev);
          const uint32_t x = v[i][j];
          const float u = __uint_as_float(x << 16), w = __uint_as_float(x & 0xffff0000u);
          out[j] = pack2(turned(u, w, cs, -sn) * a.c, turned(u, w, sn, cs) * a.c);
        }
        if (row0 + wave * 64 + r >= end_again) out = u32x4{0, 0, 0, 0};
        *reinterpret_cast<u32x4*>(park[i & 3] + (i >> 2) * 4096) = out;
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int r = r4 + 4 * i;
      u32x4 out;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        out[j] = pack2(__uint_as_float(v[i][j] << 16) * a.c, __uint_as_float(v[i][j] & 0xffff0000u) * a.c);
      if (row0 + wave * 64 + r >= end_again) out = u32x4{0, 0, 0, 0};
      *reinterpret_cast<u32x4*>(park[i & 3] + (i >> 2) * 4096) = out;
    }
  }
  wave_lds_fence();
  // ---- Q fragments: B operand of S^T = K Q^T, a[128:191].  16x16x32: lane holds dims 32ks + 8grp .. +7 of query l15 of query
  // tile t, fragment (t, ks) at a[128 + 4*(4t + ks) ..]; 32x32x16: dims 16ks + 8hi .. +7 of query l31 of column tile
  // nt, fragment (nt, ks) at a[128 + 4*(8nt + ks) ..].
  f32x16 qt[4];
  if constexpr (kCore16) {
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const u32x4 f = *reinterpret_cast<const u32x4*>(parked + (t * 16 + l15) * 256 + (((4 * ks + grp) ^ l15) << 4));
#pragma unroll
      for (int j = 0; j < 4; ++j) qt[t][4 * ks + j] = __uint_as_float(f[j]);
    }
  } else {
#pragma unroll
  for (int nt = 0; nt < 2; ++nt)
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const u32x4 f = *reinterpret_cast<const u32x4*>(parked + (nt * 32 + l31) * 256 + (((2 * ks + hi) ^ l15) << 4));
#pragma unroll
      for (int j = 0; j < 4; ++j) qt[2 * nt + (ks >> 2)][4 * (ks & 3) + j] = __uint_as_float(f[j]);
    }
  }
  __syncthreads();                    // every fragment is in registers: the second slots are free

  // address of page 0 of KV block i for this head: lane i of (tbl_lo, tbl_hi)
  const uint64_t my_off = reinterpret_cast<uint64_t>(a.pool) +
                          (uint64_t(my_slot) * a.pages_per_block * a.heads + h) * uint64_t(kPairBytes);
  const uint32_t tbl_lo = uint32_t(my_off), tbl_hi = uint32_t(my_off >> 32);
  const uint32_t stride = uint32_t(a.heads) * kPairBytes;

  // The first PV product multiplies an all-zero P tile with the last 32 keys (chunks 12..15 of every
  // row) of whatever the second V ring slot holds: make that finite.
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = tid >> 1, ch = 12 + 2 * (tid & 1) + i;
    *reinterpret_cast<u32x4*>(lds + kVRing + kPageBytes + row * 256 + ((ch ^ (row & 15)) << 4)) = u32x4{0, 0, 0, 0};
  }

  // The loop leaves few scalar registers: what the epilogue needs waits in LDS, or is read again from
  // the arguments, through a pointer the compiler cannot see to be the same.
  if (tid == 0) {
    const int part_index = a.range > 0 ? (all_pages > a.range ? xcd * kPartialsPerXcd + nth : -1)
                           : n_chunks > 1 ? (xcd * a.split_items + (item - a.full_items)) * n_chunks + chunk : -1;
    *reinterpret_cast<int4*>(lds + kPosArea) = make_int4(h, row0, rows_end, part_index);
  }
  typedef const __attribute__((address_space(4))) AttnArgs* ArgPtr;
  ArgPtr ap = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();

  // o6/o7 are not early-clobber: the block reads every VGPR input in its first instructions,
  // before it writes v[96:127], and the inputs need somewhere to live (it uses all of v[128:255])
  f32x16 o0, o1, o2, o3, o4, o5, o6, o7;
  float l0, l1, l2, l3, negm0, negm1, negm2 = 0.f, negm3 = 0.f;
  if constexpr (kCore16) {
    // K rows of a key tile: lanes 0..7 hold keys 0..7, lanes 8..15 keys 16..23 (the second tile: 8 further), so that
    // the accumulators of the two tiles hand a lane group exactly the keys of one chunk of a V row
    const uint32_t xk0 = (16 * (l15 >> 3) + (l15 & 7)) * 256 + ((grp ^ (l15 & 7)) << 4);
    const uint32_t xv0 = l15 * 256 + ((grp ^ l15) << 4);
    const uint32_t kidx = 16 * (grp >> 1) + 4 * (grp & 1);
    const uint32_t xl16 = 4 * (lane ^ 16), xl32 = 4 * (lane ^ 32);
#define CA_CORE16_OPERANDS \
    : "=&{v[0:15]}"(o0), "=&{v[16:31]}"(o1), "=&{v[32:47]}"(o2), "=&{v[48:63]}"(o3), "=&{v[64:79]}"(o4), \
    "=&{v[80:95]}"(o5), "={v[96:111]}"(o6), "={v[112:127]}"(o7), "=&{v148}"(l0), "=&{v149}"(l1), \
    "=&{v150}"(l2), "=&{v151}"(l3), "=&{v184}"(negm0), "=&{v188}"(negm1), "=&{v192}"(negm2), "=&{v196}"(negm3) \
    : "{a[128:143]}"(qt[0]), "{a[144:159]}"(qt[1]), "{a[160:175]}"(qt[2]), "{a[176:191]}"(qt[3]), \
    [xk0] "v"(xk0), [xv0] "v"(xv0), [lane_off] "v"(lane_off), [tbl_lo] "v"(tbl_lo), [tbl_hi] "v"(tbl_hi), \
    [kidx] "v"(kidx), [xl16] "v"(xl16), [xl32] "v"(xl32), \
    [n_pages] "s"(n_pages), [n_kvb] "s"(n_kvb), [kb0] "s"(kb0), [pg0] "s"(pg0), \
    [ppb] "s"(a.pages_per_block), [stride] "s"(stride), [last_valid] "s"(a.last_valid), \
    [wave] "s"(wave), [lds0] "s"(lds0), [idle] "s"(uniform(row0 + wave * 64 - rows_end)) \
    : "memory", "vcc", "scc", "m0", CA_CORE16_CLOBBERS
    if constexpr (kTails)
      asm volatile(
#include "attn_core16_tails_gfx950.inc"
          CA_CORE16_OPERANDS);
    else
      asm volatile(
#include "attn_core16_gfx950.inc"
          CA_CORE16_OPERANDS);
  } else {
    const uint32_t xo0 = l31 * 256 + ((hi ^ l15) << 4);    // row offset + swizzled chunk 0 (or 1 for hi)
    const uint32_t kidx = 4 * hi, xlane = 4 * (lane ^ 32);
#define CA_CORE_OPERANDS \
    : "=&{v[0:15]}"(o0), "=&{v[16:31]}"(o1), "=&{v[32:47]}"(o2), "=&{v[48:63]}"(o3), "=&{v[64:79]}"(o4), \
    "=&{v[80:95]}"(o5), "={v[96:111]}"(o6), "={v[112:127]}"(o7), "=&{v148}"(l0), "=&{v149}"(l1), \
    "=&{v150}"(l2), "=&{v151}"(l3), "=&{v184}"(negm0), "=&{v200}"(negm1) \
    : "{a[128:143]}"(qt[0]), "{a[144:159]}"(qt[1]), "{a[160:175]}"(qt[2]), "{a[176:191]}"(qt[3]), \
    [xo0] "v"(xo0), [lane_off] "v"(lane_off), [tbl_lo] "v"(tbl_lo), [tbl_hi] "v"(tbl_hi), \
    [kidx] "v"(kidx), [xlane] "v"(xlane), [n_pages] "s"(n_pages), [n_kvb] "s"(n_kvb), [kb0] "s"(kb0), [pg0] "s"(pg0), \
    [ppb] "s"(a.pages_per_block), [stride] "s"(stride), [last_valid] "s"(a.last_valid), \
    [wave] "s"(wave), [lds0] "s"(lds0) \
    : "memory", "vcc", "scc", "m0", CA_CORE_CLOBBERS
    if constexpr (kTails)
      asm volatile(
#include "attn_core_tails_gfx950.inc"
          CA_CORE_OPERANDS);
    else
      asm volatile(
#include "attn_core_gfx950.inc"
          CA_CORE_OPERANDS);
  }

  asm volatile("" : "+s"(ap));
  const int4 kept = *reinterpret_cast<const int4*>(lds + kPosArea);
  const int o_head = uniform(kept.x), o_row0 = uniform(kept.y), o_end = uniform(kept.z), part_index = uniform(kept.w);
  // ---- normalise and store.  The lane's accumulators are 32 groups of four consecutive dims of a row of the wave: group
  // g of o_j is register 4g of it.  16x16x32: o_j has dims 16j + 4grp .. of query l15 of tile g; 32x32x16: o_j, j = 2mt + nt, has
  // dims 32mt + 8g + 4hi .. of query l31 of tile nt.
  const f32x16 oacc[8] = {o0, o1, o2, o3, o4, o5, o6, o7};
  const float negm[4] = {negm0, negm1, negm2, negm3};
  float l_tot[4];                     // row sums per tile
  if constexpr (kCore16) {            // four lanes share a query
    const float l[4] = {l0, l1, l2, l3};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float half = l[t] + __shfl_xor(l[t], 16, 64);
      l_tot[t] = half + other_half(half);
    }
  } else {
    const float a0 = l0 + l1, a1 = l2 + l3;
    l_tot[0] = a0 + other_half(a0);
    l_tot[1] = a1 + other_half(a1);
    l_tot[2] = l_tot[3] = 0.f;
  }
  if (part_index >= 0) {
    // partial result: accumulators as they are, plus (m_ref, row sum) per row
    float* part = ap->partials + size_t(part_index) * kPartialFloats;
    float4* slab = reinterpret_cast<float4*>(part) + wave * 32 * 64 + lane;
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        slab[(4 * j + g) * 64] = make_float4(oacc[j][4 * g + 0], oacc[j][4 * g + 1], oacc[j][4 * g + 2], oacc[j][4 * g + 3]);
    float2* ml = reinterpret_cast<float2*>(part + kPartialMl) + wave * 64;
    if constexpr (kCore16) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (grp == 0) ml[t * 16 + l15] = make_float2(-negm[t], l_tot[t]);
    } else {
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
        if (hi == 0) ml[nt * 32 + l31] = make_float2(-negm[nt], l_tot[nt]);
    }
    return;
  }
  // rows leave through LDS: a wave's 64 rows in 16 KB of its own, chunks swizzled, then 16 lanes to a row
  __syncthreads();                    // no wave reads pages any more, no page load is in flight
  uint8_t* const mine = lds + wave * 64 * 256;
  float inv[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) inv[t] = 1.0f / l_tot[t];
#pragma unroll
  for (int j = 0; j < 8; ++j)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x16& o = oacc[j];
      const float f = inv[kCore16 ? g : j & 1];
      const int row = kCore16 ? g * 16 + l15 : (j & 1) * 32 + l31;
      const int piece = kCore16 ? 4 * j + grp : 8 * (j >> 1) + 2 * g + hi;          // of 8 bytes
      u32x2 w;
      w[0] = pack2(o[4 * g + 0] * f, o[4 * g + 1] * f);
      w[1] = pack2(o[4 * g + 2] * f, o[4 * g + 3] * f);
      *reinterpret_cast<u32x2*>(mine + row * 256 + (((piece >> 1) ^ l15) << 4) + 8 * (piece & 1)) = w;
    }
  wave_lds_fence();
  uint16_t* op = ap->o + int64_t(o_head) * 128 + c16 * 8;
  const int64_t o_stride = int64_t(ap->heads) * 128;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r = r4 + 4 * i, row = o_row0 + wave * 64 + r;
    const u32x4 w = *reinterpret_cast<const u32x4*>(mine + r * 256 + ((c16 ^ (r & 15)) << 4));
    if (row < o_end) *reinterpret_cast<u32x4*>(op + row * o_stride) = w;
  }
}


// Combines the partial results of the split work items: for every row, the partials are brought
// to the largest of their exponent references, summed and normalised.  Eight workgroups per tile: a wave takes
// four register groups of one row of the attention kernel's tiles, and a lane keeps the place it had
// there, so that every read of a partial tile is 1 KB of contiguous memory.
struct MergeArgs {                     // as in AttnHead; 64 bytes: a launch with more takes the host up to 1 us longer
  const float* partials;
  uint16_t* o;
  uint64_t range_segs;                 // 0: every item has `split` ranges, side by side
  int32_t heads, tiles_per_seg, items, n_seg, seg_first, seg_rows;
  int32_t split_and_items, full_items; // split + 256 split_items
  uint32_t per_seg, per_tiles;
};
static_assert(sizeof(MergeArgs) == 64, "one cache line");

template <bool kCore16, bool kRanges>
__global__ __launch_bounds__(256) void merge_partials_kernel(MergeArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l31 = lane & 31, hi = lane >> 5, l15 = lane & 15, grp = lane >> 4;
  const int xcd = blockIdx.y, sidx = blockIdx.x, piece = blockIdx.z;   // (on the XCD that wrote the partials: 1 % slower steps)
  WorkItem wi;
  int split = a.split_and_items & 255;
  uint32_t place[kMaxSplit];                                   // of range c, counted in partial results from `first_part` on
  const float* first_part = a.partials;
  if (kRanges) {
    const Share share = share_of(a, xcd);
    wi = decode_item(a, share, sidx);
    if (wi.h < 0) return;
    uint64_t segs = a.range_segs;
    uint32_t at = xcd * kPartialsPerXcd + sidx;
    split = 0;
#pragma unroll
    for (int c = 0; c < kMaxSplit; ++c, segs >>= 4) {
      place[c] = at;
      at += share.count(int(segs & 15));
      split += int(segs & 15) > wi.seg;
    }
    if (split < 2) return;                                     // written by its workgroup
  } else {
    first_part += size_t(xcd * (a.split_and_items >> 8) + sidx) * split * kPartialFloats;
#pragma unroll
    for (int c = 0; c < kMaxSplit; ++c) place[c] = c;
  }
  const int wrow = piece >> 1;                            // the attention kernel's wave
  // 16x16x32: query tile t, accumulators j0 .. j0+3 (dims 16 j0 ..); 32x32x16: column tile nt, accumulator 2 mt + nt
  const int t = 2 * (piece & 1) + (wave & 1), j0 = 4 * (wave >> 1);
  const int nt = piece & 1, mt = wave;
  const int first = kCore16 ? 16 * t : 32 * nt;
  const int row_in_tile = wrow * 64 + first + (kCore16 ? l15 : l31);
  const float* ml = first_part + kPartialMl + 2 * row_in_tile;
  constexpr int kStep = kCore16 ? 4 * 64 : 64;                 // from one of the four groups to the next
  const float4* part = reinterpret_cast<const float4*>(first_part) + (wrow * 32 + (kCore16 ? 4 * j0 + t : 4 * (2 * mt + nt))) * 64 + lane;
  // All references and row sums are requested together and with them the accumulators of the first
  // kBatch partials: a launch of this kernel is two or three memory latencies long.  With one range after the other
  // 6.0 us for 15 tiles in seven ranges and 9.2 for 60 in six, now 4.4 and 8.1.
  float2 y[kMaxSplit];
#pragma unroll
  for (int c = 0; c < kMaxSplit; ++c) {
    y[c] = make_float2(-INFINITY, 0.f);
    if (c < split) y[c] = *reinterpret_cast<const float2*>(ml + size_t(place[c]) * kPartialFloats);
  }
  constexpr int kBatch = 4;
  float4 x[kBatch][4], acc[4];
  auto request = [&](int c0) {
#pragma unroll
    for (int b = 0; b < kBatch; ++b)
      if (c0 + b < split) {
#pragma unroll
        for (int g = 0; g < 4; ++g) x[b][g] = part[size_t(place[c0 + b]) * (kPartialFloats / 4) + g * kStep];
      }
  };
  request(0);
  __builtin_amdgcn_sched_barrier(0);
  if (!kRanges) {
    wi = decode_item(a, share_of(a, xcd), a.full_items + sidx);
    if (wi.h < 0) return;
  }
  const int row = wi.row0 + row_in_tile;
  if (wi.row0 + wrow * 64 + first >= wi.rows_end) return;
  float m = y[0].x, l = 0.f;
#pragma unroll
  for (int c = 1; c < kMaxSplit; ++c) m = fmaxf(m, y[c].x);
#pragma unroll
  for (int g = 0; g < 4; ++g) acc[g] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int c0 = 0; c0 < kMaxSplit; c0 += kBatch) {
    if (c0 > 0) {
      if (split <= c0) break;
      request(c0);
    }
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      if (c0 + b >= split) break;
      const float wgt = __builtin_amdgcn_exp2f(y[c0 + b].x - m);
      l += wgt * y[c0 + b].y;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        acc[g].x += wgt * x[b][g].x; acc[g].y += wgt * x[b][g].y; acc[g].z += wgt * x[b][g].z; acc[g].w += wgt * x[b][g].w;
      }
    }
  }
  if (row >= wi.rows_end) return;
  const float inv = 1.0f / l;
  uint16_t* op = a.o + (int64_t(row) * a.heads + wi.h) * 128 + (kCore16 ? 16 * j0 + 4 * grp : 32 * mt + 4 * hi);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    u32x2 w;
    w[0] = pack2(acc[g].x * inv, acc[g].y * inv);
    w[1] = pack2(acc[g].z * inv, acc[g].w * inv);
    *reinterpret_cast<u32x2*>(op + (kCore16 ? 16 : 8) * g) = w;
  }
}

}  // namespace

// variant 0: default; 1: no tail balancing (every work item walks its whole KV range)
int32_t attn_bf16_variant_ok(int variant) { return variant == 0 || variant == 1 ? CA_OK : CA_EINVAL; }

namespace {

// How many page ranges the items are cut into that leave CUs idle: all of a launch, or what a launch of more than one round
// leaves for its last.  A walk of n pages cut in s takes ceil(n / s) page times of 1.95 us; against that stand the merge
// launch, about one page time, and every partial result that is written and read again (135 KB), 1/40 of one.
// Measured, whole forwards: 1 item of 14 pages 37.7 us whole, 26.7 in two, 18.8 in seven; 15 of 20 pages 54.8 whole, 41.1 / 30.1 /
// 32.3 in 2 / 5 / 8; 64 of 14 pages 42.0 whole, 33.9 in four; 38 of 259 pages 473 whole, 141 in six; 120 of 14 pages
// 44.9 whole, 44.2 in two.  Last rounds, whole steps: 8 of 264 items, 21 pages, 106.6 in 2, 92.8 in 11; 24 of 280, 16 pages, 90.7
// in 2, 84.9 in 4; 16 of 272, 34 pages, 139.4 in 4, 132.4 in 9.
int split_of_idle_round(int items_per_xcd, int cus_per_xcd, int items, int min_pages, int max_pages, int capacity) {
  int best = 1, best_cost = 40 * max_pages;                    // in 40ths of a page time
  for (int s = 2; s <= kMaxSplit && s * items_per_xcd <= cus_per_xcd && s <= min_pages; ++s) {
    if (8 * items_per_xcd * s > capacity) break;
    const int cost = 40 * ((max_pages + s - 1) / s + 1) + items * s;
    if (cost < best_cost) {
      best = s;
      best_cost = cost;
    }
  }
  return best;
}

// The same for launches with walks of several lengths that leave CUs idle: ranges of one length for all of them, since the
// longest range is what counts.  Fills in `range`, `range_segs`, `split` (of the longest walk) and, as full_items, the workgroups
// of an XCD.  Whole block-causal steps with each walk in as many ranges, and so: 12 heads, two
// blocks of 924 tokens over one 49.8 / 47.2 us; six, five of 756 over three 74.4 / 63.4; three, five of 1596 over one 102.5 /
// 82.8; eight, five of 252 32.1 / 30.0; two, two of 4680 over two 135.2 / 133.4; the other way three, five of 390 over two 31.3 /
// 32.4; four, three of 1200 over three 56.2 / 57.2.
void ranges_of_idle_launch(AttnArgs& a, int cus_per_xcd) {
  const int most = cus_per_xcd < kPartialsPerXcd ? cus_per_xcd : kPartialsPerXcd, max_pages = a.vis_first * a.pages_per_block;
  int64_t best_cost = 40 * int64_t(max_pages);                 // in 40ths of a page time
  for (int s = 2; s <= kMaxSplit && s <= max_pages; ++s) {
    const int range = (max_pages + s - 1) / s;
    if ((max_pages + range - 1) / range != s) continue;
    // an XCD has whole columns and of one column, at most, its first (longest) walks
    int whole = 0, first = 0;
    for (int i = 0; i < a.n_seg; ++i) {
      const int n = ((a.vis_first - i) * a.pages_per_block + range - 1) / range;
      whole += n;
      if (i < a.work_per_xcd % a.n_seg) first += n;
    }
    const int ranges = a.work_per_xcd / a.n_seg * whole + first;
    if (ranges > most) continue;
    const int64_t cost = 40 * int64_t(range + 1) + 8 * ranges;
    if (cost >= best_cost) continue;
    best_cost = cost;
    a.range = range;
    a.split = s;
    a.full_items = ranges;
  }
  for (int c = 0; a.range > 0 && c < a.split; ++c) {           // a walk has range c if it is longer than c ranges
    int segs = 0;
    while (segs < a.n_seg && (a.vis_first - segs) * a.pages_per_block > c * a.range) ++segs;
    a.range_segs |= uint64_t(segs) << (4 * c);
  }
}

// The loop on the 16x16x32 instruction draws less power a flop, the one on 32x32x16 needs fewer cycles: where most
// CUs work at once and long enough, power decides.  Whole forwards, us, 32x32x16 / 16x16x32, by workgroups of a round
// x pages of a walk: 171 x 259 545 / 528, 228 x 259 658 / 610, 228 x 43 135 / 129, 250 x 14 54.4 / 51.7, 200 x 10
// 41.1 / 40.6; 152 x 259 515 / 526, 160 x 14 46.7 / 47.1, 240 x 5 35.9 / 36.4, 14 x 1 19.5 / 21.5.  Along the line a
// few go the other way by little: 200 x 14 48.3 / 49.1, 152 x 74 168 / 159.
bool takes_core16(const AttnArgs& a, int max_pages, int n_cu) {
  const bool alone = a.full_items == 0;                        // all items cut
  const int64_t workgroups = a.range > 0 ? 8 * int64_t(a.full_items) : int64_t(a.items) * (alone ? a.split : 1);
  return 3 * workgroups >= 2 * int64_t(n_cu) && (a.range > 0 ? a.range : max_pages / (alone ? a.split : 1)) >= 10;
}

// Which launches take the loops with short pages: two steps instead of four are walked of a block's last page, and
// masked tiles find their code in fewer places.  Whole forwards, us, without / with: 12 heads, five blocks of 1170
// tokens (18 in the last page) 345 / 328, 40 heads of 180 (52) 73 / 53.5, 40 of 390 (6) 64.5 / 56, 16 of 1683 (19)
// 148.8 / 143.3.  With more than 64 tokens in the last page both loops walk the same steps and take the same time
// (55.0 / 55.3, 669 / 673).
bool has_tails(const AttnArgs& a) { return a.last_valid <= 64; }

// Fills the kernel arguments for one forward.  Splitting: `capacity` partial results fit in
// the scratch area; with adapt the split is reduced until the partials fit, without it the split
// the device's CU count asks for is kept and *partials_needed tells the caller how many it takes.
int32_t plan_attn_bf16(const AttnPlan& p, int variant, const void* q, void* out, const void* pool, void* partials_dev,
                       int capacity, bool adapt, AttnArgs* args, int* partials_needed, bool* core16) {
  if (p.head_dim != 128 || p.page_tokens != 128) return CA_EUNSUPPORTED;
  if (attn_bf16_variant_ok(variant) != CA_OK) return CA_EINVAL;
  AttnArgs& a = *args;
  a = AttnArgs{};
  a.q = static_cast<const uint16_t*>(q);
  a.o = static_cast<uint16_t*>(out);
  a.pool = static_cast<const uint8_t*>(pool);
  a.heads = p.heads;
  a.pages_per_block = p.pages_per_block;
  a.last_valid = p.block_tokens - (p.pages_per_block - 1) * 128;
  for (int i = 0; i < p.n_kv; ++i) a.lanes[kLaneSlot + i] = p.kv_slot[i];
  // Query segments: rows sharing one visible prefix are tiled together.  A bidirectional
  // cascade is one segment; block-causal gives one segment per in-flight block.
  if (p.uniform) {
    a.n_seg = 1;
    a.seg_first = 0;
    a.seg_rows = p.n_q_blocks * p.block_tokens;
    a.vis_first = p.n_vis[0];
  } else {
    // one segment per query block, the longest prefix (latest block) first
    a.n_seg = p.n_q_blocks;
    a.seg_first = (p.n_q_blocks - 1) * p.block_tokens;
    a.seg_rows = p.block_tokens;
    a.vis_first = p.n_vis[p.n_q_blocks - 1];
    for (int i = 0; i + 1 < p.n_q_blocks; ++i)                 // a later block sees one more (CacheMeta::plan_forward)
      if (p.n_vis[i + 1] != p.n_vis[i] + 1) return CA_EINVAL;
  }
  const int tiles = (a.seg_rows + kRowsPerWg - 1) / kRowsPerWg;
  a.tiles_per_seg = tiles;
  a.items = tiles * p.heads * a.n_seg;
  a.work_per_xcd = (a.items + 7) / 8;
  a.c = 1.4426950408889634f / sqrtf(float(p.head_dim));
  a.q_tok_stride = int64_t(p.heads) * 128;       // rotated queries are contiguous
  a.q_head_stride = 128;
  // Splitting.  One workgroup occupies a CU, an XCD has n_cu/8 of them, and all items of a
  // launch take about the same time: after floor(items / cus) full rounds, `rem` items would run
  // alone while the other CUs idle.  Their KV walks (the shortest of the launch) are cut into up to floor(cus / rem) ranges.
  // A launch that does not give every CU an item has all of them cut.
  int n_cu = 0;
  if (const int32_t rc = device_cu_count(&n_cu); rc != CA_OK) return rc;
  const int cus_per_xcd = n_cu >= 8 ? n_cu / 8 : 1;
  a.split = 1;
  a.split_items = 0;
  a.full_items = a.work_per_xcd;
  a.partials = static_cast<float*>(partials_dev);
  const int rem = a.work_per_xcd % cus_per_xcd;
  int min_vis = p.n_vis[0];                                    // shortest KV walk of the launch
  for (int i = 1; i < p.n_q_blocks; ++i) min_vis = p.n_vis[i] < min_vis ? p.n_vis[i] : min_vis;
  int max_vis = p.n_vis[0];
  for (int i = 1; i < p.n_q_blocks; ++i) max_vis = p.n_vis[i] > max_vis ? p.n_vis[i] : max_vis;
  const int min_pages = min_vis * p.pages_per_block, max_pages = max_vis * p.pages_per_block;
  *partials_needed = 0;
  if (partials_dev && variant == 0 && rem > 0) {
    int split = 1;
    if (a.work_per_xcd > cus_per_xcd) {
      // With walks of several lengths CUs come to the last items one after the other, and what those could gain is less: ranges
      // of at least eight pages, and as many as there are CUs.  (With the rule for walks of one length 64 of 320 items with walks
      // of 14 to 42 pages go from 120.5 us to 128.7, from whole to three ranges; with an estimate of when the CUs come 48 of 300
      // with 70 to 110 pages from 304 to 310, from five ranges to four.)
      if (a.n_seg == 1) {
        split = split_of_idle_round(rem, cus_per_xcd, 8 * rem, min_pages, max_pages, adapt ? capacity : INT32_MAX);
      } else {
        split = cus_per_xcd / rem;
        if (split > 8) split = 8;
        while (split > 1 && (min_pages < 8 * split || (adapt && 8 * rem * split > capacity))) --split;
      }
    } else if (a.n_seg > 1 && capacity >= kMaxPartials) {
      ranges_of_idle_launch(a, cus_per_xcd);
      if (a.range > 0) *partials_needed = kMaxPartials;
    } else {
      split = split_of_idle_round(rem, cus_per_xcd, a.items, min_pages, max_pages, capacity);
    }
    if (split > 1) {
      a.split = split;
      a.split_items = rem;
      a.full_items = a.work_per_xcd - rem;
      *partials_needed = 8 * rem * split;
    }
  }
  *core16 = takes_core16(a, max_pages, n_cu);
  a.per_seg = reciprocal(a.n_seg);
  a.per_tiles = reciprocal(a.tiles_per_seg);
  a.per_pages = reciprocal(a.pages_per_block);
  a.per_split = reciprocal(a.split);
  a.per_split_items = reciprocal(a.split_items);
  return CA_OK;
}

template <bool kRopeQ, bool kCore16, bool kTails>
int32_t enqueue_attn_bf16(const AttnArgs& a, void* stream) {
  const dim3 grid((unsigned)((a.full_items + a.split_items * a.split) * 8));
  const auto kernel = attn_bf16_kernel<kRopeQ, kCore16, kTails>;
  hipLaunchKernelGGL(kernel, grid, dim3(256), kAttnLds, static_cast<hipStream_t>(stream), a);
  if (a.split > 1) {
    const int cut = a.range > 0 ? a.work_per_xcd : a.split_items;        // items of an XCD
    const MergeArgs m{a.partials, a.o, a.range_segs, a.heads, a.tiles_per_seg, a.items, a.n_seg, a.seg_first, a.seg_rows,
                      a.split + 256 * cut, a.full_items, a.per_seg, a.per_tiles};
    const auto merge = a.range > 0 ? merge_partials_kernel<kCore16, true> : merge_partials_kernel<kCore16, false>;
    hipLaunchKernelGGL(merge, dim3((unsigned)cut, 8, kRowsPerWg / 32), dim3(256), 0, static_cast<hipStream_t>(stream), m);
  }
  return finish_launch("attn_bf16.hip");
}

template <bool kRopeQ>
int32_t enqueue_attn_bf16(const AttnArgs& a, bool core16, void* stream) {
  const KernelLds kernels[] = {{reinterpret_cast<const void*>(attn_bf16_kernel<kRopeQ, false, false>), kAttnLds},
                               {reinterpret_cast<const void*>(attn_bf16_kernel<kRopeQ, false, true>), kAttnLds},
                               {reinterpret_cast<const void*>(attn_bf16_kernel<kRopeQ, true, false>), kAttnLds},
                               {reinterpret_cast<const void*>(attn_bf16_kernel<kRopeQ, true, true>), kAttnLds}};
  if (const int32_t rc = ensure_dynamic_lds(kernels, 4, kRopeQ ? kLdsAttnRope : kLdsAttn); rc != CA_OK) return rc;
  if (has_tails(a)) return core16 ? enqueue_attn_bf16<kRopeQ, true, true>(a, stream) : enqueue_attn_bf16<kRopeQ, false, true>(a, stream);
  return core16 ? enqueue_attn_bf16<kRopeQ, true, false>(a, stream) : enqueue_attn_bf16<kRopeQ, false, false>(a, stream);
}

}  // namespace

int32_t launch_attn_bf16(const AttnPlan& p, int variant, const void* q, void* out, const void* pool,
                         void* partials_dev, int max_partials, void* stream) {
  AttnArgs a;
  int needed = 0;
  bool core16 = false;
  if (const int32_t rc = plan_attn_bf16(p, variant, q, out, pool, partials_dev, max_partials, true, &a, &needed, &core16);
      rc != CA_OK)
    return rc;
  return enqueue_attn_bf16<false>(a, core16, stream);
}

int32_t launch_attn_bf16_rope(const AttnPlan& p, const QRopePlan& rp, int variant, const void* q, void* out,
                              const void* pool, void* partials_dev, int max_partials, void* stream) {
  AttnArgs a;
  int needed = 0;
  bool core16 = false;
  if (const int32_t rc = plan_attn_bf16(p, variant, q, out, pool, partials_dev, max_partials, true, &a, &needed, &core16);
      rc != CA_OK)
    return rc;
  const double two_pi = 6.283185307179586476925286766559;
  for (int j = 0; j < kMaxPairs; ++j) {
    const double rev = rp.geom.freq[j] / two_pi;
    int e = 0;
    const double m = std::frexp(rev, &e);                       // rev = m 2^e, 0.5 <= m < 1
    const double head = std::ldexp(std::floor(std::ldexp(m, 12)), e - 12);
    a.rev_hi[j] = float(head);
    a.rev_lo[j] = float(rev - head);
  }
  a.pairs_t = rp.geom.pairs_t;
  a.pairs_h = rp.geom.pairs_h;
  a.grid_h = rp.geom.grid_h;
  a.grid_w = rp.geom.grid_w;
  a.plane = rp.geom.grid_h * rp.geom.grid_w;
  a.per_plane = reciprocal(a.plane);
  a.per_grid_w = reciprocal(a.grid_w);
  a.frames_per_block = p.block_tokens / a.plane;
  // what the 256 consecutive rows of a tile can meet: that many frames, rows (from the first one's on, round the
  // end), all columns
  a.tab_f = kRowsPerWg / a.plane + 2;
  a.tab_y = kRowsPerWg / a.grid_w + 2 < a.grid_h ? kRowsPerWg / a.grid_w + 2 : a.grid_h;
  // no table where it does not fit, and where a quad has pairs of all three axes
  const int to_y = a.pairs_t, to_x = a.pairs_t + a.pairs_h;
  const int64_t quads = int64_t(a.tab_f) * ((to_y + 3) / 4) + int64_t(a.tab_y) * ((to_x + 3) / 4 - to_y / 4) + int64_t(a.grid_w) * (16 - to_x / 4);
  if (quads > kTrigQuads || (to_y < to_x && to_x < 64 && to_y / 4 == to_x / 4 && to_y % 4 != 0))
    a.tab_y = 0;
  else
    a.tab_quads = int32_t(quads);
  for (int i = 0; i < p.n_q_blocks; ++i) {
    // positions must stay below 4096 for the exact head product (frames are the only axis that grows)
    if (rp.first_frame[i] < 0 || rp.first_frame[i] + p.block_tokens / a.plane >= 4096) return CA_EUNSUPPORTED;
    a.lanes[kLaneFrame + i] = int32_t(rp.first_frame[i]);
  }
  if (rp.geom.grid_h >= 4096 || rp.geom.grid_w >= 4096) return CA_EUNSUPPORTED;
  a.q_tok_stride = rp.tok_stride;
  a.q_head_stride = rp.head_stride;
  return enqueue_attn_bf16<true>(a, core16, stream);
}

// ---- the same launch with the partial results in device memory this library holds itself, for
// callers that cannot hand over or allocate any: a file-scope array, one copy per GPU, which
// stays with the process.  Host code never uses the array's name as an address: the address on
// the current device is looked up once per device and kept.
namespace {

constexpr int kStaticPartials = 256;      // 256 tiles x 256 rows x 132 floats = 34.6 MB per GPU
static __device__ __align__(256) float scratch[size_t(kStaticPartials) * kPartialFloats];

std::atomic<float*> g_static_scratch[kMaxDevices];

int32_t static_scratch_on_current_device(float** out) {
  int dev = 0;
  if (const hipError_t e = hipGetDevice(&dev); e != hipSuccess) return device_failure("hipGetDevice", e);
  if (dev < 0 || dev >= kMaxDevices) return CA_EUNSUPPORTED;
  float* ptr = g_static_scratch[dev].load(std::memory_order_acquire);
  if (!ptr) {
    void* sym = nullptr;
    if (const hipError_t e = hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch)); e != hipSuccess || !sym)
      return device_failure("hipGetSymbolAddress(scratch)", e);
    ptr = static_cast<float*>(sym);
    g_static_scratch[dev].store(ptr, std::memory_order_release);
  }
  *out = ptr;
  return CA_OK;
}

}  // namespace

void attn_static_scratch_prepare() {
  float* ptr = nullptr;
  if (static_scratch_on_current_device(&ptr) != CA_OK) (void)hipGetLastError();   // the entry point will try again
}

int32_t launch_attn_bf16_static(const AttnPlan& p, int variant, const void* q, void* out, const void* pool,
                                void* stream) {
  float* ptr = nullptr;
  if (const int32_t rc = static_scratch_on_current_device(&ptr); rc != CA_OK) return rc;
  AttnArgs a;
  int needed = 0;
  bool core16 = false;
  // the split the device's CU count asks for, as launch_attn_bf16 takes it when its area is large
  // enough; what does not fit the static area is refused, not shrunk
  if (const int32_t rc = plan_attn_bf16(p, variant, q, out, pool, ptr, kStaticPartials, false, &a, &needed, &core16); rc != CA_OK)
    return rc;
  if (needed > kStaticPartials) return CA_ETOOBIG;
  return enqueue_attn_bf16<false>(a, core16, stream);
}

}  // namespace ca
