// Y[M,N] = X[M,K] . W[N,K]^T in bf16 with fp32 accumulation: the linear maps either side of the
// attention inside a DiT layer (QKV projection before it, output projection after it).
//
//   Plain products that fill the chip with tiles of 256 columns are gemm_rows.hip's, the others gemm_tiles.hip's
//   (dispatch_gemm_plain picks).
//   gemm_bf16_kernel is the QKV projection of the blocks in flight with the publication of
//   their K/V fused into its epilogue (Sec. 3.3: every block's K/V go to the shared pool at every
//   self-attention layer): row tiles are counted per block, so that a wave's 128 x 128 sub-tile is
//   exactly one page of one head; K sub-tiles are rotated and stored as K pages, V sub-tiles are
//   stored transposed as V pages, Q sub-tiles go to a packed tensor -- the same bytes the separate
//   cache-write kernel produces from the projection's output, without that output ever being
//   written.
//   Workgroup = 4 waves = a tile of 256 or 128 x 256 of Y, one wave per SIMD; the main loop (K in stages of 64, both operands
//   through rings in LDS that together fill its 160 KB) is the assembly emitted by gen_gemm_core.py, which documents
//   the pipeline and the register map.  This file holds the set-up, the epilogue (the tile goes through LDS) and the launch.
//   Workgroups are numbered so that the 32 running together on one XCD share rows of X and W in its L2 (tile_of_workgroup).
#include <hip/hip_runtime.h>

#include "ca_internal.hpp"

namespace ca {
namespace {

#include "rope_device.hpp"
#include "gemm_tiles.hpp"
#include "gemm_tile_kernel.hpp"

typedef __attribute__((ext_vector_type(16))) uint32_t u32x16;

constexpr int kTile = 256;
constexpr int kEpiWave = 128 * kEpiRow;
// kGemmLds: main loop: 3 W stages + 2 X stages of 32 KB; epilogue: 4 x kEpiWave
static_assert(4 * kEpiWave + 2 * kTrigBytes <= kGemmLds, "epilogue staging and two trig tables fit");

// What the publishing epilogue needs beyond the product itself.
struct PublishArgs {
  RopeGeom g;
  uint8_t* pool;
  int32_t heads, pages_per_block;
  int32_t slot[kMaxInflight];
  int64_t first_frame[kMaxInflight];
  TrigTable tab;                                  // per-page cos/sin table (n_f == 0: threads evaluate their own)
};

struct GemmArgs {
  const uint16_t* x;
  const uint16_t* w;
  uint16_t* y;                                    // publishing: the packed queries [M][heads * 128]
  int32_t M, N, K;
  int64_t ldx, ldw, ldy;                          // row strides in elements
  int32_t tiles_m, tiles_n, more;                 // as in LinearArgs
  int32_t block_cols;                             // columns of 8 x 4 blocks where tiles go by blocks (publishing), or 0
  // Row tiles are counted inside row blocks of block_rows rows, tiles_per_block each (the last
  // one ragged): one block spanning all of M for the plain product, one per in-flight block when
  // publishing.
  int32_t block_rows, tiles_per_block;
  PublishArgs pub;                                // publishing only
};

template <>
struct TileArgsOf<true> {
  using type = GemmArgs;
};

#include "gemm_core_clobbers.inc"

// ---- publishing epilogue.  A 128 x 128 tile in LDS (`tile`, rows of kEpiRow bytes, kEpiRowV in the v section) is one
// head of q, k or v (output rows are ordered q|k|v, head, dim: `col` is its first) for the 128 tokens of page `page`
// of block `blk`, rows m0 .. of the product.  kThreads threads share it, this one is number t; a page's cos / sin table
// is filled by fill_n threads, this one number fill_t.  Every thread of the workgroup calls this (there is a barrier in
// it) and all tiles of a workgroup are of one section.
template <int kThreads, typename Args>
__device__ __forceinline__ void publish_tile(const Args& a, const uint8_t* tile, int col, int blk, int page, int m0,
                                             float2* trig, int t, int fill_t, int fill_n) {
  constexpr int kRowsPerTrip = kThreads / 16;
  const PublishArgs& pb = a.pub;
  const int width = pb.heads * 128;
  const int section = col / width, head = (col - section * width) >> 7;
  const int tok0 = page * 128;                                                // first token of the page in its block
  const int c = t & 15, r4 = t >> 4;
  if (section == 0) {                      // q: as it is (the attention kernel rotates it), packed rows
#pragma unroll 4
    for (int it = 0; it < 128 / kRowsPerTrip; ++it) {
      const int row = it * kRowsPerTrip + r4;
      const u32x4 v = *reinterpret_cast<const u32x4*>(tile + row * kEpiRow + c * 16);
      if (tok0 + row < a.block_rows)
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(a.y + int64_t(m0 + row) * a.ldy + head * 128 + c * 8));
    }
    return;
  }
  const bool has_page = page < pb.pages_per_block;
  uint8_t* kpage = pb.pool + ((int64_t(pb.slot[blk]) * pb.pages_per_block + (has_page ? page : 0)) * pb.heads + head) *
                                 int64_t(2 * 128 * 128 * 2);
  if (section == 1) {                      // k: rotate by the token's position, K page rows, pad rows zero
    TrigLayout lay{};
    if (pb.tab.n_f > 0) {
      lay = trig_layout(pb.g, pb.tab, tok0, a.block_rows, pb.first_frame[blk]);
      if (has_page) trig_fill(pb.g, lay, trig, fill_t, fill_n);
    }
    __syncthreads();
    if (!has_page) return;
    // the thread's rows are tokens tok0 + r4 + kRowsPerTrip it
    TokenPos p = token_pos(min(tok0 + r4, a.block_rows - 1), pb.first_frame[blk], pb.g.grid_h, pb.g.grid_w);
#pragma unroll 2
    for (int it = 0; it < 128 / kRowsPerTrip; ++it, p = token_advance(p, kRowsPerTrip, pb.g.grid_h, pb.g.grid_w)) {
      const int row = it * kRowsPerTrip + r4;
      U4 kk = {0, 0, 0, 0};
      if (tok0 + row < a.block_rows) {
        float cs[4], sn[4];
        if (pb.tab.n_f > 0) {
          trig_pick(pb.g, lay, trig, p, c, cs, sn);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) pair_cs<false>(pb.g, p, c * 4 + j, &cs[j], &sn[j]);
        }
        const U4 raw = *reinterpret_cast<const U4*>(tile + row * kEpiRow + c * 16);
        Vec8<uint16_t> e;
        e.v[0] = bf16_lo(raw.x); e.v[1] = bf16_hi(raw.x); e.v[2] = bf16_lo(raw.y); e.v[3] = bf16_hi(raw.y);
        e.v[4] = bf16_lo(raw.z); e.v[5] = bf16_hi(raw.z); e.v[6] = bf16_lo(raw.w); e.v[7] = bf16_hi(raw.w);
        rotate8(e, cs, sn);
        kk.x = pack_bf16(e.v[0], e.v[1]); kk.y = pack_bf16(e.v[2], e.v[3]);
        kk.z = pack_bf16(e.v[4], e.v[5]); kk.w = pack_bf16(e.v[6], e.v[7]);
      }
      store_once(kpage + row * 256 + ((c ^ (row & 15)) << 4), kk);
    }
    return;
  }
  // v: V page rows are dims; chunk c of a row holds tokens 16 (c / 2) + 4 (c % 2) + {0..3, 8..11}
  if (!has_page) return;
  uint8_t* vpage = kpage + 128 * 128 * 2;
  const int tb = 16 * (c >> 1) + 4 * (c & 1);
#pragma unroll 2
  for (int it = 0; it < 128 / kRowsPerTrip; ++it) {
    const int d = it * kRowsPerTrip + r4;
    uint32_t e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int tok = tb + (j & 3) + 8 * (j >> 2);
      const uint32_t w = *reinterpret_cast<const uint16_t*>(tile + tok * kEpiRowV + d * 2);
      e[j] = tok0 + tok < a.block_rows ? w : 0u;
    }
    U4 o;
    o.x = e[0] | (e[1] << 16); o.y = e[2] | (e[3] << 16);
    o.z = e[4] | (e[5] << 16); o.w = e[6] | (e[7] << 16);
    store_once(vpage + d * 256 + ((c ^ (d & 15)) << 4), o);
  }
}

// Which tile a workgroup of gemm_bf16_kernel takes, if any.  Tiles are numbered down bands of eight row tiles and
// dealt to the XCDs (workgroup b runs on b % 8) 32 at a time, so that the workgroups that run together on one share 8
// row slabs of X and 4 of W in its L2, and those of all XCDs lie close together; what is left over for the last round
// goes by last_round_share.  Blocks of 8 x 4 tiles counted in a grid of such blocks, as they were dealt before, leave
// some XCDs with twice the tiles of others where the grid's edge cuts blocks: 4680 x 1536 x 1536 in 222 tiles 39 us,
// now 23; 9360 x 5120 x 5120 404 / 332, 14040 x 15360 x 5120 1500 / 1465.  Where it does not they are up to 1 %
// ahead, within the noise: 23400 x 15360 x 5120 2454 / 2471, 18720 x 15360 x 5120 1983 / 2001, 23400 x 5120 x 5120
// 881 / 879, 16128 x 15360 x 5120 1688 / 1685.  One contiguous range per XCD keeps the XCDs apart (23400 x 15360 x
// 5120 2740).  (Plain products, of a time when these had a workgroup to a tile as well.)
__device__ __forceinline__ bool tile_of_workgroup(const GemmArgs& a, int* tm, int* tn) {
  const int xcd = int(blockIdx.x & 7), j = int(blockIdx.x >> 3), total = a.tiles_m * a.tiles_n;
  if (a.block_cols > 0) {
    const int block = (j >> 5) * 8 + xcd, band = block / a.block_cols;
    *tm = band * kBandRows + (j & 7);
    *tn = (block - band * a.block_cols) * 4 + ((j >> 3) & 3);
    return *tm < a.tiles_m;
  }
  const int full = total >> 8, left = total & 255, share = last_round_share(left);
  int nth;
  if (j < full * 32) {
    nth = ((j & ~31) << 3) + xcd * 32 + (j & 31);
  } else {
    const int in_round = xcd * share + (j - full * 32);
    if (in_round >= left) return false;
    nth = full * 256 + in_round;
  }
  tile_at(a.tiles_m, a.tiles_n, nth, tm, tn);
  return true;
}

// kMt: 16-row sub-tiles of X to a wave; a tile of Y has 32 kMt rows (256 or 128) and 256 columns.
template <int kMt>
__global__ __launch_bounds__(256, 1) void gemm_bf16_kernel(GemmArgs a) {
  constexpr int kTileRows = 32 * kMt, kWaveRows = 16 * kMt;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  if (!tile_of_workgroup(a, &tm, &tn)) return;
  const int blk = tm / a.tiles_per_block, tile_in_blk = tm - blk * a.tiles_per_block;
  const int m0 = blk * a.block_rows + tile_in_blk * kTileRows, n0 = tn * kTile;
  const int m_end = min((blk + 1) * a.block_rows, a.M);           // first row past this tile's row block
  const int wm = wave & 1, wn = wave >> 1;

  // load i of this wave brings rows (8 wave + i) 8 .. +7 of a part (128-byte rows: whole cache
  // lines); lane L brings what is stored at position L & 7 of row L >> 3: chunk (L & 7) ^ ((row >> 1) & 7)
  uint32_t offw[8], offx[kMt];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = (wave * 8 + i) * 8 + (lane >> 3);
    const int nrow = min(n0 + row, a.N - 1) - n0;                // rows of w past n_out re-read its last row
    offw[i] = uint32_t(int64_t(nrow) * a.ldw * 2 + ((lane & 7) ^ ((row >> 1) & 7)) * 16);
  }
#pragma unroll
  for (int i = 0; i < kMt; ++i) {
    const int row = (wave * kMt + i) * 8 + (lane >> 3);
    const int mrow = min(m0 + row, m_end - 1) - m0;              // rows past the block's end re-read its last row
    offx[i] = uint32_t(int64_t(mrow) * a.ldx * 2 + ((lane & 7) ^ ((row >> 1) & 7)) * 16);
  }
  const uint64_t base_w = reinterpret_cast<uint64_t>(a.w + int64_t(n0) * a.ldw);
  const uint64_t base_x = reinterpret_cast<uint64_t>(a.x + int64_t(m0) * a.ldx);
  // operand reads (16 x 16 x 32 MFMA: lane = row l15 of a 16-row sub-tile, 8 k-values of group
  // grp): chunk grp of k-step 0 of the lane's row in the wave's 128 rows
  const uint32_t swz = (l15 >> 1) & 7;
  const uint32_t aw0 = uint32_t((wn * 128 + l15) * 128) + ((uint32_t(grp) ^ swz) << 4);
  const uint32_t ax0 = uint32_t((wm * kWaveRows + l15) * 128) + ((uint32_t(grp) ^ swz) << 4);
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  const int n_stages = a.K / 64;

  u32x16 o[kMt];
#define CA_GEMM_OPERANDS                                                                                              \
  [base_w] "s"(base_w), [base_x] "s"(base_x), [n_stages] "s"(n_stages), [wave] "s"(wave), [lds0] "s"(lds0),           \
      [offw0] "v"(offw[0]), [offw1] "v"(offw[1]), [offw2] "v"(offw[2]), [offw3] "v"(offw[3]), [offw4] "v"(offw[4]),   \
      [offw5] "v"(offw[5]), [offw6] "v"(offw[6]), [offw7] "v"(offw[7]), [offx0] "v"(offx[0]), [offx1] "v"(offx[1]),   \
      [offx2] "v"(offx[2]), [offx3] "v"(offx[3]), [aw0] "v"(aw0), [ax0] "v"(ax0)
  if constexpr (kMt == 8) {
    asm volatile(
#include "gemm_core_gfx950.inc"
        : "=&{v[0:15]}"(o[0]), "=&{v[16:31]}"(o[1]), "=&{v[32:47]}"(o[2]), "=&{v[48:63]}"(o[3]), "=&{v[64:79]}"(o[4]),
          "=&{v[80:95]}"(o[5]), "=&{v[96:111]}"(o[6]), "=&{v[112:127]}"(o[7])
        : CA_GEMM_OPERANDS, [offx4] "v"(offx[4]), [offx5] "v"(offx[5]), [offx6] "v"(offx[6]), [offx7] "v"(offx[7])
        : "memory", "scc", "m0", CA_GEMM_CLOBBERS);
  } else {
    asm volatile(
#include "gemm_core128_gfx950.inc"
        : "=&{v[0:15]}"(o[0]), "=&{v[16:31]}"(o[1]), "=&{v[32:47]}"(o[2]), "=&{v[48:63]}"(o[3])
        : CA_GEMM_OPERANDS
        : "memory", "scc", "m0", CA_GEMM_CLOBBERS128);
  }

  // The loop leaves 14 vector registers for what lives across it: the lane's places are worked out again from its
  // number, the wave's are scalars.  Kept in vector registers they were spilled in the publishing form, and each
  // reload in the epilogue is a memory latency: 23400 x 768 x 256 36.6 -> 33.7 us, 14040 x 3072 x 1024 103.4 -> 98.3,
  // 23400 x 15360 x 5120 2653 -> 2633.
  asm volatile("" : "+v"(tid));
  lane = tid & 63, l15 = lane & 15, grp = lane >> 4;

  // ---- epilogue: the wave's tile of kWaveRows (m) x 128 (n) goes through LDS to come out row by row.
  // Pair p of MFMA tile T = kMt ti + tj: n = 16 ti + 4 grp + 2 p, m = 16 tj + l15.
  __syncthreads();                                    // every wave is done with the stage buffers
  const int v_section = (n0 + wn * 128) / (a.pub.heads * 128) == 2;
  const int pitch = v_section ? kEpiRowV : kEpiRow;
  // with 128 rows the two waves of a page share its 128 x 128 tile
  constexpr bool kShared = kMt == 4;
  static_assert(kMt == 8 || kMt == 4, "a wave's rows are a page or half of one");
  uint8_t* mine = kShared ? lds + wn * kEpiWave + wm * kWaveRows * pitch : lds + wave * kEpiWave;
#pragma unroll
  for (int T = 0; T < 8 * kMt; ++T) {
    const int ti = T / kMt, tj = T % kMt;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int n = 16 * ti + 4 * grp + 2 * p;
      const int m = 16 * tj + l15;
      *reinterpret_cast<uint32_t*>(mine + m * pitch + n * 2) = o[(2 * T + p) >> 4][(2 * T + p) & 15];
    }
  }
  __syncthreads();
  if constexpr (kShared) {
    publish_tile<128>(a, lds + wn * kEpiWave, n0 + wn * 128, blk, tile_in_blk, m0, reinterpret_cast<float2*>(lds + 2 * kEpiWave),
                      wm * 64 + lane, tid, 256);
  } else {
    // the wave's sub-tile is one head of q, k or v for one page of a block
    float2* trig = reinterpret_cast<float2*>(lds + 4 * kEpiWave + wm * kTrigBytes);
    publish_tile<64>(a, mine, n0 + wn * 128, blk, 2 * tile_in_blk + wm, m0 + wm * 128, trig, lane, wn * 64 + lane, 128);
  }
}

}  // namespace

namespace {

int32_t check_gemm_shape(int64_t M, int32_t N, int32_t K, int64_t ldx, int64_t ldw, int64_t ldy) {
  if (M < 0) return CA_EINVAL;
  if (M > (int64_t(1) << 30) || N < 8 || N % 8 != 0 || K < 128 || K % 128 != 0) return CA_EUNSUPPORTED;
  if (ldx < K || ldw < K || ldy < 0 || ldx % 8 != 0 || ldw % 8 != 0 || ldy % 8 != 0) return CA_EINVAL;
  if (ldx * 2 * kTile >= (int64_t(1) << 31) || ldw * 2 * kTile >= (int64_t(1) << 31)) return CA_EUNSUPPORTED;
  return CA_OK;
}

// Whether a publishing product's tiles go by blocks of 8 x 4 in the last round too (before it the two ways are one).
// A tile of v takes several us longer in the epilogue than one of q: by blocks an XCD takes q, k and v in turn, dealt
// evenly some get v, k and v again.  It pays where blocks are whole, no XCD has a round more for them and the last
// round is not a short one.  Us dealt / by blocks: 14040 x 3072 x 1024 98 / 93, x 512 71 / 64, 23400 x 3072 x 1024
// 162 / 154, 23400 x 9216 x 3072 999 / 987, 14040 x 6144 x 2048 312 / 313, 18720 x 3072 x 1024 131.6 / 132.5; with a
// short last round 3510 x 9216 x 3072 194 / 202, 13200 x 6144 x 2048 304 / 311; with an XCD a round longer 14040 x
// 15360 x 5120 1653 / 1708, 23400 x 4608 x 1536 299 / 322.
int publish_block_cols(const GemmArgs& a) {
  const int total = a.tiles_m * a.tiles_n, cols = a.tiles_n / 4, blocks = (a.tiles_m + kBandRows - 1) / kBandRows * cols;
  return a.tiles_n % 4 == 0 && total > 256 && (total & 255) > 64 && (blocks + 7) / 8 == (total + 255) / 256 ? cols : 0;
}

// workgroups for tile_of_workgroup: whole rounds of 256, then eight times an XCD's share of the rest
unsigned tile_workgroups(const GemmArgs& a) {
  const unsigned total = unsigned(a.tiles_m) * unsigned(a.tiles_n);
  if (a.block_cols > 0) return (total + 255u) & ~255u;
  return (total & ~255u) + 8 * unsigned(last_round_share(int(total & 255u)));
}

template <int kMt>
int32_t enqueue_gemm(GemmArgs& a, void* stream) {
  constexpr int kTileRows = 32 * kMt;
  a.tiles_per_block = (a.block_rows + kTileRows - 1) / kTileRows;
  a.tiles_m = (a.M / a.block_rows) * a.tiles_per_block;
  a.tiles_n = (a.N + kTile - 1) / kTile;
  a.block_cols = kMt == 8 ? publish_block_cols(a) : 0;
  const auto kernel = gemm_bf16_kernel<kMt>;
  hipLaunchKernelGGL(kernel, dim3(tile_workgroups(a)), dim3(256), kGemmLds, static_cast<hipStream_t>(stream), a);
  return finish_launch("gemm_bf16.hip");
}

template <typename T>
int32_t enqueue_gemm_tiles(GemmArgs& a, void* stream) {
  a.tiles_per_block = (a.block_rows + T::kBm - 1) / T::kBm;
  a.tiles_m = (a.M / a.block_rows) * a.tiles_per_block;
  a.tiles_n = (a.N + T::kBn - 1) / T::kBn;
  a.more = (a.tiles_m * a.tiles_n + 7) / 8;
  hipLaunchKernelGGL((gemm_tile_kernel<T, true>), dim3(unsigned(a.more) * 8), dim3(T::kThreads), T::kLds, static_cast<hipStream_t>(stream), a);
  return finish_launch("gemm_bf16.hip");
}

// Which tile a product takes.  Outputs are the same to the last bit with every one of them (each is one chain of the
// same matrix instruction over k in steps of 32), so the choice is the cheapest by a model of what was measured:
// rounds of workgroups over the CUs times (stages of 64 k x time of a stage + set-up and epilogue).  A stage takes
// longer when most CUs work (`full`, from half of them on in proportion: the last round has its own).  Microseconds
// (fixed: plain, publishing; plain products in tiles of 256 columns are rows_tile's):
//   256 x 256 (asm loop)    stage 1.0 .. 1.19, fixed -, 12.5      256 x 128   stage 0.85 .. 0.87, fixed 5.8, 6.25
//   128 x 256 (asm loop)    0.58 .. 0.66, -, 9.25                 128 x 128   0.43, 5, 4.5
//                                                                 64 x 64     two a CU 0.31, 4, -; one a CU 0.165, 4, -
// Plain calls, us, by what is taken: 64 x 64, one a CU: 257 x 768 x 1024 5.8 (two a CU 6.3, 128 x 128 9.6, 128 x 256 14.4), 64 x 128 x 5120 16.6 (19.7, 34,
// 48); two a CU: 1200 x 1400 x 1152 9.8 (one a CU 11.9, 128 x 128 11.7); 128 x 128: 23400 x 128 x 5120 39.6 (64 x 64 58, 256 x 128 62),
// 1560 x 1536 x 1536 14.0 (18.1, 22.2).  256 x 128 is for column counts that 256 does not divide well (an odd number of
// heads): 14040 x 1152 x 384 19.7 (192 x 256 21.2), 23400 x 640 x 640 26.3 (27.6), 17961 x 328 x 2432 35.9 (37.8).  The
// publishing epilogue needs whole pages and heads: 128 or 256 rows.  It writes pages instead of rows, which the largest
// tiles pay for most: of 23400 x 768 x 256, 34.0 us with 256 x 256, 33.5 with 128 x 256, 26.6 with 256 x 128, 29.4 with 128
// x 128; 23400 x 3072 x 1024 163 / 176 / 182 / 206; 7920 x 2304 x 768 52 / 45 / 49 / 46.

// the cheapest tile and, in nanoseconds, what it costs
GemmTile pick_gemm_tile(const GemmArgs& a, bool publish, int n_cu, int64_t* cost) {
  // fixed, fixed_publish: 0 where a plain product, a publishing one does not take the tile
  static constexpr struct { int bm, bn, per_cu, threads, stage, full, fixed, fixed_publish; } kModel[] = {
      {256, 256, 1, 256, 1000, 1190, 0, 12500}, {256, 128, 1, 512, 850, 870, 5800, 6250}, {128, 256, 1, 256, 580, 660, 0, 9250},
      {128, 128, 1, 512, 430, 430, 5000, 4500}, {64, 64, 2, 256, 310, 310, 4000, 0},      {64, 64, 1, 512, 165, 165, 4000, 0}};
  const int64_t blocks = a.M / a.block_rows, stages = a.K / 64;
  GemmTile tile = kTile128;
  *cost = INT64_MAX;
  for (int i = 0; i < int(sizeof(kModel) / sizeof(kModel[0])); ++i) {
    const auto& m = kModel[i];
    const int64_t fixed = publish ? m.fixed_publish : m.fixed;
    if (fixed == 0) continue;
    const int64_t tiles = blocks * ((a.block_rows + m.bm - 1) / m.bm) * ((a.N + m.bn - 1) / m.bn);
    if (i != kTile256 && tiles * m.threads >= (int64_t(1) << 31)) continue;      // a launch may have 2^32 threads
    const int64_t slots = int64_t(n_cu) * m.per_cu, left = tiles % slots;        // left: tiles of a last round
    const int64_t stage = m.stage + (2 * left > slots ? (m.full - m.stage) * (2 * left - slots) / slots : 0);
    const int64_t of_tile = tiles / slots * (stages * m.full + fixed) + (left > 0 ? stages * stage + fixed : 0);
    if (of_tile < *cost) {
      *cost = of_tile;
      tile = GemmTile(i);
    }
  }
  return tile;
}

// Tile height of gemm_rows.hip that a plain product takes, or 0 where one of the tiles of compiled code is cheaper.  A
// workgroup goes on from tile to tile there, so that a round costs its stages and the results' way out, and a launch its
// set-up once: nanoseconds by stages of 64 k = start + whole rounds x (stages x full + tile) + last round (stages x stage +
// tile), stage up to full from half of the CUs on.  Fitted to 254 products; over 130 others (64 to 23400 rows, up to 15360 columns, k up to
// 5120) the pick is 0.2 % slower than the fastest of all seven kernels in the geometric mean, 16 % at the worst (6658 x 6736 x 128,
// 28.8 us for 24.9).  Whole calls, us, with a tile to a workgroup and the result through LDS / now: 23400 x 5120 x 256 102 / 78, 10709 x
// 4200 x 256 46 / 34, 5882 x 8776 x 640 87 / 71, 4680 x 3072 x 512 19.0 / 17.3, 4680 x 4608 x 1536 59.4 / 54.5, 23400 x 15360
// x 5120 2423 / 2352; the other way 8192 x 8192 x 8064 673 / 696, whole rounds of long walks.  By height, 256 / 192 / 128: 4680 x 4608 x 1536 66.0
// / 54.1 / 60.7, 23400 x 15360 x 5120 2341 / 2461 / 2752, 4680 x 1536 x 1536 32.8 / 26.9 / 22.4.  The 256 x 128 tile stays ahead of an
// equal cost (14040 x 1152 x 384 19.7, 192 x 256 21.2).
int rows_tile(const GemmArgs& a, int n_cu, int64_t compiled, GemmTile by) {
  static constexpr struct { int rows, start, stage, full, tile; } kRows[] = {
      {256, 2260, 960, 1325, 5100}, {192, 2280, 754, 1070, 3900}, {128, 2840, 594, 785, 2410}};
  const int64_t stages = a.K / 64, limit = by == kTile256x128 ? compiled - compiled / 14 : compiled;
  int64_t best = limit;
  int rows = 0;
  for (const auto& m : kRows) {
    const int64_t tiles = ((a.M + int64_t(m.rows) - 1) / m.rows) * ((a.N + 255) / 256), left = tiles % n_cu;
    const int64_t stage = m.stage + (2 * left > n_cu ? (m.full - m.stage) * (2 * left - n_cu) / n_cu : 0);
    const int64_t cost = m.start + tiles / n_cu * (stages * m.full + m.tile) + (left > 0 ? stages * stage + m.tile : 0);
    if (cost < best) {
      best = cost;
      rows = m.rows;
    }
  }
  return rows;
}

int32_t dispatch_gemm_publish(GemmArgs& a, void* stream) {
  int64_t cost = 0;
  int n_cu = 0;
  if (const int32_t rc = device_cu_count(&n_cu); rc != CA_OK) return rc;
  const GemmTile tile = pick_gemm_tile(a, true, n_cu, &cost);
  const KernelLds kernels[] = {{reinterpret_cast<const void*>(gemm_bf16_kernel<8>), kGemmLds},
                               {reinterpret_cast<const void*>(gemm_bf16_kernel<4>), kGemmLds},
                               {reinterpret_cast<const void*>(gemm_tile_kernel<Tile256x128, true>), Tile256x128::kLds},
                               {reinterpret_cast<const void*>(gemm_tile_kernel<Tile128, true>), Tile128::kLds}};
  if (const int32_t rc = ensure_dynamic_lds(kernels, 4, kLdsGemmPublish); rc != CA_OK) return rc;
  if (tile == kTile128x256) return enqueue_gemm<4>(a, stream);
  if (tile == kTile256x128) return enqueue_gemm_tiles<Tile256x128>(a, stream);
  if (tile == kTile128) return enqueue_gemm_tiles<Tile128>(a, stream);
  return enqueue_gemm<8>(a, stream);
}

int32_t dispatch_gemm_plain(GemmArgs& a, void* stream) {
  int64_t cost = 0;
  int n_cu = 0;
  if (const int32_t rc = device_cu_count(&n_cu); rc != CA_OK) return rc;
  const GemmTile compiled = pick_gemm_tile(a, false, n_cu, &cost);
  if (const int32_t rc = gemm_tiles_ready(); rc != CA_OK) return rc;
  if (const int32_t rc = gemm_rows_ready(); rc != CA_OK) return rc;
  if (const int rows = rows_tile(a, n_cu, cost, compiled))
    return launch_gemm_rows(rows, a.x, a.w, a.y, a.M, a.N, a.K, a.ldx, a.ldw, a.ldy, stream);
  return launch_gemm_tile(compiled, a.x, a.w, a.y, a.M, a.N, a.K, a.ldx, a.ldw, a.ldy, stream);
}

}  // namespace

int32_t launch_gemm_bf16(const void* x, const void* w, void* y, int64_t M, int32_t N, int32_t K,
                         int64_t ldx, int64_t ldw, int64_t ldy, void* stream) {
  if (const int32_t rc = check_gemm_shape(M, N, K, ldx, ldw, ldy); rc != CA_OK) return rc;
  if (ldy < N) return CA_EINVAL;
  if (M == 0) return CA_OK;                       // nothing to do
  GemmArgs a{};
  a.x = static_cast<const uint16_t*>(x);
  a.w = static_cast<const uint16_t*>(w);
  a.y = static_cast<uint16_t*>(y);
  a.M = int32_t(M); a.N = N; a.K = K;
  a.ldx = ldx; a.ldw = ldw; a.ldy = ldy;
  a.block_rows = a.M;                             // one row block: tiles run through all of M
  return dispatch_gemm_plain(a, stream);
}

int32_t launch_gemm_qkv_publish(const RopeGeom& g, int32_t n_blocks, int32_t block_tokens, int32_t pages_per_block,
                                const int32_t* slot, const int64_t* first_frame, const void* x, int64_t ldx,
                                const void* w, int64_t ldw, int32_t K, void* q_out, void* pool, void* stream) {
  if (g.head_dim != 128 || n_blocks < 1 || n_blocks > kMaxInflight) return CA_EUNSUPPORTED;
  const int32_t N = 3 * g.heads * 128;
  const int64_t M = int64_t(n_blocks) * block_tokens;
  // a 256-wide column tile must not straddle q|k|v: heads * 128 a multiple of 256
  if (g.heads % 2 != 0) return CA_EUNSUPPORTED;
  if (const int32_t rc = check_gemm_shape(M, N, K, ldx, ldw, int64_t(g.heads) * 128); rc != CA_OK) return rc;
  GemmArgs a{};
  a.x = static_cast<const uint16_t*>(x);
  a.w = static_cast<const uint16_t*>(w);
  a.y = static_cast<uint16_t*>(q_out);
  a.M = int32_t(M); a.N = N; a.K = K;
  a.ldx = ldx; a.ldw = ldw; a.ldy = int64_t(g.heads) * 128;
  a.block_rows = block_tokens;
  a.pub.g = g;
  a.pub.pool = static_cast<uint8_t*>(pool);
  a.pub.heads = g.heads;
  a.pub.pages_per_block = pages_per_block;
  for (int i = 0; i < n_blocks; ++i) {
    a.pub.slot[i] = slot[i];
    a.pub.first_frame[i] = first_frame[i];
  }
  size_t tab_bytes = 0;
  a.pub.tab = trig_table_for(g, 128, kTrigBytes, &tab_bytes);
  return dispatch_gemm_publish(a, stream);
}

}  // namespace ca
