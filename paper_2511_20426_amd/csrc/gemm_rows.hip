// Y[M,N] = X[M,K] . W[N,K]^T in bf16 with fp32 accumulation, for products that fill the chip with tiles of 256 columns
// (launch_gemm_bf16 picks).  A workgroup of 4 waves, one per SIMD, takes one tile of 256, 192 or 128 rows after the other: the
// loop over stages and tiles, the results' way to memory included, is the assembly emitted by gen_gemm_rows.py, which
// documents the pipeline and the register map.  This file holds the set-up and the launch.
#include <hip/hip_runtime.h>

#include "ca_internal.hpp"

namespace ca {
namespace {

#include "gemm_tiles.hpp"
#include "gemm_rows_clobbers.inc"

constexpr int kTileCols = 256;
constexpr int kRowsLds = 160 * 1024;              // 3 stages of W, 2 of X
constexpr int kFormThrough = 1, kFormPast = 2;    // results written through L2, past the caches; 0: left in L2
constexpr int kList = 64;                         // tiles of a workgroup: one to a lane

// kMt: 16-row sub-tiles of X to a wave; a tile of Y has 32 kMt rows and 256 columns.
// Tiles are numbered down bands of eight row tiles and dealt to the XCDs (workgroup b runs on b % 8) 32 at a time, what is
// left for the last round by last_round_share; tile i of workgroup b of a group of 256 is the one that workgroup 256 i + b
// would have if each took one.
template <int kMt>
__global__ __launch_bounds__(256, 1) void gemm_rows_kernel(LinearArgs a) {
  constexpr int kTileRows = 32 * kMt, kWaveRows = 16 * kMt;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  // ---- this workgroup's tiles, one to a lane
  const int xcd = int(blockIdx.x & 7), j = int(blockIdx.x >> 3) & 31, first = int(blockIdx.x >> 8) * kList;
  const int total = a.tiles_m * a.tiles_n, full = total >> 8, left = total & 255, share = last_round_share(left);
  const int mine = full + (j < share && xcd * share + j < left ? 1 : 0);
  const int tiles = min(mine - first, kList);
  if (tiles <= 0) return;
  const int r = min(first + lane, mine - 1);
  int list_m, list_n;
  tile_at(a.tiles_m, a.tiles_n, r < full ? r * 256 + xcd * 32 + j : full * 256 + xcd * share + j, &list_m, &list_n);

  // ---- the lane's part in loads: load i of a wave brings rows (8 wave + i) 8 .. +7 of W, (kMt wave + i) 8 .. of X, 128 bytes of each
  const int roww = wave * 64 + (lane >> 3), rowx = wave * 8 * kMt + (lane >> 3);
  const int chunkw = ((lane & 7) ^ ((lane >> 4) & 1)) * 16, chunkx = ((lane & 7) ^ (lane >> 4)) * 16;
  // ... in operand reads (lane = row l15 of a sub-tile, 8 k-values of group grp) ...
  const int aw0 = (wn * 128 + 8 * (l15 >> 2) + (l15 & 3)) * 128 + ((grp ^ (l15 >> 1)) << 4);
  const int ax0 = (wm * kWaveRows + l15) * 128 + ((grp ^ (l15 >> 1)) << 4);
  // ... and of the results: of the first eight rows of sub-tile 0 row l15 % 8, columns 32 (l15 / 8) + 8 grp ..
  const int row = wm * kWaveRows + (l15 & 7), col = wn * 128 + 32 * (l15 >> 3) + 8 * grp;
  const uint64_t ylane = uint64_t(row) * uint64_t(a.ldy) * 2 + uint64_t(col) * 2;
  const uint64_t x = reinterpret_cast<uint64_t>(a.x), w = reinterpret_cast<uint64_t>(a.w), y = reinterpret_cast<uint64_t>(a.y);
  const uint64_t tile_y = uint64_t(a.ldy) * 2 * kTileRows, row8 = uint64_t(a.ldy) * 2 * 8;
  const uint32_t ldw2 = uint32_t(a.ldw) * 2, ldx2 = uint32_t(a.ldx) * 2;        // below 2^23 (check_gemm_shape)
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
#define CA_GEMM_ROWS_OPERANDS                                                                                          \
  [x_lo] "s"(uint32_t(x)), [x_hi] "s"(uint32_t(x >> 32)), [w_lo] "s"(uint32_t(w)), [w_hi] "s"(uint32_t(w >> 32)),      \
      [y_lo] "s"(uint32_t(y)), [y_hi] "s"(uint32_t(y >> 32)), [tile_x] "s"(ldx2 * kTileRows),                          \
      [tile_w] "s"(ldw2 * kTileCols), [tile_y_lo] "s"(uint32_t(tile_y)), [tile_y_hi] "s"(uint32_t(tile_y >> 32)),      \
      [row8_lo] "s"(uint32_t(row8)), [row8_hi] "s"(uint32_t(row8 >> 32)), [ldw2] "s"(ldw2), [ldx2] "s"(ldx2),      \
      [M] "s"(a.M), [N] "s"(a.N), [n_stages] "s"(a.K / 64), [tiles] "s"(tiles), [form] "s"(a.more), [wave] "s"(wave), [lds0] "s"(lds0),    \
      [list_m] "v"(list_m), [list_n] "v"(list_n), [roww] "v"(roww), [rowx] "v"(rowx), [chunkw] "v"(chunkw),            \
      [chunkx] "v"(chunkx), [aw0] "v"(aw0), [ax0] "v"(ax0), [row] "v"(row), [col] "v"(col),                            \
      [ylane_lo] "v"(uint32_t(ylane)), [ylane_hi] "v"(uint32_t(ylane >> 32))
  if constexpr (kMt == 8) {
    asm volatile(
#include "gemm_rows256_gfx950.inc"
        :: CA_GEMM_ROWS_OPERANDS : "memory", "vcc", "scc", "m0", CA_GEMM_ROWS_CLOBBERS256);
  } else if constexpr (kMt == 6) {
    asm volatile(
#include "gemm_rows192_gfx950.inc"
        :: CA_GEMM_ROWS_OPERANDS : "memory", "vcc", "scc", "m0", CA_GEMM_ROWS_CLOBBERS192);
  } else {
    asm volatile(
#include "gemm_rows128_gfx950.inc"
        :: CA_GEMM_ROWS_OPERANDS : "memory", "vcc", "scc", "m0", CA_GEMM_ROWS_CLOBBERS128);
  }
}

template <int kMt>
int32_t enqueue_gemm_rows(LinearArgs& a, void* stream) {
  a.tiles_m = (a.M + 32 * kMt - 1) / (32 * kMt);
  a.tiles_n = (a.N + kTileCols - 1) / kTileCols;
  const int64_t total = int64_t(a.tiles_m) * a.tiles_n, rounds = (total + 255) / 256;
  const unsigned workgroups = total < 256 ? 8 * unsigned(last_round_share(int(total))) : 256 * unsigned((rounds + kList - 1) / kList);
  // How results leave.  Rows of whole lines (128 bytes) go past the caches, those of a workgroup's last tile, which the end of the
  // launch waits for, through L2.  Rows that share lines stay in L2, which merges the pieces; what it then still holds at the end of
  // the launch, up to 32 MB, is less than half a round where there is one round only, and is written through there.  Us, left in L2 /
  // last tile through / all through / past the caches and the last through: 14040 x 15360 x 256 138.6 / 137.0 / 134.9 / 130.7,
  // 23400 x 5120 x 1536 283.8 / 282.4 / 286.7 / 276.1, 4680 x 3072 x 256 (one round) 15.1 / 12.5 / 12.5 / 12.5; rows that share lines:
  // 23400 x 5128 x 256 78.1 / 81.2 / 117.4 / 111.1, 23400 x 5128 x 1536 281.1 / 286.1 / 317.5 / 286.0, one round 2340 x 4616 x 512
  // 16.0 / 15.5 / 15.4 / 15.5, 4680 x 3080 x 512 19.4 / 19.5 / 19.5 / 19.5.
  const bool whole_lines = a.ldy % 64 == 0 && reinterpret_cast<uintptr_t>(a.y) % 128 == 0;
  a.more = whole_lines ? kFormPast | kFormThrough << 2 : (rounds <= 1 ? kFormThrough << 2 : 0);
  const auto kernel = gemm_rows_kernel<kMt>;
  hipLaunchKernelGGL(kernel, dim3(workgroups), dim3(256), kRowsLds, static_cast<hipStream_t>(stream), a);
  return finish_launch("gemm_rows.hip");
}

}  // namespace

int32_t gemm_rows_ready() {
  const KernelLds kernels[] = {{reinterpret_cast<const void*>(gemm_rows_kernel<8>), kRowsLds},
                               {reinterpret_cast<const void*>(gemm_rows_kernel<6>), kRowsLds},
                               {reinterpret_cast<const void*>(gemm_rows_kernel<4>), kRowsLds}};
  return ensure_dynamic_lds(kernels, 3, kLdsGemmRows);
}

int32_t launch_gemm_rows(int tile_rows, const void* x, const void* w, void* y, int32_t M, int32_t N, int32_t K,
                         int64_t ldx, int64_t ldw, int64_t ldy, void* stream) {
  LinearArgs a{};
  a.x = static_cast<const uint16_t*>(x);
  a.w = static_cast<const uint16_t*>(w);
  a.y = static_cast<uint16_t*>(y);
  a.M = M; a.N = N; a.K = K;
  a.ldx = int32_t(ldx); a.ldw = int32_t(ldw); a.ldy = ldy;          // (below 2^22: check_gemm_shape)
  if (tile_rows == 256) return enqueue_gemm_rows<8>(a, stream);
  if (tile_rows == 192) return enqueue_gemm_rows<6>(a, stream);
  return enqueue_gemm_rows<4>(a, stream);
}

}  // namespace ca
