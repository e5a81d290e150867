// The arguments of a plain linear map, and how its tiles are numbered and dealt to the XCDs, shared by its kernels.
// (Included inside namespace ca { namespace { ... } }.)
#pragma once

enum GemmTile { kTile256, kTile256x128, kTile128x256, kTile128, kTile64, kTile64Wide };

constexpr int kBandRows = 8;                      // row tiles of a band

// 64 bytes, because a launch with more takes the host longer: 2.6 us with up to 64 bytes of arguments, 3.3 with 128 to 256, 3.7
// with 384 to 1024 (small products are bound by it: 257 x 768 x 1024 5.82 -> 5.56 us a call).
struct LinearArgs {
  const uint16_t* x;
  const uint16_t* w;
  uint16_t* y;
  int64_t ldy;                                    // row strides in elements
  int32_t M, N, K, ldx, ldw;
  int32_t tiles_m, tiles_n;
  int32_t more;                                   // gemm_rows_kernel: how results are written; gemm_tile_kernel: tiles of an XCD
};
static_assert(sizeof(LinearArgs) == 64, "one cache line");

// Tiles are numbered down bands of eight row tiles.
__device__ __forceinline__ void tile_at(int tiles_m, int tiles_n, int nth, int* tm, int* tn) {
  const int band = nth / (kBandRows * tiles_n), in_band = nth - band * kBandRows * tiles_n;
  const int height = min(kBandRows, tiles_m - band * kBandRows);
  *tn = in_band / height;
  *tm = band * kBandRows + in_band - *tn * height;
}

// Tiles that an XCD takes in the last round of `left`.  Up to 64 go 16 to an XCD: with a few each, the tiles of an
// XCD have hardly a slab in common.  Us dealt evenly / 16 to an XCD, 256 x 256 tiles of x 5120 x 5120 by whole rounds
// and tiles left: 7 + 8 882 / 857, 7 + 28 891 / 874, 7 + 48 908 / 883, 4 + 16 513 / 508, 3 + 12 407 / 406, 6 + 44 724
// / 724, 6 + 24 the other way 731 / 743; with K 1536 4 + 2 179.3 / 177.1, 5 + 16 217.0 / 214.5.  More than 64 go
// evenly: 16 to an XCD gives little and not always, 6 + 84 750 / 750, 7 + 68 900 / 894, 7 + 108 923 / 913, 3 + 72 407
// / 407, 32 to an XCD 3 + 72 425, 5 + 80 622 / 635.
__host__ __device__ constexpr int last_round_share(int left) { return left > 0 && left <= 64 ? 16 : (left + 7) >> 3; }
