// Y[M,N] = X[M,K] . W[N,K]^T in bf16 with fp32 accumulation, for products that a tile of up to 128 columns is for (launch_gemm_bf16
// picks): the launch of gemm_tile_kernel.hpp's kernel.
// This file is compiled with its loops at multiples of 64 bytes (_build.py); the publishing kernels, which have many
// loops beside the main one, are not, for there it costs 1 % (60 projections: 0.995 in the geometric mean, 1.005 without).
#include <hip/hip_runtime.h>

#include "ca_internal.hpp"

namespace ca {
namespace {

#include "rope_device.hpp"
#include "gemm_tiles.hpp"
#include "gemm_tile_kernel.hpp"

template <typename T>
int32_t enqueue_gemm_tile(LinearArgs& a, void* stream) {
  a.tiles_m = (a.M + T::kBm - 1) / T::kBm;
  a.tiles_n = (a.N + T::kBn - 1) / T::kBn;
  a.more = (a.tiles_m * a.tiles_n + 7) / 8;
  hipLaunchKernelGGL((gemm_tile_kernel<T, false>), dim3(unsigned(a.more) * 8), dim3(T::kThreads), T::kLds, static_cast<hipStream_t>(stream), a);
  return finish_launch("gemm_tiles.hip");
}

}  // namespace

int32_t gemm_tiles_ready() {
  const KernelLds kernels[] = {{reinterpret_cast<const void*>(gemm_tile_kernel<Tile256x128, false>), Tile256x128::kLds},
                               {reinterpret_cast<const void*>(gemm_tile_kernel<Tile128, false>), Tile128::kLds},
                               {reinterpret_cast<const void*>(gemm_tile_kernel<Tile64, false>), Tile64::kLds},
                               {reinterpret_cast<const void*>(gemm_tile_kernel<Tile64Wide, false>), Tile64Wide::kLds}};
  return ensure_dynamic_lds(kernels, 4, kLdsGemm);
}

int32_t launch_gemm_tile(int tile, const void* x, const void* w, void* y, int32_t M, int32_t N, int32_t K,
                         int64_t ldx, int64_t ldw, int64_t ldy, void* stream) {
  LinearArgs a{static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w), static_cast<uint16_t*>(y), ldy, M, N, K,
               int32_t(ldx), int32_t(ldw), 0, 0, 0};                // (below 2^22: check_gemm_shape)
  if (tile == kTile64) return enqueue_gemm_tile<Tile64>(a, stream);
  if (tile == kTile64Wide) return enqueue_gemm_tile<Tile64Wide>(a, stream);
  if (tile == kTile256x128) return enqueue_gemm_tile<Tile256x128>(a, stream);
  return enqueue_gemm_tile<Tile128>(a, stream);
}

}  // namespace ca
