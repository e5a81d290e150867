// The compiled tiles of the linear maps and their kernel: gemm_tiles.hip has the plain products, gemm_bf16.hip the publishing
// projection.  (Included inside namespace ca { namespace { ... } }, behind rope_device.hpp and gemm_tiles.hpp.)
#pragma once

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kEpiRow = 272;                      // bytes per row of a wave's 128 x 128 bf16 tile in LDS
constexpr int kEpiRowV = 260;                     // the same for a V sub-tile of the publishing epilogue, which is read
                                                  // back two bytes at a time down its columns: 65 dwords per row spread
                                                  // the 16 token groups a wave reads at once over 16 banks
constexpr int kTrigBytes = 12288;                 // per 128-token page; two pages per workgroup behind the staging area
constexpr int kGemmLds = 160 * 1024;

// Smaller tiles, for products whose 256 x 256 tiles would leave CUs idle: K walked in the same stages of 64, through
// a ring of kStages in LDS filled by global -> LDS loads, kWavesM x kWavesN waves of 16 x 16 tiles, operands read one
// k-step ahead.  What bounds them: LDS reads and fills (128 x 128 in eight waves: 128 KB a stage = 1024 cycles, 1000
// measured, for 512 of the matrix pipe), at 64 x 64 with few workgroups the latency of a stage; that is why the
// smallest takes eight waves and six stages.
template <int BM, int BN, int kWavesM, int kWavesN, int kStages>
struct TileShape {
  static constexpr int kBm = BM, kBn = BN, kWavesAlongM = kWavesM, kRing = kStages;
  static constexpr int kWaves = kWavesM * kWavesN, kThreads = 64 * kWaves;
  static constexpr int kTm = BM / kWavesM / 16, kTn = BN / kWavesN / 16;   // 16 x 16 tiles of a wave
  static constexpr int kStageBytes = (BM + BN) * 128;
  static constexpr int kLoadsW = BN / 8 / kWaves, kLoadsX = BM / 8 / kWaves;   // 1 KB loads of a wave per stage
  static constexpr int kPitch = BN * 2 + 16;
  static constexpr int kEpi = BM * kPitch + (BN == 128 ? BM / 128 * kTrigBytes : 0);
  static constexpr int kLds = kStages * kStageBytes > kEpi ? kStages * kStageBytes : kEpi;
  static_assert(kLoadsW * 8 * kWaves == BN && kLoadsX * 8 * kWaves == BM && kLds <= kGemmLds, "shape");
};

using Tile256x128 = TileShape<256, 128, 4, 2, 3>;
using Tile128 = TileShape<128, 128, 2, 4, 4>;
using Tile64 = TileShape<64, 64, 2, 2, 4>;
using Tile64Wide = TileShape<64, 64, 2, 4, 6>;

// the publishing projection's are GemmArgs
template <bool kPublish>
struct TileArgsOf {
  using type = LinearArgs;
};

template <int kThreads, typename Args>
__device__ void publish_tile(const Args& a, const uint8_t* tile, int col, int blk, int page, int m0, float2* trig, int t, int fill_t, int fill_n);

template <typename T, bool kPublish>
__global__ __launch_bounds__(T::kThreads) void gemm_tile_kernel(typename TileArgsOf<kPublish>::type a) {
  constexpr int BM = T::kBm, BN = T::kBn, kWavesM = T::kWavesAlongM, kStages = T::kRing;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l15 = lane & 15, grp = lane >> 4;
  const int wm = wave % kWavesM, wn = wave / kWavesM;
  // XCD x takes a contiguous range of the tiles.  Dealing them as gemm_rows_kernel does costs a short kernel its longer
  // set-up: 220 x 2696 x 3072 12.0 us, 12.7 dealt; 2868 x 992 x 512 7.5, 7.6.
  const int nth = int(blockIdx.x & 7) * a.more + int(blockIdx.x >> 3);
  if (nth >= a.tiles_m * a.tiles_n) return;
  int tm, tn;
  tile_at(a.tiles_m, a.tiles_n, nth, &tm, &tn);
  int blk = 0, tile_in_blk = tm, m0 = tm * BM, m_end = a.M;
  if constexpr (kPublish) {
    blk = tm / a.tiles_per_block, tile_in_blk = tm - blk * a.tiles_per_block;
    m0 = blk * a.block_rows + tile_in_blk * BM, m_end = min((blk + 1) * a.block_rows, a.M);
  }
  const int n0 = tn * BN;

  // as in gemm_bf16_kernel: load i of a wave brings 8 whole 128-byte rows, chunks swizzled by the row
  uint32_t offw[T::kLoadsW], offx[T::kLoadsX];
#pragma unroll
  for (int i = 0; i < T::kLoadsW; ++i) {
    const int row = (wave * T::kLoadsW + i) * 8 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
    offw[i] = uint32_t(int64_t(min(n0 + row, a.N - 1) - n0) * a.ldw * 2 + c * 16);
  }
#pragma unroll
  for (int i = 0; i < T::kLoadsX; ++i) {
    const int row = (wave * T::kLoadsX + i) * 8 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
    offx[i] = uint32_t(int64_t(min(m0 + row, m_end - 1) - m0) * a.ldx * 2 + c * 16);
  }
  uint64_t base_w = reinterpret_cast<uint64_t>(a.w + int64_t(n0) * a.ldw);
  uint64_t base_x = reinterpret_cast<uint64_t>(a.x + int64_t(m0) * a.ldx);
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  const int n_stages = a.K / 64;
  int issued = 0;
  uint32_t fill = lds0;                       // ring slot the next stage goes to
  auto issue = [&]() {
#pragma unroll
    for (int i = 0; i < T::kLoadsW; ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :: "s"(fill + (wave * T::kLoadsW + i) * 1024), "v"(offw[i]), "s"(base_w) : "memory", "m0");
#pragma unroll
    for (int i = 0; i < T::kLoadsX; ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :: "s"(fill + BN * 128 + (wave * T::kLoadsX + i) * 1024), "v"(offx[i]), "s"(base_x) : "memory", "m0");
    // past the last stage the loads repeat it, into slots nothing reads any more: the wait counts stay exact
    ++issued;
    base_w += issued < n_stages ? 128 : 0;
    base_x += issued < n_stages ? 128 : 0;
    fill += T::kStageBytes;
    fill = fill == lds0 + kStages * T::kStageBytes ? lds0 : fill;
  };
  const uint32_t swz = (l15 >> 1) & 7;
  const uint32_t aw0 = uint32_t((wn * T::kTn * 16 + l15) * 128) + ((uint32_t(grp) ^ swz) << 4);
  const uint32_t ax0 = uint32_t(BN * 128 + (wm * T::kTm * 16 + l15) * 128) + ((uint32_t(grp) ^ swz) << 4);

  f32x4 acc[T::kTn][T::kTm];
#pragma unroll
  for (int i = 0; i < T::kTn; ++i)
#pragma unroll
    for (int j = 0; j < T::kTm; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 fw[2][T::kTn], fx[2][T::kTm];
  uint32_t slot = 0;
  auto read = [&](int kk) {
#pragma unroll
    for (int i = 0; i < T::kTn; ++i) fw[kk][i] = *reinterpret_cast<const bf16x8*>(lds + slot + (aw0 ^ (kk << 6)) + i * 2048);
#pragma unroll
    for (int j = 0; j < T::kTm; ++j) fx[kk][j] = *reinterpret_cast<const bf16x8*>(lds + slot + (ax0 ^ (kk << 6)) + j * 2048);
    __builtin_amdgcn_sched_barrier(0);        // reads stay ahead of the products they run beside
  };
  auto multiply = [&](int kk) {
#pragma unroll
    for (int i = 0; i < T::kTn; ++i)
#pragma unroll
      for (int j = 0; j < T::kTm; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[kk][i], fx[kk][j], acc[i][j], 0, 0, 0);
  };
#pragma unroll
  for (int s = 0; s < kStages; ++s) issue();
  constexpr int kFlying = (kStages - 1) * (T::kLoadsW + T::kLoadsX);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(kFlying) : "memory");
  read(0);
  // operands are read one k-step ahead of their products, across stages too: the barrier stands before a
  // stage's second k-step
  for (int s = 0; s < n_stages; ++s) {
    read(1);
    multiply(0);
    __builtin_amdgcn_sched_barrier(0);
    // the next stage has landed; every wave has this one in registers: its slot takes the next loads
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(kFlying - T::kLoadsW - T::kLoadsX) : "memory");
    issue();
    slot += T::kStageBytes;
    slot = slot == kStages * T::kStageBytes ? 0 : slot;
    read(0);
    multiply(1);
    __builtin_amdgcn_sched_barrier(0);
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");     // the ring is free

  int pitch = T::kPitch;
  if constexpr (kPublish) pitch = n0 / (a.pub.heads * 128) == 2 ? kEpiRowV : kEpiRow;
#pragma unroll
  for (int i = 0; i < T::kTn; ++i)
#pragma unroll
    for (int j = 0; j < T::kTm; ++j) {
      uint32_t* to = reinterpret_cast<uint32_t*>(lds + ((wm * T::kTm + j) * 16 + l15) * pitch +
                                                 ((wn * T::kTn + i) * 16 + 4 * grp) * 2);
      to[0] = pack_bf16(acc[i][j][0], acc[i][j][1]);
      to[1] = pack_bf16(acc[i][j][2], acc[i][j][3]);
    }
  __syncthreads();
  if constexpr (kPublish) {
    constexpr int kPages = BM / 128, kShare = T::kThreads / kPages;      // threads of a page
    const int part = wave / (kShare / 64), t = tid % kShare;
    publish_tile<kShare>(a, lds + part * 128 * pitch, n0, blk, kPages * tile_in_blk + part, m0 + part * 128,
                         reinterpret_cast<float2*>(lds + BM * kEpiRow + part * kTrigBytes), t, t, kShare);
    return;
  }
  constexpr int kChunks = BN / 8, kRows = T::kThreads / kChunks;
  const int c = tid % kChunks;
#pragma unroll 4
  for (int row = tid / kChunks; row < BM; row += kRows) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(lds + row * T::kPitch + c * 16);
    if (m0 + row < m_end && n0 + c * 8 < a.N)
      __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(a.y + int64_t(m0 + row) * a.ldy + n0 + c * 8));
  }
}
