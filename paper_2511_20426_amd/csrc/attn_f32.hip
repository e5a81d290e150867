// fp32 block-cascaded attention for the small fp32 configurations (head_dim 32/64/128, pages of any
// size): the exact path one checks a model with.  All arithmetic is fp32; the two products run on
// the fp32 matrix instruction v_mfma_f32_16x16x4_f32 (fused multiply-adds, fp32 accumulation).
//
// What bounds it: at the sizes it serves (10^2..10^4 keys, a few heads) the length of one wave's
// serial chain, then the fp32 matrix rate (256 flop/clk per CU).  So a workgroup takes only 16 query
// rows of one head, and its waves share the KEYS: each walks its own contiguous range of 16-key
// tiles with a running reference, and the partial results meet in LDS at the end.  An fp32 MFMA keeps vector
// instructions out, of its own wave and of the other one on the SIMD (measured: 32 cycles each alone, 49 with two v_add
// behind each, 40.5 per wave with two waves): what a tile costs beside its 64 products is its count of vector
// instructions, which is what the code below is written to keep down.
//
// Per tile, S^T = K Q^T and O^T += V^T P^T.  The order of the contraction index is free: for QK lane (g, r) = (lane /
// 16, lane % 16) holds dims 16j + 4g .. +3 of key r, and k-step (j, i) multiplies dims 16j + 4g + i; for PV k-step i
// multiplies keys 4g + i, which is what the S^T accumulator (keys 4g + i of query r in register i) hands over without
// any movement; an accumulator tile c of O^T holds dims 4m + c (2m + c at head_dim 32), so that one 16-byte load per
// key feeds four tiles.  V is loaded that way straight from the pool: 16 lanes to a row.  K would meet 16 rows in an
// instruction (64 cache accesses for V's 16), so it is loaded as it lies and turned through 16 rows of LDS of the
// wave's own.  A tile's V is requested before its K is multiplied, K two tiles ahead.  Within a page and a block rows
// lie one behind the other, and a load needs no address of its own; a tile that crosses into another page or ends its
// block finds its rows one by one.
//
// Weights are exp2(s c + n) with c = log2(e) / sqrt(D) and n = -(reference) c: one fused multiply-add and v_exp_f32
// (within an ulp).  A row's reference moves only when four of its weights sum to more than kSlack, so that the common
// tile has no maximum, no cross-lane step and no rescaling.  Errors against fp64 over 18 shapes and scales, six seeds
// each: 8.49e-8 .. 1.03e-6, where weights of expf of rounded logits had 8.56e-8 ..  1.06e-6.
//
// Measured (4 heads x 3 blocks of 576 rows, 3..5 KV blocks of 576, head_dim 128; whole step with two other launches):
// 118.8 us when loads stood in a bunch and a tile took 117 vector instructions, 114.7 with 30, 101 with loads dealt
// out, 93 with the second round of workgroups in reverse order (attention 82 us = 99 TFLOP/s; a loop of nothing but
// these MFMAs reaches 137 at the 2.1 GHz it holds).  Two waves a SIMD take 2380 cycles a tile of each, one alone
// 2765, of which 2048 are products.  2 heads x 144 rows x 432 keys, head_dim 64: 10.5 us, launch and loads from cold
// caches.
//
// Visibility per block pair follows Sec. 3.1 (a block is bidirectional inside), Sec. 3.3
// (cached blocks visible to all) and Sec. 3.4 / 4.2 (bidirectional or block-causal cascade).
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>

#include "ca_internal.hpp"

namespace ca {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kTileRows = 16;                  // queries per workgroup
constexpr int kTileKeys = 16;                  // keys per step of a wave
constexpr float kSlack = 4096.f;               // weights up to 2^12 cost a 32-bit sum nothing

struct F32Args {
  AttnPlan p;
  const float* q;
  float* out;
  const float* pool;
  int32_t row_tiles, cols, cols_per_xcd;       // cols = heads * row tiles
  int32_t fold_from, fold_sum;                 // item i >= fold_from of an XCD is item fold_sum - i
  float c;                                     // log2(e) / sqrt(head_dim)
};

template <int D>
struct Shape {
  static constexpr int kVecs = D / 16;         // 16-byte pieces of a K row per lane
  static constexpr int kW = D >= 64 ? 4 : 2;   // dims of a V row per piece
  static constexpr int kPieces = D / (16 * kW);
  static constexpr int kChunks = D / 4;        // 16-byte chunks of a row
  static constexpr int kRowsPerLoad = 64 / kChunks;   // rows of K that one load of a wave covers
};

// A wave's place in its walk over 16-key tiles.
struct Tile {
  const char* first;                           // K row of the tile's first key, for this head
  int row0, kb, in_blk;                        // that row in its page; visible KV block; tile of the block
};

struct Geometry {                              // of the pool, in bytes
  size_t page_step, v_off;                     // to the same head's next page; from a K page to its V page
  uint32_t jump;                               // what a row past the end of its page is further on than in line (not kFar)
  float inv_page;                              // 1 / page_tokens
};

// Row `row` of the tile (keys past the block's end: its last one, `valid` exist), from the tile's first row on, in
// bytes.  kFar: pages of less than 16 tokens, of which a tile may span several, or farther apart than 32 bits of
// bytes; otherwise a tile crosses into one more page at most.
template <int D, bool kFar>
__device__ __forceinline__ auto row_offset(const AttnPlan& p, const Geometry& geo, const Tile& t, int row, int valid) {
  const int r = min(row, valid - 1);
  if constexpr (!kFar) {
    return uint32_t(r * D * 4) + (t.row0 + r >= p.page_tokens ? geo.jump : 0u);
  } else {
    const int in = t.row0 + r;                                // < page_tokens + 16
    const int pg = int((float(in) + 0.5f) * geo.inv_page);      // in / page_tokens: at most 16, 0.5 / 4096 from an integer
    return size_t(pg) * geo.page_step + size_t(in - pg * p.page_tokens) * D * 4 - size_t(t.row0) * D * 4;
  }
}

// what a wave wrote to LDS is there for its other lanes (a wave's LDS accesses complete in order)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <int D, int kWaves, bool kFar>
__global__ __launch_bounds__(64 * kWaves, 2) void attn_f32_kernel(F32Args a) {
  using T = Shape<D>;
  typedef __attribute__((ext_vector_type(T::kW))) float VPiece;
  const AttnPlan& p = a.p;
  // XCD x takes a contiguous range of (head, row tile) columns, all of them for the latest query block
  // (longest KV prefix) first: what runs together shares K/V in its L2, and every XCD gets the same work
  int nth = int(blockIdx.y * (gridDim.x >> 3) + (blockIdx.x >> 3));
  nth = nth >= a.fold_from ? a.fold_sum - nth : nth;
  const int seg = nth / a.cols_per_xcd;
  const int col = int(blockIdx.x & 7) * a.cols_per_xcd + (nth - seg * a.cols_per_xcd);
  if (seg >= p.n_q_blocks || col >= a.cols) return;
  const int h = col / a.row_tiles, qb = p.n_q_blocks - 1 - seg;
  const int row0 = (col - h * a.row_tiles) * kTileRows;
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int L = p.block_tokens;
  __shared__ __attribute__((aligned(16))) float stage[kWaves][16 * D];   // a wave's K tile; in the end its accumulators
  __shared__ float2 row_stat[kWaves][16];                                // n and row sum

  Geometry geo;
  geo.v_off = size_t(p.page_tokens) * D * 4;
  geo.page_step = size_t(p.heads) * 2 * geo.v_off;
  geo.jump = uint32_t(geo.page_step - geo.v_off);
  geo.inv_page = 1.0f / float(p.page_tokens);
  const int block_tiles = (L + kTileKeys - 1) / kTileKeys;
  const int tiles = p.n_vis[qb] * block_tiles;
  const int t_begin = int(int64_t(tiles) * wave / kWaves), t_end = int(int64_t(tiles) * (wave + 1) / kWaves);
  auto first_page = [&](int kb) {
    return reinterpret_cast<const char*>(a.pool) + (size_t(p.kv_slot[kb]) * p.pages_per_block * p.heads + h) * 2 * geo.v_off;
  };
  auto advance = [&](Tile& t) {
    ++t.in_blk;
    t.row0 += kTileKeys;
    t.first += kTileKeys * D * 4;
    if (__builtin_expect(t.in_blk == block_tiles, 0)) {
      t.in_blk = t.row0 = 0;
      t.first = first_page(++t.kb);
    } else if (kFar) {
      const int pg = t.row0 / p.page_tokens;
      t.first += pg * (geo.page_step - geo.v_off);
      t.row0 -= pg * p.page_tokens;
    } else if (t.row0 >= p.page_tokens) {
      t.first += geo.jump;
      t.row0 -= p.page_tokens;
    }
  };
  auto keys_of = [&](const Tile& t) { return min(kTileKeys, L - t.in_blk * kTileKeys); };
  auto in_line = [&](const Tile& t) { return !kFar && keys_of(t) == kTileKeys && t.row0 + kTileKeys <= p.page_tokens; };

  // ---- K: whole rows to registers, to LDS (chunk c of row r at position c ^ r, or c ^ (r % 8) with 8 chunks to a row), to operands
  f32x4 k[T::kVecs], kin[T::kVecs];
  const int in_row = lane / T::kChunks, in_chunk = lane % T::kChunks;
  float* const mine = stage[wave];
  // Where a lane's rows of a tile are: the same from tile to tile while rows lie in line, so found again only for a
  // tile where they do not and for the one behind it
  decltype(row_offset<D, kFar>(p, geo, Tile(), 0, 0)) k_off[T::kVecs], v_off[4];
  bool k_in_line = false, v_in_line = false;
  auto place_k = [&](const Tile& t) {
    const bool line = in_line(t);
    if (!(line && k_in_line)) {
      const int valid = keys_of(t);
#pragma unroll
      for (int j = 0; j < T::kVecs; ++j) k_off[j] = row_offset<D, kFar>(p, geo, t, j * T::kRowsPerLoad + in_row, valid) + 16u * in_chunk;
    }
    k_in_line = line;
  };
  auto place_v = [&](const Tile& t) {
    const bool line = in_line(t);
    if (!(line && v_in_line)) {
      const int valid = keys_of(t);
#pragma unroll
      for (int i = 0; i < 4; ++i) v_off[i] = row_offset<D, kFar>(p, geo, t, 4 * g + i, valid) + 4u * T::kW * r;
    }
    v_in_line = line;
  };
  auto request_k = [&](const Tile& t, int j) {
    kin[j] = *reinterpret_cast<const f32x4*>(t.first + k_off[j]);
  };
  auto turn_k = [&](int j) {
    const int row = j * T::kRowsPerLoad + in_row;
    *reinterpret_cast<f32x4*>(mine + row * D + 4 * (in_chunk ^ (row & (T::kChunks - 1) & 15))) = kin[j];
  };
  auto read_k = [&](int j) { k[j] = *reinterpret_cast<const f32x4*>(mine + r * D + 4 * ((4 * j + g) ^ (r & (T::kChunks - 1)))); };
  Tile now, next, later;                       // the tile multiplied, the one whose K is on its way, the one behind
  now.kb = t_begin / block_tiles;
  now.in_blk = t_begin - now.kb * block_tiles;
  if (t_begin < t_end) {
    const int n0 = now.in_blk * kTileKeys, pg = n0 / p.page_tokens;
    now.row0 = n0 - pg * p.page_tokens;
    now.first = first_page(now.kb) + pg * geo.page_step + now.row0 * D * 4;
    place_k(now);
#pragma unroll
    for (int j = 0; j < T::kVecs; ++j) request_k(now, j);
  }

  const int qrow = min(row0 + r, L - 1);
  const float* qp = a.q + ((int64_t(qb) * L + qrow) * p.heads + h) * D + 4 * g;
  f32x4 q[T::kVecs];
#pragma unroll
  for (int j = 0; j < T::kVecs; ++j) q[j] = *reinterpret_cast<const f32x4*>(qp + 16 * j);

  f32x4 o[D / 16];
#pragma unroll
  for (int c = 0; c < D / 16; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  // l: of this lane's keys 4g .. 4g+3 only.  n is finite from the start, so that a tile of scores that are all -inf
  // has weights of 0; the first other one has infinite ones and moves the reference
  float n = FLT_MAX, l = 0.f;

  if (t_begin < t_end) {
#pragma unroll
    for (int j = 0; j < T::kVecs; ++j) turn_k(j);
    wave_lds_fence();
    next = now;
    if (t_begin + 1 < t_end) advance(next);
    place_k(next);
#pragma unroll
    for (int j = 0; j < T::kVecs; ++j) {
      request_k(next, j);
      read_k(j);
    }
  }
  // A wave's loads and LDS accesses are dealt out among its products, four of those at a time: in a bunch, 8 loads and
  // 16 LDS accesses hold it up for 1000 to 1400 cycles a tile.
  for (int t = t_begin; t < t_end; ++t) {
    place_v(now);
    const int valid = keys_of(now);
    constexpr int kGroups = T::kVecs, kHalf = kGroups / 2, kLoadsV = 4 * T::kPieces / kGroups;
    VPiece v[4][T::kPieces];
    const char* v_base = now.first + geo.v_off;
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};   // two half sums: half as many roundings in a chain
#pragma unroll
    for (int m = 0; m < kGroups; ++m) {
#pragma unroll
      for (int e = m * kLoadsV; e < (m + 1) * kLoadsV; ++e) {
        const int i = e / T::kPieces, c = e % T::kPieces;
        v[i][c] = *reinterpret_cast<const VPiece*>(v_base + 256 * c + v_off[i]);
      }
      __builtin_amdgcn_sched_barrier(0);      // what is dealt out stays where it is
      s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[m][0], q[m][0], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[m][1], q[m][1], s1, 0, 0, 0);
      s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[m][2], q[m][2], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[m][3], q[m][3], s1, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (m == 0) {
        later = next;                          // past the end: the last tile again
        if (t + 2 < t_end) advance(later);
      }
      if (m == 1) place_k(later);
    }
    float s[4], w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = s0[i] + s1[i];
    if (__builtin_expect(valid < kTileKeys, 0)) {             // keys that do not exist: weight 0, and 0 x a re-read inf would be NaN
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[i] = 4 * g + i < valid ? s[i] : -INFINITY;
#pragma unroll
        for (int c = 0; c < D / 16; ++c) v[i][c / T::kW][c % T::kW] = 4 * g + i < valid ? v[i][c / T::kW][c % T::kW] : 0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = __builtin_amdgcn_exp2f(fmaf(s[i], a.c, n));
    float tile_sum = (w[0] + w[1]) + (w[2] + w[3]);
    if (__builtin_expect(__any(tile_sum > kSlack), 0)) {      // on the first tile with a score above -inf, and seldom after
      float tm = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
      tm = fmaxf(tm, __shfl_xor(tm, 16));
      tm = fmaxf(tm, __shfl_xor(tm, 32));
      const float n_new = fminf(n, -tm * a.c);                // the reference never moves down
      const float alpha = __builtin_amdgcn_exp2f(n_new - n);  // 0 on the first tile
      l *= alpha;
      n = n_new;
#pragma unroll
      for (int c = 0; c < D / 16; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[c][i] *= alpha;
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = __builtin_amdgcn_exp2f(fmaf(s[i], a.c, n));
      tile_sum = (w[0] + w[1]) + (w[2] + w[3]);
    }
    l += tile_sum;
    wave_lds_fence();
    // beside O^T += V^T P^T: the next tile's K to LDS, the one behind it requested, the next one's operands read
#pragma unroll
    for (int m = 0; m < kGroups; ++m) {
      if (m < kHalf) {
        turn_k(2 * m);
        turn_k(2 * m + 1);
      }
      if (m == kHalf) wave_lds_fence();
      request_k(later, m);
      if (m >= kHalf) {
        read_k(2 * (m - kHalf));
        read_k(2 * (m - kHalf) + 1);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 4 * m; e < 4 * m + 4; ++e) {
        const int i = e / (D / 16), c = e % (D / 16);
        o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[i][c / T::kW][c % T::kW], w[i], o[c], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    now = next;
    next = later;
  }

  // ---- the waves' partial results meet: all of them to LDS, then each wave adds up its share of the accumulators over all
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (g == 0) row_stat[wave][r] = make_float2(n, l);
  wave_lds_fence();
#pragma unroll
  for (int c = 0; c < D / 16; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) mine[(4 * c + i) * 64 + lane] = o[c][i];
  __syncthreads();
  float2 stat[kWaves];
  float least = FLT_MAX;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    stat[w] = row_stat[w][r];
    least = fminf(least, stat[w].x);
  }
#pragma unroll
  for (int w = 0; w < kWaves; ++w) stat[w].x = __builtin_amdgcn_exp2f(least - stat[w].x);
  // sum of a value per wave, weighted, in pairs: fewer roundings in a row than one after the other
  auto over_waves = [&](auto value) {
    float x[kWaves / 2];
#pragma unroll
    for (int w = 0; w < kWaves / 2; ++w) x[w] = fmaf(stat[2 * w].x, value(2 * w), stat[2 * w + 1].x * value(2 * w + 1));
#pragma unroll
    for (int step = 1; step < kWaves / 2; step *= 2)
#pragma unroll
      for (int w = 0; w < kWaves / 2; w += 2 * step) x[w] += x[w + step];
    return x[0];
  };
  const float inv = 1.0f / over_waves([&](int w) { return stat[w].y; });
  float* const op = a.out + ((int64_t(qb) * L + row0 + r) * p.heads + h) * D;
#pragma unroll
  for (int part = wave; part < 4 * T::kPieces; part += kWaves) {
    const int c = part >> 2, i = part & 3;
    float sum[T::kW];
#pragma unroll
    for (int e = 0; e < T::kW; ++e)
      sum[e] = over_waves([&](int w) { return stage[w][(4 * (T::kW * c + e) + i) * 64 + lane]; });
    if (row0 + r < L) {
      float* to = op + 16 * T::kW * c + T::kW * (4 * g + i);
      if (T::kW == 4)
        *reinterpret_cast<float4*>(to) = make_float4(sum[0] * inv, sum[1] * inv, sum[T::kW - 2] * inv, sum[T::kW - 1] * inv);
      else
        *reinterpret_cast<float2*>(to) = make_float2(sum[0] * inv, sum[1] * inv);
    }
  }
}

template <int D, int kWaves>
void enqueue_attn_f32(const F32Args& a, dim3 grid, hipStream_t s) {
  const bool far = a.p.page_tokens < kTileKeys || size_t(a.p.heads) * 2 * a.p.page_tokens * D * 4 >= (size_t(1) << 31);
  const auto kernel = far ? attn_f32_kernel<D, kWaves, true> : attn_f32_kernel<D, kWaves, false>;
  hipLaunchKernelGGL(kernel, grid, dim3(64 * kWaves), 0, s, a);
}

}  // namespace

int32_t launch_attn_f32(const AttnPlan& p, const void* q, void* out, const void* pool, void* stream) {
  F32Args a{};
  a.p = p;
  a.q = static_cast<const float*>(q);
  a.out = static_cast<float*>(out);
  a.pool = static_cast<const float*>(pool);
  a.row_tiles = (p.block_tokens + kTileRows - 1) / kTileRows;
  const int64_t cols = int64_t(p.heads) * a.row_tiles, items = cols * p.n_q_blocks;
  if (items > (int64_t(1) << 30)) return CA_EUNSUPPORTED;
  a.cols = int32_t(cols);
  a.cols_per_xcd = (a.cols + 7) / 8;
  a.c = 1.4426950408889634f / sqrtf(float(p.head_dim));
  const int per_xcd = a.cols_per_xcd * p.n_q_blocks;
  constexpr int kMaxX = 1 << 16;                              // workgroups in x per XCD; a launch may have 2^32 threads in x
  const int gx = per_xcd < kMaxX ? per_xcd : kMaxX;
  const dim3 grid(unsigned(gx) * 8, unsigned((per_xcd + gx - 1) / gx));
  int n_cu = 0;
  if (const int32_t rc = device_cu_count(&n_cu); rc != CA_OK) return rc;
  const int cus_per_xcd = n_cu >= 8 ? n_cu / 8 : 1;
  // Two workgroups share a CU.  Where the launch is between one and two of them a CU, the second round goes the other
  // way, so that the CUs with the longest walks get the shortest ones as their second: walks of 5 and 4 blocks then
  // meet with 3 and 4 (8 at the most, 93 us) instead of 4 and 3 (9, 101 us).  Longer launches keep the longest first.
  const bool fold = per_xcd > cus_per_xcd && per_xcd <= 2 * cus_per_xcd;
  a.fold_from = fold ? cus_per_xcd : INT32_MAX;
  a.fold_sum = cus_per_xcd + per_xcd - 1;
  // Eight waves share out the key tiles of a row tile.  At head_dim 128 a wave needs 211 registers, so a CU holds one
  // workgroup of eight waves but two of four: four once every CU has a workgroup anyway.  Measured on 256 CUs, a
  // whole step of 432 row tiles: 93 us with four, 108 with eight.
  const bool narrow = p.head_dim == 128 && items > n_cu;
  hipStream_t s = static_cast<hipStream_t>(stream);
  switch (p.head_dim) {
    case 32: enqueue_attn_f32<32, 8>(a, grid, s); break;
    case 64: enqueue_attn_f32<64, 8>(a, grid, s); break;
    case 128:
      if (narrow) enqueue_attn_f32<128, 4>(a, grid, s);
      else enqueue_attn_f32<128, 8>(a, grid, s);
      break;
    default: return CA_EUNSUPPORTED;
  }
  return finish_launch("attn_f32.hip");
}

}  // namespace ca
