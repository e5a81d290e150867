// fp32 block-cascaded attention for the small fp32 configurations (head_dim 32/64/128, pages of any
// size): the exact path one checks a model with.  All arithmetic is fp32; the two products run on
// the fp32 matrix instruction v_mfma_f32_16x16x4_f32 (fused multiply-adds, fp32 accumulation).
//
// What bounds it: at the sizes it serves (10^2..10^4 keys, a few heads) the length of one wave's
// serial chain, then the fp32 matrix rate (256 flop/clk per CU).  So a workgroup takes only 16 query
// rows of one head, and its waves share the KEYS: each walks its own contiguous range of 16-key
// tiles with a running maximum, and the partial results meet in LDS at the end.
//
// Per tile, S^T = K Q^T and O^T += V^T P^T.  The order of the contraction index is free, so operands
// are loaded as 16-byte pieces of rows straight from the pool (no LDS): for QK lane (g, r) = (lane /
// 16, lane % 16) takes dims 16j + 4g .. +3 of key r, and k-step (j, i) multiplies dims 16j + 4g + i;
// for PV k-step i multiplies keys 4g + i, which is what the S^T accumulator (keys 4g + i of query r in
// register i) hands over without any movement; an accumulator tile c of O^T holds dims 4m + c
// (2m + c at head_dim 32), so that one 16-byte load per key feeds four tiles.  The next tile's rows are
// requested before the present one is multiplied.
//
// A row's exponent reference stays until a score exceeds it by kSlack: the common tile needs no cross-lane maximum and no
// rescaling (219 -> 120 vector instructions a tile beside its 64 products).
//
// Measured (2 heads x 144 rows x 432 keys, head_dim 64): 318 -> 11 us; (4 heads x 3 blocks of 576 rows,
// 3..5 KV blocks of 576, head_dim 128): 12.2 ms -> 117 us = 70 TFLOP/s of the 157 the fp32 matrix
// instruction has; one thread per query row walked every key before.  A CU takes 3200 cycles per round of four tiles
// with one wave a SIMD as with two (2048 of them products): what bounds it now is the 16 KB a tile fetches from L2.
//
// Visibility per block pair follows Sec. 3.1 (a block is bidirectional inside), Sec. 3.3
// (cached blocks visible to all) and Sec. 3.4 / 4.2 (bidirectional or block-causal cascade).
#include <hip/hip_runtime.h>

#include <cfloat>

#include "ca_internal.hpp"

namespace ca {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kTileRows = 16;                  // queries per workgroup
constexpr int kTileKeys = 16;                  // keys per step of a wave
constexpr int kMaxWaves = 8;

struct F32Args {
  AttnPlan p;
  const float* q;
  float* out;
  const float* pool;
  int32_t row_tiles, cols, cols_per_xcd;       // cols = heads * row tiles
};

template <int D>
struct Shape {
  static constexpr int kVecs = D / 16;         // 16-byte pieces of a K row per lane
  static constexpr int kW = D >= 64 ? 4 : 2;   // dims of a V row per piece
  static constexpr int kPieces = D / (16 * kW);
};

// One 16-key tile of the walk: where its rows are.
struct TilePos {
  const float* page;                           // K page of the tile's first key, for this head
  size_t page_step, v_off;                     // to the same head's next page; from a K page to its V page
  int row0, page_tokens, valid;                // first key's row in its page; keys of the tile that exist
  float inv_page;                              // 1 / page_tokens
  // keys past the block's end re-read its last one; pages of 16 tokens or more: a tile crosses into one more at most
  template <bool kTinyPages>
  __device__ __forceinline__ const float* row(int key, int d) const {
    const int r = row0 + min(key, valid - 1);                 // < page_tokens + 16
    if (!kTinyPages) return page + (r >= page_tokens ? page_step - size_t(page_tokens * d) : 0) + uint32_t(r * d);
    const int pg = int((float(r) + 0.5f) * inv_page);         // r / page_tokens: at most 16, 0.5 / 4096 from an integer
    return page + uint32_t(pg) * page_step + uint32_t((r - pg * page_tokens) * d);
  }
};

// exp(x) for x <= kSlack + a little, the softmax's range: 2^t with t = x log2 e in two parts, the second one applied to the
// result to first order.  v_exp_f32 is within an ulp; expf spends its further instructions on the rest of the range.
__device__ __forceinline__ float softmax_exp(float x) {
  const float t = x * 1.44269504f;
  const float e = fmaf(x, 1.44269504f, -t) + x * 1.92596299e-8f;         // log2 e = 1.44269504 + 1.92596299e-8
  const float r = __builtin_amdgcn_exp2f(t);
  return x > -126.f ? fmaf(r, e * 0.693147181f, r) : r;                   // far below (or -inf): r is 0 or next to it
}

// A row's exponent reference moves only when a score exceeds it by more than this: weights up to e^8 cost a 32-bit sum nothing
constexpr float kSlack = 8.f;

__device__ __forceinline__ TilePos tile_pos(const AttnPlan& p, const float* pool, int h, int kb, int n0, int d) {
  TilePos t;
  const int pg = n0 / p.page_tokens;           // wave-uniform
  t.v_off = size_t(p.page_tokens) * d;
  t.page_step = size_t(p.heads) * 2 * t.v_off;
  t.page = pool + (size_t(p.kv_slot[kb]) * p.pages_per_block * p.heads + h) * 2 * t.v_off + pg * t.page_step;
  t.row0 = n0 - pg * p.page_tokens;
  t.page_tokens = p.page_tokens;
  t.inv_page = 1.0f / float(p.page_tokens);
  t.valid = min(kTileKeys, p.block_tokens - n0);
  return t;
}

template <int D, bool kTinyPages>
__global__ __launch_bounds__(64 * kMaxWaves) void attn_f32_kernel(F32Args a) {
  using T = Shape<D>;
  const AttnPlan& p = a.p;
  // XCD x takes a contiguous range of (head, row tile) columns, all of them for the latest query block
  // (longest KV prefix) first: what runs together shares K/V in its L2, and every XCD gets the same work
  const int nth = int(blockIdx.y * (gridDim.x >> 3) + (blockIdx.x >> 3));
  const int seg = nth / a.cols_per_xcd;
  const int col = int(blockIdx.x & 7) * a.cols_per_xcd + (nth - seg * a.cols_per_xcd);
  if (seg >= p.n_q_blocks || col >= a.cols) return;
  const int h = col / a.row_tiles, qb = p.n_q_blocks - 1 - seg;
  const int row0 = (col - h * a.row_tiles) * kTileRows;
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  const int L = p.block_tokens;

  const int qrow = min(row0 + r, L - 1);
  const float* qp = a.q + ((int64_t(qb) * L + qrow) * p.heads + h) * D + 4 * g;
  f32x4 q[T::kVecs];
#pragma unroll
  for (int j = 0; j < T::kVecs; ++j) q[j] = *reinterpret_cast<const f32x4*>(qp + 16 * j);

  const float scale = 1.0f / sqrtf(float(D));
  f32x4 o[D / 16];
#pragma unroll
  for (int c = 0; c < D / 16; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  // l: of this lane's keys 4g .. 4g+3 only; m is finite from the start, so that a tile of scores that are all -inf has weights of 0
  float m = -FLT_MAX, l = 0.f;

  const int block_tiles = (L + kTileKeys - 1) / kTileKeys;
  const int tiles = p.n_vis[qb] * block_tiles;
  const int t_begin = int(int64_t(tiles) * wave / waves), t_end = int(int64_t(tiles) * (wave + 1) / waves);
  int kb = t_begin / block_tiles, in_blk = t_begin - kb * block_tiles;
  f32x4 k[T::kVecs];
  TilePos pos = tile_pos(p, a.pool, h, min(kb, p.n_vis[qb] - 1), in_blk * kTileKeys, D);
  auto load_k = [&]() {
    const float* kr = pos.row<kTinyPages>(r, D) + 4 * g;
#pragma unroll
    for (int j = 0; j < T::kVecs; ++j) k[j] = *reinterpret_cast<const f32x4*>(kr + 16 * j);
  };
  if (t_begin < t_end) load_k();
  for (int t = t_begin; t < t_end; ++t) {
    // V of this tile is on its way while K is multiplied, K of the next one during softmax and PV
    float v[4][T::kPieces][T::kW];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* vr = pos.row<kTinyPages>(4 * g + i, D) + pos.v_off + T::kW * r;
#pragma unroll
      for (int c = 0; c < T::kPieces; ++c) {
        if (T::kW == 4) {
          const float4 x = *reinterpret_cast<const float4*>(vr + 64 * c);
          v[i][c][0] = x.x; v[i][c][1] = x.y; v[i][c][T::kW - 2] = x.z; v[i][c][T::kW - 1] = x.w;
        } else {
          const float2 x = *reinterpret_cast<const float2*>(vr);
          v[i][c][0] = x.x; v[i][c][1] = x.y;
        }
      }
    }
    const int valid = pos.valid;
    __builtin_amdgcn_sched_barrier(0);        // loads stay where they are: left alone they sink to their uses
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};   // two chains: the result latency is hidden
#pragma unroll
    for (int j = 0; j < T::kVecs; ++j) {
      s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[j][0], q[j][0], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[j][1], q[j][1], s1, 0, 0, 0);
      s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[j][2], q[j][2], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[j][3], q[j][3], s1, 0, 0, 0);
    }
    // no branch around the loads (the last tile's are repeated, unused): the compiler's wait counts stay exact
    in_blk += t + 1 < t_end ? 1 : 0;
    kb += in_blk == block_tiles ? 1 : 0;
    in_blk = in_blk == block_tiles ? 0 : in_blk;
    pos = tile_pos(p, a.pool, h, kb, in_blk * kTileKeys, D);
    load_k();
    __builtin_amdgcn_sched_barrier(0);
    float s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = 4 * g + i < valid ? (s0[i] + s1[i]) * scale : -INFINITY;
    float tm = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    if (__builtin_expect(__any(tm > m + kSlack), 0)) {        // on the first tile, whatever its scores unless they are all -inf
      tm = fmaxf(tm, __shfl_xor(tm, 16));
      tm = fmaxf(tm, __shfl_xor(tm, 32));
      const float m_new = fmaxf(m, tm);
      const float alpha = expf(m - m_new);                    // 0 on the first tile
      l *= alpha;
      m = m_new;
#pragma unroll
      for (int c = 0; c < D / 16; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[c][i] *= alpha;
    }
    float w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = softmax_exp(s[i] - m);
    l += (w[0] + w[1]) + (w[2] + w[3]);
    if (__builtin_expect(valid < kTileKeys, 0)) {             // keys that do not exist: 0 x a re-read inf would be NaN
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < D / 16; ++c) v[i][c / T::kW][c % T::kW] = 4 * g + i < valid ? v[i][c / T::kW][c % T::kW] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < D / 16; ++c)
        o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[i][c / T::kW][c % T::kW], w[i], o[c], 0, 0, 0);
  }

  // ---- the waves' partial results meet: the upper half hands over to the lower until one is left
  __shared__ float stage[kMaxWaves / 2][D / 4 + 2][64];
  for (int half = waves >> 1; half >= 1; half >>= 1) {
    if (wave >= half && wave < 2 * half) {
      float (*to)[64] = stage[wave - half];
#pragma unroll
      for (int c = 0; c < D / 16; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) to[4 * c + i][lane] = o[c][i];
      to[D / 4][lane] = m;
      to[D / 4 + 1][lane] = l;
    }
    __syncthreads();
    if (wave < half) {
      const float (*from)[64] = stage[wave];
      const float mb = from[D / 4][lane], mm = fmaxf(m, mb);
      const float wa = expf(m - mm), wb = expf(mb - mm);
      l = l * wa + from[D / 4 + 1][lane] * wb;
      m = mm;
#pragma unroll
      for (int c = 0; c < D / 16; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[c][i] = o[c][i] * wa + from[4 * c + i][lane] * wb;
    }
    __syncthreads();
  }
  if (wave == 0) {
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (row0 + r < L) {
      const float inv = 1.0f / l;
      float* op = a.out + ((int64_t(qb) * L + row0 + r) * p.heads + h) * D;
#pragma unroll
      for (int c = 0; c < T::kPieces; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int e = 0; e < T::kW; ++e)
            op[16 * T::kW * c + T::kW * (4 * g + i) + e] = o[T::kW * c + e][i] * inv;
    }
  }
}

template <int D>
void enqueue_attn_f32(const F32Args& a, dim3 grid, int waves, hipStream_t s) {
  const auto kernel = a.p.page_tokens < kTileKeys ? attn_f32_kernel<D, true> : attn_f32_kernel<D, false>;
  hipLaunchKernelGGL(kernel, grid, dim3(unsigned(64 * waves)), 0, s, a);
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
  const int per_xcd = a.cols_per_xcd * p.n_q_blocks;
  constexpr int kMaxX = 1 << 16;                              // workgroups in x per XCD; a launch may have 2^32 threads in x
  const int gx = per_xcd < kMaxX ? per_xcd : kMaxX;
  const dim3 grid(unsigned(gx) * 8, unsigned((per_xcd + gx - 1) / gx));
  // Eight waves share out the key tiles of a row tile.  At head_dim 128 a wave needs 160 registers, so a CU holds one
  // workgroup of eight waves but three of four: four once every CU has a workgroup anyway.  Measured on 256 CUs, a
  // whole step: 432 row tiles 153 us with four, 162 with eight; 162 tiles 75 with four, 73 with eight; at
  // head_dim 64 (98 registers, 432 tiles) 101 with four, 98 with eight.
  int n_cu = 0;
  if (const int32_t rc = device_cu_count(&n_cu); rc != CA_OK) return rc;
  const int waves = p.head_dim == 128 && items > n_cu ? 4 : kMaxWaves;
  hipStream_t s = static_cast<hipStream_t>(stream);
  switch (p.head_dim) {
    case 32: enqueue_attn_f32<32>(a, grid, waves, s); break;
    case 64: enqueue_attn_f32<64>(a, grid, waves, s); break;
    case 128: enqueue_attn_f32<128>(a, grid, waves, s); break;
    default: return CA_EUNSUPPORTED;
  }
  return finish_launch("attn_f32.hip");
}

}  // namespace ca
