"""Kernel variants and dispatch branches at the sizes where they can go wrong: edges of tiles,
remainders, the smallest and the largest of their range -- against the fp64 oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import cascade_oracle as orc
from tests import _harness as Hn

pytestmark = pytest.mark.gpu

BI, CA = orc.BIDIRECTIONAL, orc.BLOCK_CAUSAL
DIMS = {32: (12, 10, 10), 64: (24, 20, 20), 128: (44, 42, 42)}


# fp32 attention: 16-key tiles shared out over the waves of a workgroup.  One key in all (most
# waves get none), one tile, a tile and a key, pages shorter than a tile, several tiles per wave.
@pytest.mark.parametrize("head_dim", [32, 64, 128])
@pytest.mark.parametrize("fpb,gh,gw,page,nc,ni", [(1, 1, 1, 1, 0, 1), (1, 4, 4, 48, 0, 1), (1, 1, 17, 1, 0, 1),
                                                  (1, 3, 11, 5, 1, 2), (3, 7, 13, 100, 2, 3)])
def test_f32_key_tiles(head_dim, fpb, gh, gw, page, nc, ni):
    w = W.small_variant(W.CONFIGS["c1_tiny_f32"], heads=3, grid_h=gh, grid_w=gw, frames_per_block=fpb, head_dim=head_dim,
                        rope_dims=DIMS[head_dim], page_tokens=page, n_cached=nc, n_inflight=ni, max_inflight=3)
    cached, infl = list(range(nc)), list(range(nc, nc + ni))
    q, k, v = W.draw_config(w, seed=5, scale=1.5)
    pool = Hn.gpu_setup(w, k, v, cached, infl)
    for mode in (BI, CA):
        out = Hn.gpu_forward(w, pool, q, infl, mode)
        ref = np.concatenate(Hn.oracle_forward(w, q, k, v, cached, infl, mode))
        Hn.assert_close(out, ref, "f32", f"f32 tiles D={head_dim} L={w.block_tokens} page={page} mode={mode}")


# ... and shared out over four waves instead of eight, at head_dim 128 from more work items (heads x row tiles x
# blocks) than CUs on: 288 and 258 items, and 256, where it is eight still.
@pytest.mark.parametrize("heads,fpb,gh,gw,ni", [(4, 2, 5, 37, 3), (3, 1, 19, 36, 2), (4, 1, 10, 25, 4)])
def test_f32_waves_per_row_tile(heads, fpb, gh, gw, ni):
    w = W.small_variant(W.CONFIGS["c1_tiny_f32"], heads=heads, grid_h=gh, grid_w=gw, frames_per_block=fpb, head_dim=128, rope_dims=DIMS[128],
                        page_tokens=100, n_cached=1, n_inflight=ni, max_inflight=4)
    infl = list(range(1, 1 + ni))
    q, k, v = W.draw_config(w, seed=15, scale=1.5)
    pool = Hn.gpu_setup(w, k, v, [0], infl)
    for mode in (BI, CA):
        out = Hn.gpu_forward(w, pool, q, infl, mode)
        ref = np.concatenate(Hn.oracle_forward(w, q, k, v, [0], infl, mode))
        Hn.assert_close(out, ref, "f32", f"f32 waves heads={heads} L={w.block_tokens} blocks={ni} mode={mode}")


# ... and whose rows lie in line or not: pages just longer than a tile (every tile crosses into the next page), a
# little shorter than two, whole tiles with a ragged last one; 480 items, whose second round is taken in reverse
# order.
@pytest.mark.parametrize("head_dim", [32, 64, 128])
@pytest.mark.parametrize("heads,fpb,gh,gw,page,nc,ni", [(2, 1, 7, 11, 17, 2, 1), (2, 1, 9, 13, 31, 1, 2), (1, 2, 8, 9, 64, 1, 2), (4, 2, 16, 20, 100, 1, 3)])
def test_f32_tiles_across_pages(head_dim, heads, fpb, gh, gw, page, nc, ni):
    w = W.small_variant(W.CONFIGS["c1_tiny_f32"], heads=heads, grid_h=gh, grid_w=gw, frames_per_block=fpb, head_dim=head_dim,
                        rope_dims=DIMS[head_dim], page_tokens=page, n_cached=nc, n_inflight=ni, max_inflight=3)
    cached, infl = list(range(nc)), list(range(nc, nc + ni))
    q, k, v = W.draw_config(w, seed=25, scale=1.5)
    pool = Hn.gpu_setup(w, k, v, cached, infl)
    out = Hn.gpu_forward(w, pool, q, infl, CA)
    ref = np.concatenate(Hn.oracle_forward(w, q, k, v, cached, infl, CA))
    Hn.assert_close(out, ref, "f32", f"f32 across pages D={head_dim} L={w.block_tokens} page={page}")


# fp32 attention, an infinite V in a block's last row: its dimension is infinite, all else finite.  (The tile that row
# is in is filled up with keys that do not exist.)
@pytest.mark.parametrize("head_dim", [32, 64, 128])
@pytest.mark.parametrize("fpb,gh,gw,page,nc", [(1, 1, 17, 48, 0), (1, 3, 11, 5, 1), (2, 5, 5, 16, 1)])
def test_f32_infinite_value_in_the_last_row(head_dim, fpb, gh, gw, page, nc):
    w = W.small_variant(W.CONFIGS["c1_tiny_f32"], heads=2, grid_h=gh, grid_w=gw, frames_per_block=fpb, head_dim=head_dim,
                        rope_dims=DIMS[head_dim], page_tokens=page, n_cached=nc, n_inflight=1)
    q, k, v = W.draw_config(w, seed=5)
    v[w.block_tokens - 1, 1, 3] = np.inf
    pool = Hn.gpu_setup(w, k, v, list(range(nc)), [nc])
    out = Hn.gpu_forward(w, pool, q, [nc], BI)
    assert (out[:, 1, 3] == np.inf).all()
    v[w.block_tokens - 1, 1, 3] = 0
    out[:, 1, 3] = 0
    ref = np.concatenate(Hn.oracle_forward(w, q, k, v, list(range(nc)), [nc], BI))
    ref[:, 1, 3] = 0
    Hn.assert_close(out, ref, "f32", f"infinite V D={head_dim} L={w.block_tokens} page={page}")


def _minus_infinity_scores(w, seed, low, high):
    """q, k, v whose scores are minus infinity in fp32 for the keys low <= n < high of block 0 and ordinary for all others: block 0 is at
    frame 0, where pairs of the frame axis are not rotated, and the slowest of them hardly turns at frame 1."""
    q, k, v = (W.to_f64(x).astype(np.float32) for x in W.draw_config(w, seed=seed))
    j = w.rope_dims[0] - 2
    q[:, :, j:j + 2] = k[:, :, j:j + 2] = 0
    q[:, :, j] = 1e10
    k[low:high, :, j] = -3e38
    return tuple(W.store(x, w.dtype) for x in (q, k, v))


# fp32 attention, scores of minus infinity (a product out of range) over the whole first tile of some of a workgroup's
# waves: weight 0
@pytest.mark.parametrize("head_dim", [32, 64, 128])
@pytest.mark.parametrize("low,high", [(5, 300), (16, 17), (16, 100), (0, 300)])
def test_f32_scores_of_minus_infinity(head_dim, low, high):
    w = W.small_variant(W.CONFIGS["c1_tiny_f32"], heads=2, grid_h=15, grid_w=20, frames_per_block=1, head_dim=head_dim,
                        rope_dims=DIMS[head_dim], page_tokens=48, n_cached=1, n_inflight=1)
    q, k, v = _minus_infinity_scores(w, 5, low, high)
    pool = Hn.gpu_setup(w, k, v, [0], [1])
    out = Hn.gpu_forward(w, pool, q, [1], BI)
    ref = np.concatenate(Hn.oracle_forward(w, q, k, v, [0], [1], BI))
    Hn.assert_close(out, ref, "f32", f"-inf scores D={head_dim} keys {low}..{high}")


# bf16 attention of launches that leave CUs idle: every KV walk cut into page ranges.  One item in as many
# ranges as it has pages (the last one ragged), items absent on some XCDs, walks of different lengths
# (block-causal) in ranges that begin and end inside blocks.
@pytest.mark.parametrize("heads,gh,gw,nc,ni", [(1, 4, 11, 1, 1), (1, 9, 10, 3, 1), (3, 9, 13, 1, 3), (9, 5, 9, 5, 1), (2, 20, 30, 0, 2)])
def test_bf16_split_small_launch(heads, gh, gw, nc, ni):
    w = W.small_variant(W.CONFIGS["c3_wan1p3b_cascade5"], heads=heads, grid_h=gh, grid_w=gw, n_cached=nc, n_inflight=ni)
    cached, infl = list(range(nc)), list(range(nc, nc + ni))
    q, k, v = W.draw_config(w, seed=6)
    pool = Hn.gpu_setup(w, k, v, cached, infl)
    for mode in (BI, CA):
        pool.pool[pool.pool.numel() - (256 * 256 * 132 * 4):].fill_(0xFF)       # partial results start as NaN
        out = Hn.gpu_forward(w, pool, q, infl, mode)
        ref, bound = (np.concatenate(x) for x in Hn.oracle_forward_bounded(w, q, k, v, cached, infl, mode))
        Hn.assert_close(out, ref, "bf16", f"split heads={heads} grid={gh}x{gw} nc={nc} ni={ni} mode={mode}", bound=bound)


# The same with enough ranges of ten pages or more for the 16x16x32 loop (208 to 234 workgroups on 256 CUs): 26 items
# of 96 pages in eight ranges each, 52 of 63 and 66 pages in four, 39 of 66 in six.  Queries rotated before and by the
# kernel.
@pytest.mark.parametrize("nc,ni,mode", [(31, 1, BI), (20, 2, CA), (20, 2, BI)])
def test_bf16_split_launch_that_fills_the_chip(nc, ni, mode):
    w = W.small_variant(W.CONFIGS["c5_wan1p3b_rollout"], heads=13, grid_h=6, grid_w=43, frames_per_block=1, n_cached=nc, n_inflight=ni,
                        sink_blocks=0, window_blocks=nc, max_inflight=ni)
    cached, infl = list(range(nc)), list(range(nc, nc + ni))
    q, k, v = W.draw_config(w, seed=16)
    pool = Hn.gpu_setup(w, k, v, cached, infl)
    heads = [0, 7, 12]
    ref, bound = (np.concatenate(x) for x in Hn.oracle_forward_bounded(w, q, k, v, cached, infl, mode, heads=heads))
    for form in (Hn.gpu_forward, Hn.gpu_forward_rope):
        pool.pool[pool.pool.numel() - (256 * 256 * 132 * 4):].fill_(0xFF)       # partial results start as NaN
        out = form(w, pool, q, infl, mode)
        assert np.isfinite(out).all()
        Hn.assert_close(out[:, heads], ref, "bf16", f"cut launch on many workgroups nc={nc} ni={ni} mode={mode} {form.__name__}", bound=bound)


# What launches of more than one round leave for the last: 8 of 264 items in eleven ranges of one or two pages, 24 of 280 in four, 16 of
# 272 in nine.  Each of an XCD's first heads has none of these items, its last one has.
@pytest.mark.parametrize("heads,gh,gw,nc,ni", [(24, 20, 43, 0, 1), (40, 15, 9, 0, 4), (16, 21, 33, 0, 2)])
def test_bf16_split_last_round(heads, gh, gw, nc, ni):
    w = W.small_variant(W.CONFIGS["c3_wan1p3b_cascade5"], heads=heads, grid_h=gh, grid_w=gw, n_cached=nc, n_inflight=ni)
    cached, infl = list(range(nc)), list(range(nc, nc + ni))
    q, k, v = W.draw_config(w, seed=8)
    pool = Hn.gpu_setup(w, k, v, cached, infl)
    some = [0, heads // 8 - 1, heads - 1]
    ref, bound = (np.concatenate(x) for x in Hn.oracle_forward_bounded(w, q, k, v, cached, infl, BI, heads=some))
    pool.pool[pool.pool.numel() - (256 * 256 * 132 * 4):].fill_(0xFF)       # partial results start as NaN
    print(f"last round heads={heads} grid={gh}x{gw}", flush=True)
    out = Hn.gpu_forward(w, pool, q, infl, BI)
    assert np.isfinite(out).all()
    Hn.assert_close(out[:, some], ref, "bf16", f"last round heads={heads} grid={gh}x{gw}", bound=bound)


# Tiles of the linear map: one row, a tile and one row, column counts that end inside a tile, the shortest and
# longer walks over k, several tiles per band and XCD.  (Two stages are fewer than any ring holds.)
@pytest.mark.parametrize("M,N,K", [(1, 8, 128), (65, 72, 128), (129, 200, 768), (1100, 1400, 256), (2050, 1160, 128), (1345, 3000, 256),
                                   (1300, 4104, 128), (4680, 1544, 384), (9001, 136, 1024), (4100, 4104, 128)])
def test_linear_tiles(M, N, K):
    import torch
    from paper_2511_20426_amd.runner import linear
    x, w = W.draw_linear(M, N, K, seed=M + N)
    yt = torch.full((M + 2, N + 8), 7.0, dtype=torch.bfloat16, device="cuda:0")
    print(f"linear tiles {M}x{N}x{K}", flush=True)
    linear(Hn.to_torch(x, "bf16"), Hn.to_torch(w, "bf16"), out=yt[:M, :N])
    torch.cuda.synchronize()
    got = Hn.from_torch(yt, "bf16")
    assert (got[M:] == 7.0).all() and (got[:, N:] == 7.0).all()
    # one rounding to bf16 and fp32 accumulation: half an ulp is 2^-9 relative, 2^-8 and 1e-5 of sum |x||w| allowed
    rows = np.unique(np.concatenate([np.arange(0, M, max(1, M // 300)), [M - 1]]))
    xf, wf = W.to_f64(x[rows]), W.to_f64(w)
    ref = orc.layer_linear(xf, wf)
    bound = np.abs(ref) * 2.0 ** -8 + 1e-5 * orc.layer_linear(np.abs(xf), np.abs(wf)) + 1e-30
    assert (np.abs(got[rows, :N].astype(np.float64) - ref) <= bound).all(), f"linear {M}x{N}x{K}"


# The publishing projection in each of its tiles writes the bytes that projection and cache write do: blocks of one page,
# a ragged page, an odd number of pages (256-row tiles whose second page does not exist).
@pytest.mark.parametrize("heads,fpb,gh,gw,ids,k_in", [(2, 1, 4, 8, (1,), 128), (2, 3, 13, 17, (0, 1, 2), 256), (4, 3, 19, 27, (2, 3), 128),
                                                      (24, 3, 10, 12, (0, 1, 2), 128), (12, 3, 30, 52, (4,), 256)])
def test_publish_tiles(heads, fpb, gh, gw, ids, k_in):
    import torch
    from paper_2511_20426_amd.runner import CascadePool, linear
    w = W.small_variant(W.CONFIGS["c3_wan1p3b_cascade5"], heads=heads, frames_per_block=fpb, grid_h=gh, grid_w=gw)
    L, n, width = w.block_tokens, len(ids) * w.block_tokens, heads * 128
    x, wq = W.draw_linear(n, 3 * width, k_in, seed=17)
    xt, wt = Hn.to_torch(x, "bf16"), Hn.to_torch(wq, "bf16")
    two, one = CascadePool.for_workload(w), CascadePool.for_workload(w)
    pages = two.pool.numel() - (256 * 256 * 132 * 4)
    two.pool.fill_(0xAB); one.pool.fill_(0xAB)
    print(f"publish tiles heads={heads} L={L} blocks={ids} k_in={k_in}", flush=True)
    qkv = linear(xt, wt).view(n, 3, heads, 128)
    ts = [250] * len(ids)
    two.append_batch(list(ids), ts, 1, [qkv[i * L:(i + 1) * L, 1] for i in range(len(ids))],
                     [qkv[i * L:(i + 1) * L, 2] for i in range(len(ids))])
    q = one.qkv_publish(xt, wt, list(ids), ts, 1)
    torch.cuda.synchronize()
    assert torch.equal(q.view(torch.int16), qkv[:, 0].contiguous().view(torch.int16))
    assert torch.equal(one.pool[:pages], two.pool[:pages])


# ... more of them, plain (last row and column tiles of one row and of a few columns) and publishing (pages of one
# token).
@pytest.mark.parametrize("M,N,K", [(1921, 2200, 256), (2881, 2824, 128), (2900, 2896, 384)])
def test_linear_tall_tiles(M, N, K):
    test_linear_tiles(M, N, K)


@pytest.mark.parametrize("heads,gh,gw,k_in", [(4, 19, 27, 128), (6, 13, 20, 384)])
def test_publish_tall_tiles(heads, gh, gw, k_in):
    test_publish_tiles(heads, 1, gh, gw, (1, 2, 3, 4, 5), k_in)


# Every kernel by name (the cost models may send the products above elsewhere), assembly loops by their rows: last row and column
# tiles of one row and eight columns, the shortest walk and a longer one; 256 rows also with a short last round of 6 and of 18
# tiles behind six whole ones.
LINEAR_TILES = [(256, 769, 13064, 128), (256, 4097, 3592, 768), (256, 65537, 1288, 512), (256, 66049, 1288, 512),
                (192, 1537, 4872, 128), (192, 2881, 2824, 384), (128, 513, 11016, 128), (128, 1025, 3720, 128),
                ("kTile256x128", 16385, 264, 128), ("kTile256x128", 4680, 1544, 384), ("kTile128", 2050, 1160, 128),
                ("kTile64", 1100, 1400, 256), ("kTile64Wide", 129, 200, 768)]


@pytest.mark.parametrize("tile,M,N,K", LINEAR_TILES)
def test_linear_tile_by_name(tile, M, N, K):
    assert Hn.linear_kernel(M, N, K) == tile
    test_linear_tiles(M, N, K)


# ... and publishing: blocks whose last page has one to four tokens, an odd number of pages; 256 x 256 dealt evenly
# and (8 heads, 420 tiles) by blocks.
PUBLISH_TILES = [("kTile256", 18, 10, 13, 5, 128), ("kTile256", 8, 57, 27, 5, 128), ("kTile128x256", 16, 13, 20, 3, 128), ("kTile256x128", 4, 19, 27, 5, 128),
                 ("kTile128", 2, 13, 51, 3, 256)]


@pytest.mark.parametrize("tile,heads,gh,gw,blocks,k_in", PUBLISH_TILES)
def test_publish_tile_by_name(tile, heads, gh, gw, blocks, k_in):
    assert Hn.publish_tile(blocks * gh * gw, 3 * heads * 128, k_in, gh * gw) == tile
    test_publish_tiles(heads, 1, gh, gw, tuple(range(1, 1 + blocks)), k_in)


# The cache write in workgroups of a page, half a page or a quarter of one (by pages x heads of the launch): all
# blocks in one launch and one by one, which take different ones but for the first (40 and 10 pages a quarter; 400 a
# page and 100 a quarter, 260 a half and 65 a quarter, 480 a page and 120 a quarter, 600 a half and 150 a quarter, 880
# a page and 220 a half), write the same bytes, padding and swizzle included; the smallest is compared with the oracle
# elsewhere.
@pytest.mark.parametrize("heads,gh,gw", [(5, 11, 23), (50, 11, 23), (13, 21, 27), (20, 21, 31), (30, 20, 32), (44, 20, 32)])
def test_cache_write_workgroup_sizes(heads, gh, gw):
    import torch
    from paper_2511_20426_amd.runner import CascadePool
    w = W.small_variant(W.CONFIGS["c3_wan1p3b_cascade5"], heads=heads, frames_per_block=1, grid_h=gh, grid_w=gw)
    gen = torch.Generator(device="cuda:0").manual_seed(6)
    ks, vs = ([torch.randn((w.block_tokens, heads, 128), generator=gen, device="cuda:0").to(torch.bfloat16) for _ in range(4)] for _ in range(2))
    two, one = CascadePool.for_workload(w), CascadePool.for_workload(w)
    two.pool.fill_(0xAB); one.pool.fill_(0xAB)
    two.append_batch([1, 2, 3, 4], [250] * 4, 0, ks, vs)
    for i in range(4):
        one.append(1 + i, 250, 0, ks[i], vs[i])
    pages = two.pool.numel() - (256 * 256 * 132 * 4)
    assert torch.equal(one.pool[:pages], two.pool[:pages])


# Queries rotated by the attention kernel: cos and sin from a table in LDS per tile.  Many frames and rows to a tile,
# one row or column, a tile that begins in the middle of a frame and goes round its end, the widest grid whose table
# fits (171 columns do not always: their lanes evaluate their own), axes without pairs, query blocks that are not
# consecutive.
@pytest.mark.parametrize("fpb,gh,gw,dims,infl", [(40, 1, 7, (44, 42, 42), (2, 3)), (3, 29, 3, (44, 42, 42), (2, 5)), (2, 9, 31, (44, 42, 42), (2, 3)),
                                                 (1, 2, 140, (44, 42, 42), (2, 3)), (1, 2, 171, (44, 42, 42), (2, 4)), (300, 1, 1, (44, 42, 42), (2,)),
                                                 (2, 11, 13, (0, 64, 64), (2, 3)), (2, 11, 13, (64, 64, 0), (2, 3)), (2, 11, 13, (126, 0, 2), (2, 3))])
def test_bf16_rotation_table(fpb, gh, gw, dims, infl):
    w = W.small_variant(W.CONFIGS["c3_wan1p3b_cascade5"], heads=2, grid_h=gh, grid_w=gw, frames_per_block=fpb, rope_dims=dims, n_cached=2,
                        n_inflight=len(infl), window_blocks=6)
    rng = np.random.default_rng(4)
    L, H, D = w.block_tokens, w.heads, w.head_dim
    q, k, v = (W.store(rng.standard_normal((n, H, D), dtype=np.float32), "bf16") for n in (len(infl) * L, (2 + len(infl)) * L, (2 + len(infl)) * L))
    print(f"rotation table {fpb} x {gh} x {gw} {dims}", flush=True)
    pool = Hn.gpu_setup(w, k, v, [0, 1], list(infl))
    import torch
    for mode in (BI, CA):
        got = Hn.gpu_forward_rope(w, pool, q, list(infl), mode)
        # the same rows through rope3d_apply, block by block, and the forward on rotated queries: two roundings of Q
        # for one
        qt = Hn.to_torch(q, "bf16")
        rot = torch.cat([pool.rope(qt[i * L:(i + 1) * L], fpb * g) for i, g in enumerate(infl)])
        ref = Hn.from_torch(pool.forward(rot, list(infl), mode), "bf16")
        assert np.isfinite(got).all() and Hn.rel_l2(got, ref) < 8e-3, (fpb, gh, gw, dims, mode, Hn.rel_l2(got, ref))


# Queries rotated by the attention kernel are scaled by log2(e) / sqrt(D) behind the rotation: a pair that the
# rotation takes out of fp32's range is infinite there as it is in rope3d_apply, and its row NaN, since K is zero in
# that pair.  With the table of angles and without.
@pytest.mark.parametrize("gh,gw", [(3, 5), (1, 200)])
def test_bf16_rotation_out_of_range(gh, gw):
    w = W.small_variant(W.CONFIGS["c3_wan1p3b_cascade5"], heads=2, grid_h=gh, grid_w=gw, frames_per_block=1, n_cached=1, n_inflight=1)
    q, k, v = (W.to_f64(x).astype(np.float32) for x in W.draw_config(w, seed=8))
    k[:, :, :2] = 0
    q[3, 1, :2] = q[11, 0, :2] = 3e38                        # pair 0 turns by 1 rad at frame 1: 3e38 (sin 1 + cos 1) = 4.1e38
    q, k, v = (W.store(x, "bf16") for x in (q, k, v))
    pool = Hn.gpu_setup(w, k, v, [0], [1])
    two, one = Hn.gpu_forward(w, pool, q, [1], BI), Hn.gpu_forward_rope(w, pool, q, [1], BI)
    want = np.ones(two.shape, bool)
    want[3, 1] = want[11, 0] = False
    assert (np.isfinite(two) == want).all() and (np.isfinite(one) == want).all()
    assert Hn.rel_l2(one[want], two[want]) < 8e-3


# bf16 attention on the 16x16x32 instruction (launches of many workgroups and ten pages or more): every class of ragged
# last page, blocks that begin inside a step, rows past the last query; two heads checked whole.
@pytest.mark.parametrize("gh,gw,nc", [(3, 43, 4), (3, 53, 4), (10, 16, 4), (7, 23, 4), (12, 16, 4), (223, 1, 4), (14, 16, 4), (15, 15, 4),
                                      (15, 17, 5), (16, 16, 4), (1, 40, 14)])
def test_bf16_many_workgroups(gh, gw, nc):
    w = W.small_variant(W.CONFIGS["c5_wan1p3b_rollout"], heads=181, grid_h=gh, grid_w=gw, frames_per_block=1, n_cached=nc, n_inflight=1,
                        sink_blocks=0, window_blocks=16)
    cached, infl = list(range(nc)), [nc]
    q, k, v = W.draw_config(w, seed=8)
    print(f"many workgroups L={w.block_tokens}", flush=True)
    pool = Hn.gpu_setup(w, k, v, cached, infl)
    heads = [0, 180]
    ref, bound = (np.concatenate(x) for x in Hn.oracle_forward_bounded(w, q, k, v, cached, infl, BI, heads=heads))
    Hn.assert_close(Hn.gpu_forward(w, pool, q, infl, BI)[:, heads], ref, "bf16", f"many workgroups L={w.block_tokens}", bound=bound)


# ... and on few workgroups: last pages of 1 .. 64 tokens, of which half the steps are walked, and one token more;
# blocks of one such page only; walks cut in front of, behind and between them; the reference moving beside a masked
# tile.
@pytest.mark.parametrize("heads,gh,gw,nc,ni,scale", [(1, 8, 8, 4, 1, 1), (2, 3, 11, 2, 3, 1), (1, 3, 43, 3, 1, 1), (3, 10, 16, 2, 2, 1), (2, 7, 23, 3, 1, 4),
                                                     (1, 12, 16, 4, 2, 1), (2, 5, 13, 3, 2, 1), (1, 1, 1, 5, 1, 1)])
def test_bf16_short_last_pages(heads, gh, gw, nc, ni, scale):
    w = W.small_variant(W.CONFIGS["c3_wan1p3b_cascade5"], heads=heads, grid_h=gh, grid_w=gw, frames_per_block=1, n_cached=nc, n_inflight=ni,
                        window_blocks=6)
    cached, infl = list(range(nc)), list(range(nc, nc + ni))
    q, k, v = W.draw_config(w, seed=18, scale=0.5 * scale)
    pool = Hn.gpu_setup(w, k, v, cached, infl)
    for mode in (BI, CA):
        ref, bound = (np.concatenate(x) for x in Hn.oracle_forward_bounded(w, q, k, v, cached, infl, mode))
        print(f"short pages L={w.block_tokens} mode={mode}", flush=True)
        Hn.assert_close(Hn.gpu_forward(w, pool, q, infl, mode), ref, "bf16", f"short last pages L={w.block_tokens} mode={mode}", bound=bound,
                        **({} if scale == 1 else {"max_abs": 0.12, "rel": 1.2e-2}))


# ... and its moving exponent reference: rising, falling, past the fp32 exponent range, from one key to the next.  The
# bars are those of the same ramps on few workgroups (the bf16 rounding of K moves logits of 25 by 5e-2, of 400 by
# 0.8).
@pytest.mark.parametrize("ramp,bar", [((1.0, 24.0), 2e-2), ((24.0, 1.0), 2e-2), ((1.0, 400.0), 8e-2), ((1.0, 400.0, "step"), 8e-2)])
@pytest.mark.parametrize("gw", [13, 15])                     # with short last pages and without
def test_bf16_many_workgroups_moving_maximum(ramp, bar, gw):
    w = W.small_variant(W.CONFIGS["c3_wan1p3b_cascade5"], heads=90, grid_h=10, grid_w=gw, n_cached=2, n_inflight=1)
    q, k, v = W.draw_config(w, seed=31, k_ramp=ramp)
    pool = Hn.gpu_setup(w, k, v, [0, 1], [2])
    heads = [0, 89]
    got = Hn.gpu_forward(w, pool, q, [2], BI)
    ref = np.concatenate(Hn.oracle_forward(w, q, k, v, [0, 1], [2], BI, heads=heads))
    assert np.isfinite(got).all()
    Hn.assert_close(got[:, heads], ref, "bf16", f"many workgroups, ramp {ramp}", max_abs=bar * float(np.abs(ref).max()) * 4, rel=bar)


# One eager call of any size readies the others for capture: products of several tiles and a forward of each loop recorded
# after small eager calls, replayed three times on new inputs.
def test_capture_of_other_sizes_than_the_eager_call():
    import torch
    from paper_2511_20426_amd.runner import CascadePool, linear
    gen = torch.Generator(device="cuda:0").manual_seed(3)

    def draw(*shape):
        return (torch.randn(shape, generator=gen, device="cuda:0") * 0.3).to(torch.bfloat16)

    linear(draw(8, 128), draw(8, 128))
    xs = [(draw(m, k), draw(n, k), torch.empty((m, n), dtype=torch.bfloat16, device="cuda:0"))
          for m, n, k in ((1100, 1400, 256), (1300, 4104, 128), (4100, 4104, 128))]
    small, large = (CascadePool.for_workload(W.small_variant(W.CONFIGS["c3_wan1p3b_cascade5"], heads=h, grid_h=10, grid_w=13, n_cached=2,
                                                             n_inflight=1)) for h in (2, 90))
    for p in (small, large):
        for g in range(3):
            p.append(g, 0, 0, draw(390, p.heads, 128), draw(390, p.heads, 128))
            if g < 2:
                p.ctx.kv_cache_promote(g)
    small.forward_rope(draw(390, 2, 128), [2], BI)
    q, o = draw(390, 90, 128), torch.empty((390, 90, 128), dtype=torch.bfloat16, device="cuda:0")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for x, w, y in xs:
            linear(x, w, out=y)
        large.forward_rope(q, [2], BI, out=o)
    for _ in range(3):
        for x, _w, y in xs:
            x.copy_(draw(*x.shape))
            y.zero_()
        q.copy_(draw(*q.shape))
        o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for x, w, y in xs:
            assert torch.equal(linear(x, w), y)
        assert torch.equal(large.forward_rope(q, [2], BI), o)


# Row sums are those of the probabilities before their rounding to bf16, in both main loops.  One key of weight 0.9
# outside a walk's first tile, its V zero, the others' 1 +- 0.3: a rounded weight in the row sum scales the whole row
# by up to 0.9 x 2^-8.  The reference takes the kernel's own operands (Q scaled and rounded, K as its pages hold it),
# so that a row's mean ratio to it keeps, of relative variance E2 each, the rounding of 128 results and of the light
# keys' weights: bars at 8 sigma a row, 2 sigma over the rows.
@pytest.mark.parametrize("heads", [2, 181])
def test_bf16_row_sums_with_one_heavy_key(heads):
    w = W.small_variant(W.CONFIGS["c5_wan1p3b_rollout"], heads=heads, grid_h=10, grid_w=15, frames_per_block=1, n_cached=4, n_inflight=1,
                        sink_blocks=0, window_blocks=16)
    L, blocks, heavy = w.block_tokens, 5, 2 * w.block_tokens + 37
    rng = np.random.default_rng(12)
    _, k, v = W.draw_config(w, seed=9)
    u = np.sign(rng.standard_normal(128))
    q = W.f32_to_bf16_bits((u + 0.1 * rng.standard_normal((L, heads, 128))).astype(np.float32))
    at = orc.token_positions(2, w.frames_per_block, w.grid_h, w.grid_w)[37:38]
    flip = np.tile([1.0, -1.0], 64)                                  # the rotation by the opposite angle
    k[heavy] = W.f32_to_bf16_bits((orc.rope3d((0.8 * u * flip)[None, None], at, w.rope_dims, w.rope_theta)[0, 0] * flip).astype(np.float32))
    v[:] = W.f32_to_bf16_bits((1 + 0.3 * rng.standard_normal(v.shape)).astype(np.float32))
    v[heavy] = 0
    pool = Hn.gpu_setup(w, k, v, [0, 1, 2, 3], [4])
    print(f"one heavy key, {heads} heads", flush=True)
    out = Hn.from_torch(pool.forward(Hn.to_torch(q, "bf16"), [4], BI), "bf16")
    raw = pool.pool.cpu().numpy()
    c = np.float32(1.4426950408889634) / np.sqrt(np.float32(128))
    for h in (0, heads - 1):
        kp = np.concatenate([W.to_f64(np.concatenate([Hn.decode_bf16_pages(raw, pool.ctx.kv_cache_page_index(g, pg, h))[0]
                                                      for pg in range(2)])[:L]) for g in range(blocks)])
        p = np.exp2(W.to_f64(W.f32_to_bf16_bits(W.bf16_bits_to_f32(q[:, h]) * c)) @ kp.T)
        p /= p.sum(axis=1, keepdims=True)
        assert 0.8 < p[:, heavy].min()
        err = (out[:, h] / (p @ W.to_f64(v[:, h])) - 1).mean(axis=1)
        light = np.delete(p, heavy, axis=1)
        sigma = np.sqrt(Hn.E2_BF16 * (1 / 128 + (light ** 2).sum(axis=1) / light.sum(axis=1) ** 2))
        print(f"[row sums] {heads} heads, head {h}: rms {np.sqrt((err ** 2).mean()):.2e} max {np.abs(err).max():.2e} sigma {sigma.mean():.2e}", flush=True)
        assert (np.abs(err) <= 8 * sigma).all() and np.sqrt((err ** 2).mean()) <= 2 * sigma.mean()


# Scores of minus infinity over the whole first tile of a range of a cut walk (one head: every page a range), and of a
# walk: weight 0 (181 heads: one range an item, the 16x16x32 loop).
@pytest.mark.parametrize("heads", [1, 181])
@pytest.mark.parametrize("low,high", [(5, 600), (32, 257), (0, 600), (0, 32)])
def test_bf16_scores_of_minus_infinity(heads, low, high):
    w = W.small_variant(W.CONFIGS["c5_wan1p3b_rollout"], heads=heads, grid_h=20, grid_w=30, frames_per_block=1, n_cached=1, n_inflight=1,
                        sink_blocks=0, window_blocks=16)
    q, k, v = _minus_infinity_scores(w, 5, low, high)
    print(f"-inf scores {heads} heads keys {low}..{high}", flush=True)
    pool = Hn.gpu_setup(w, k, v, [0], [1])
    check = sorted({0, heads - 1})
    got = Hn.gpu_forward(w, pool, q, [1], BI)[:, check]
    ref = np.concatenate(Hn.oracle_forward(w, q, k, v, [0], [1], BI, heads=check))
    Hn.assert_close(got, ref, "bf16", f"-inf scores {heads} heads keys {low}..{high}")


def test_mfma_microbench_on_the_smaller_instruction():
    """16x16x32: below the nominal peak and above half of it; zero operands are not slower than random ones."""
    import torch
    from paper_2511_20426_amd import binding as B
    probe = torch.empty(1 << 16, dtype=torch.uint8, device="cuda:0")
    rnd, zer = (B.mfma_microbench(16 + k, 20000, probe.data_ptr(), probe.numel(), torch.cuda.current_stream().cuda_stream) for k in (1, 0))
    print(f"mfma only, 16x16x32: random {rnd[0]:.0f} TFLOP/s at {rnd[1]:.2f} GHz, zeros {zer[0]:.0f} TFLOP/s at {zer[1]:.2f} GHz", flush=True)
    for t, c in (rnd, zer):
        assert 1000.0 < t < 2600.0 and 1.0 < c < 2.6
    assert zer[0] > 0.95 * rnd[0]
    with pytest.raises(B.CascadeAttnError):
        B.mfma_microbench(18, 10, probe.data_ptr(), probe.numel(), 0)
