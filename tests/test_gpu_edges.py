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
