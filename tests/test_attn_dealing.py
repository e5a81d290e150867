"""How the work items of the bf16 attention are shared out to the eight XCDs: columns and segments that eight does not divide."""
import numpy as np
import pytest

import workloads as W
from oracle import cascade_oracle as orc
from tests import _harness as Hn


def _item(items, n_seg, xcd, item):
    """decode_item: segment and column, or None."""
    (first, first_segs), (to, to_segs) = divmod(xcd * items // 8, n_seg), divmod((xcd + 1) * items // 8, n_seg)
    seg, col, end = 0, first + (first_segs > 0) + item, to + (to_segs > 0)
    while col >= end:
        seg += 1
        if seg == n_seg:
            return None
        col += first + (seg < first_segs) - end
        end = to + (seg < to_segs)
    return seg, col


@pytest.mark.parametrize("n_seg", range(1, 9))
def test_every_item_once_and_longest_walks_first(n_seg):
    for cols in [*range(1, 41), 60, 228, 460, 3680]:
        items, seen = cols * n_seg, []
        for xcd in range(8):
            own = [_item(items, n_seg, xcd, i) for i in range((items + 7) // 8)]
            n = (xcd + 1) * items // 8 - xcd * items // 8
            assert None not in own[:n] and own[n:] in ([], [None]) and own[:n] == sorted(own[:n])
            seen += own[:n]
        assert sorted(seen) == [(s, c) for s in range(n_seg) for c in range(cols)]


@pytest.mark.gpu
@pytest.mark.parametrize("heads,gh,gw,inflight", [(1, 4, 5, 1), (1, 4, 5, 5), (1, 11, 13, 3), (3, 11, 13, 5), (5, 9, 10, 2), (9, 11, 13, 5), (12, 7, 13, 4),
                                                  (15, 11, 13, 5)])
def test_columns_that_eight_does_not_divide(heads, gh, gw, inflight):
    w = W.small_variant(W.CONFIGS["c3_wan1p3b_cascade5"], heads=heads, grid_h=gh, grid_w=gw, n_cached=2, n_inflight=inflight)
    q, k, v = W.draw_config(w, seed=heads + inflight)
    ids = list(range(2, 2 + inflight))
    print(f"heads {heads} grid {gh} x {gw} blocks {inflight}", flush=True)
    pool = Hn.gpu_setup(w, k, v, [0, 1], ids)
    for mode in (orc.BIDIRECTIONAL, orc.BLOCK_CAUSAL):
        out = Hn.gpu_forward(w, pool, q, ids, mode)
        ref, bound = (np.concatenate(x) for x in Hn.oracle_forward_bounded(w, q, k, v, [0, 1], ids, mode))
        Hn.assert_close(out, ref, "bf16", f"mode {mode}", bound=bound)
