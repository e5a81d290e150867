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


def _ranges(cols, n_seg, longest, ppb, cus=32):
    """ranges_of_idle_launch: pages of a range and workgroups of an XCD, or None."""
    work, best = (cols * n_seg + 7) // 8, (40 * longest * ppb, None)
    pages = [(longest - i) * ppb for i in range(n_seg)]
    for s in range(2, min(16, pages[0]) + 1):
        r = -(-pages[0] // s)
        n = [-(-p // r) for p in pages]
        groups = work // n_seg * sum(n) + sum(n[:work % n_seg])
        if n[0] == s and groups <= cus:
            best = min(best, (40 * (r + 1) + 8 * groups, (r, groups)), key=lambda b: b[0])
    return best[1]


@pytest.mark.parametrize("n_seg", range(2, 9))
def test_every_page_in_one_range(n_seg):
    """A workgroup's item and pages as attn_bf16_kernel finds them, and where merge_partials_kernel looks for its result."""
    cut = 0
    for cols in range(1, 256 // n_seg):
        for longest in (n_seg, n_seg + 2, n_seg + 7):
            for ppb in (1, 3, 13):
                plan, items = _ranges(cols, n_seg, longest, ppb), cols * n_seg
                if plan is None:
                    continue
                cut += 1
                (r, groups), pages = plan, [(longest - i) * ppb for i in range(n_seg)]
                segs = [sum(p > c * r for p in pages) for c in range(16)]
                found, slots = {}, {}
                for xcd in range(8):
                    own = (xcd + 1) * items // 8 - xcd * items // 8
                    seg_of = [_item(items, n_seg, xcd, i)[0] for i in range(own)]
                    count = [sum(s < n for s in seg_of) for n in segs]
                    assert sum(count) <= groups <= 32
                    for nth in range(groups):
                        item, c = nth, 0
                        while c < 16 and item >= count[c]:
                            item, c = item - count[c], c + 1
                        if c < 16:
                            seg, col = _item(items, n_seg, xcd, item)
                            found.setdefault((seg, col), []).append((c * r, min(c * r + r, pages[seg])))
                            slots[seg, col, c] = 32 * xcd + nth
                    for i in range(own):
                        seg, col = _item(items, n_seg, xcd, i)
                        assert all(slots[seg, col, c] == 32 * xcd + i + sum(count[:c]) for c in range(sum(n > seg for n in segs)))
                assert len(found) == items and len(set(slots.values())) == len(slots) and max(slots.values()) < 256
                assert all([x for lo, hi in f for x in range(lo, hi)] == list(range(pages[seg])) for (seg, _), f in found.items())
    assert cut > 20


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
