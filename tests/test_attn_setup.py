"""What a workgroup of the bf16 attention does ahead of its walk: scalar divisions and the table of angles, followed on the CPU, and on
the GPU for axes that end at every place of a lane's four pairs."""
import numpy as np
import pytest

import workloads as W
from oracle import cascade_oracle as orc
from tests import _harness as Hn

QUADS = (160 * 1024 - 4 * 32768 - 256 * 16) // 32          # of four pairs, that the LDS beside the page rings holds


def _div_by(n, d):
    q = n * ((1 << 32) // d if d > 1 else 0xffffffff) >> 32
    r = n - q * d
    return (q + 1, r - d) if r >= d else (q, r)


def test_division_by_launch_constants():
    rng = np.random.default_rng(0)
    for d in [1, 2, 3, 255, 256, 1560, 4680, 2 ** 22 - 1, 2 ** 31 - 1] + [int(x) for x in rng.integers(1, 2 ** 22, 3000)]:
        for n in [0, d - 1, d, 2 ** 31 - 1] + [int(x) for x in rng.integers(0, 2 ** 31, 20)]:
            assert _div_by(n, d) == divmod(n, d)
    # by a float reciprocal an ulp off, of half more than n
    for d in list(range(1, 4096, 7)) + [32768]:
        inv = np.float32(1) / np.float32(d)
        for x in (inv, np.nextafter(inv, np.float32(0)), np.nextafter(inv, np.float32(2))):
            for n in (0, d - 1, d, 2 * d - 1, 4351, 32767, 32768 // d * d):
                assert int(np.float32((np.float32(n) + np.float32(0.5)) * x)) == n // d


def _table(fpb, gh, gw, dims, first, row0, rows_end):
    """Whether a tile has a table; every place that its rows' lanes read holds the entry of that pair and value."""
    to_y, to_x, plane = dims[0] // 2, (dims[0] + dims[1]) // 2, gh * gw
    tab_f, tab_y, pairs_w = 256 // plane + 2, min(256 // gw + 2, gh), 64 - to_x
    of_t, of_y, of_x = (to_y + 3) // 4, (to_x + 3) // 4 - to_y // 4, 16 - to_x // 4
    quads = tab_f * of_t + tab_y * of_y + gw * of_x
    if quads > QUADS or (to_y < to_x < 64 and to_y // 4 == to_x // 4 and to_y % 4):
        return False
    (frame0, in_plane), last = divmod(row0, plane), (rows_end - 1) // plane
    y0, x0 = divmod(in_plane, gw)
    in_y, in_x = tab_f * of_t - to_y // 4, tab_f * of_t + tab_y * of_y - to_x // 4
    n_t, n_ty = tab_f * to_y, tab_f * to_y + tab_y * (to_x - to_y)
    table = {}
    for e in range(n_ty + gw * pairs_w):
        axis = 0 if e < n_t else (1 if e < n_ty else 2)
        val, k = divmod(e - (0, n_t, n_ty)[axis], (to_y, to_x - to_y, pairs_w)[axis])
        pair, frame = (0, to_y, to_x)[axis] + k, min(frame0 + val, last)
        value = (first[frame // fpb] + frame % fpb, y0 + val - (gh if y0 + val >= gh else 0), val)[axis]
        quad = (0, in_y, in_x)[axis] + val * (of_t, of_y, of_x)[axis] + pair // 4
        at = 16 * (quad + (quads if pair & 2 else 0)) + 8 * (pair & 1)
        assert 0 <= quad < quads and at not in table and at + 8 <= 32 * QUADS
        table[at] = (pair, axis, value)
    for tid in range(256):
        along = x0 + min(tid, rows_end - 1 - row0)
        down, x = divmod(along, gw)
        frames, y = divmod(y0 + down, gh)
        frame = frame0 + frames
        place = (16 * frames * of_t, 16 * (in_y + (y - y0 + (gh if y < y0 else 0)) * of_y), 16 * (in_x + x * of_x))
        axis_of = [0 if p < to_y else (1 if p < to_x else 2) for p in range(64)]
        for p in range(64):
            # with no axis that ends behind a lane's first pair, the reads of pairs 0 and 2 bring 1 and, but where the axis ends, 3
            by = p if to_y % 4 == 1 or to_x % 4 == 1 or p % 4 == 3 and axis_of[p] != axis_of[p - 1] else p & ~1
            at = 16 * (p // 4 + (quads if p & 2 else 0)) + 8 * (p & 1) + place[axis_of[by]]
            assert table[at] == (p, axis_of[p], (first[frame // fpb] + frame % fpb, y, x)[axis_of[p]])
    return True


@pytest.mark.parametrize("dims,some", [((44, 42, 42), True), ((42, 44, 42), True), ((42, 42, 44), True), ((46, 40, 42), True), ((64, 32, 32), True),
                                       ((0, 64, 64), True), ((64, 64, 0), True), ((126, 0, 2), True), ((2, 124, 2), True), ((124, 2, 2), False),
                                       ((60, 2, 66), False), ((2, 2, 124), False)])
def test_table_of_angles(dims, some):
    found = False
    for fpb, gh, gw in ((3, 10, 13), (3, 30, 52), (1, 1, 1), (2, 1, 60), (3, 60, 1), (1, 5, 7)):
        L = fpb * gh * gw
        for row0, end in [(r, 3 * L) for r in list(range(0, 3 * L, 256))[:3] + [3 * L - 3 * L % 256 - 256 if L > 200 else 0]] + [(L, 2 * L)]:
            found |= _table(fpb, gh, gw, dims, [100, 107, 140], row0, end)
    assert found == some


@pytest.mark.gpu
@pytest.mark.parametrize("dims", [(42, 44, 42), (42, 42, 44), (46, 40, 42), (64, 32, 32), (2, 124, 2), (124, 2, 2), (60, 2, 66)])
def test_axes_that_end_inside_a_lane(dims):
    """Queries rotated by the attention kernel against rope3d_apply and the forward on rotated queries (two roundings of Q for one)."""
    import torch
    fpb, gh, gw, infl = 2, 11, 13, (2, 4)
    w = W.small_variant(W.CONFIGS["c3_wan1p3b_cascade5"], heads=2, grid_h=gh, grid_w=gw, frames_per_block=fpb, rope_dims=dims, n_cached=2,
                        n_inflight=len(infl), window_blocks=6)
    rng = np.random.default_rng(6)
    L, H, D = w.block_tokens, w.heads, w.head_dim
    q, k, v = (W.store(rng.standard_normal((n, H, D), dtype=np.float32), "bf16") for n in (len(infl) * L, (2 + len(infl)) * L, (2 + len(infl)) * L))
    print(f"axes {dims}", flush=True)
    pool = Hn.gpu_setup(w, k, v, [0, 1], list(infl))
    for mode in (orc.BIDIRECTIONAL, orc.BLOCK_CAUSAL):
        got = Hn.gpu_forward_rope(w, pool, q, list(infl), mode)
        qt = Hn.to_torch(q, "bf16")
        rot = torch.cat([pool.rope(qt[i * L:(i + 1) * L], fpb * g) for i, g in enumerate(infl)])
        ref = Hn.from_torch(pool.forward(rot, list(infl), mode), "bf16")
        assert np.isfinite(got).all() and Hn.rel_l2(got, ref) < 8e-3, (dims, mode, Hn.rel_l2(got, ref))


@pytest.mark.gpu
@pytest.mark.parametrize("axis", range(3))
def test_a_pair_is_rotated_the_same_wherever_axes_end(axis):
    """The first pair of an axis turns by the position on it in every geometry.  With nothing else in Q and K the outputs are the same to
    the last bit, whichever of its lane's four pairs it is and whether their factors come from the table in pairs, one by
    one, or without a table: about one rotated value in 2^15 rounds the other way to bf16 if the two products of a rotation
    are joined in another order."""
    import torch
    from paper_2511_20426_amd.runner import CascadePool
    gen = torch.Generator(device="cuda:0").manual_seed(12)
    H, D, L = 12, 128, 3 * 30 * 52
    pairs = [torch.randn((n, H, 2), generator=gen, device="cuda:0").to(torch.bfloat16) for n in (2 * L, 3 * L)]
    v = torch.randn((3 * L, H, D), generator=gen, device="cuda:0").to(torch.bfloat16)
    outs = []
    for dims in ((44, 42, 42), (42, 44, 42), (42, 42, 44), (46, 40, 42), (40, 42, 46), (6, 60, 62), (124, 2, 2), (60, 2, 66)):
        w = W.small_variant(W.CONFIGS["c3_wan1p3b_cascade5"], heads=H, grid_h=30, grid_w=52, rope_dims=dims, n_cached=1, n_inflight=2)
        first = sum(dims[:axis])
        q, k = (torch.zeros((p.shape[0], H, D), dtype=torch.bfloat16, device="cuda:0") for p in pairs)
        q[..., first:first + 2], k[..., first:first + 2] = pairs
        print(f"axis {axis} of {dims}", flush=True)
        pool = CascadePool.for_workload(w)
        for i in range(3):
            pool.append(i, 0, 0, k[i * L:(i + 1) * L], v[i * L:(i + 1) * L])
            if i == 0:
                pool.ctx.kv_cache_promote(0)
        outs.append(pool.forward_rope(q, [1, 2], orc.BIDIRECTIONAL))
        print("rows that differ", int((outs[0] != outs[-1]).any(-1).sum()), flush=True)
    assert all(torch.equal(outs[0].view(torch.int16), o.view(torch.int16)) for o in outs[1:])
