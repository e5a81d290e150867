"""The linear maps in tiles of 256 columns (gen_gemm_rows.py, gemm_rows.hip): the generated program of a workgroup followed on the CPU
over several tiles, and products on the GPU against fp64."""
import importlib.util
import os
import re
import sys

import numpy as np
import pytest

import workloads as W
from oracle import cascade_oracle as orc
from tests import _harness as Hn

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_20426_amd", "csrc")


def _load(name):
    spec = importlib.util.spec_from_file_location(name, os.path.join(CSRC, name + ".py"))
    mod = sys.modules[name] = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


rows = _load("gen_gemm_rows")
X_AT, W_AT, Y_AT = 1 << 33, 5 << 34, 3 << 40
U32 = 0xffffffff


class _Lds:
    """What lies in each 16 bytes of LDS: (row of the operand, 16-byte chunk of it), who has it on its way, when it was read."""
    def __init__(self):
        n = 160 * 1024 // 16
        self.row, self.chunk, self.op = (np.full(n, -1) for _ in range(3))
        self.visible, self.read_at = np.zeros(n, bool), np.full(n, -1)


class _Wave:
    """One of the four waves of a workgroup: scalars as integers, vector registers as 64 integers, fragments and sums as what they hold."""
    def __init__(self, mt, wave, text, lds, shape, tiles, pad, form):
        M, N, K = shape
        self.mt, self.text, self.lds, self.shape, self.tiles, self.wave = mt, text, lds, shape, tiles, wave
        self.label = {ln[:-1]: k for k, ln in enumerate(text) if ln.endswith(":")}
        self.ldx, self.ldw, self.ldy = 2 * (K + 8 * pad), 2 * (K + 16 * pad), 2 * (N + 24 * pad)
        lane = np.arange(64, dtype=np.int64)
        l15, grp, wm, wn, rows_ = lane & 15, lane >> 4, wave & 1, wave >> 1, 32 * mt
        row, col = wm * 16 * mt + (l15 & 7), wn * 128 + 32 * (l15 >> 3) + 8 * grp
        at_list = np.minimum(lane, len(tiles) - 1)
        ylane, tile_y, row8 = row * self.ldy + col * 2, rows_ * self.ldy, 8 * self.ldy
        self.arg = {"x_lo": X_AT & U32, "x_hi": X_AT >> 32, "w_lo": W_AT & U32, "w_hi": W_AT >> 32, "y_lo": Y_AT & U32, "y_hi": Y_AT >> 32,
                    "tile_x": self.ldx * rows_, "tile_w": self.ldw * 256, "tile_y_lo": tile_y & U32, "tile_y_hi": tile_y >> 32,
                    "row8_lo": row8 & U32, "row8_hi": row8 >> 32, "ldw2": self.ldw, "ldx2": self.ldx, "M": M, "N": N, "n_stages": K // 64,
                    "tiles": len(tiles), "form": form, "wave": wave, "lds0": 0,
                    "list_m": np.array([t[0] for t in tiles])[at_list], "list_n": np.array([t[1] for t in tiles])[at_list],
                    "roww": wave * 64 + (lane >> 3), "rowx": wave * 8 * mt + (lane >> 3),
                    "chunkw": ((lane & 7) ^ ((lane >> 4) & 1)) * 16, "chunkx": ((lane & 7) ^ (lane >> 4)) * 16,
                    "aw0": (wn * 128 + 8 * (l15 >> 2) + (l15 & 3)) * 128 + ((grp ^ (l15 >> 1)) << 4),
                    "ax0": (wm * 16 * mt + l15) * 128 + ((grp ^ (l15 >> 1)) << 4), "row": row, "col": col,
                    "ylane_lo": ylane & U32, "ylane_hi": ylane >> 32}
        self.s, self.v, self.a = {}, {}, {}
        self.scc, self.m0, self.exec = 0, None, np.ones(64, bool)
        self.queue, self.flying, self.held, self.barriers, self.tile = [], [], {}, 0, 0
        self.written, self.written_at, self.forms = {}, {}, {}

    def val(self, x):
        x = x.strip()
        if x.startswith("%["):
            return self.arg[x[2:-1]]
        if x in ("vcc", "exec"):
            return self.s[x] if x == "vcc" else self.exec
        if re.fullmatch(r"v\d+", x):
            return self.v[int(x[1:])]
        if x.startswith("s["):
            a = int(x[2:].split(":")[0])
            return self.s[a] if isinstance(self.s[a], np.ndarray) else self.s[a] | self.s[a + 1] << 32
        if re.fullmatch(r"s\d+", x):
            return self.s[int(x[1:])]
        if "-" in x[1:]:
            p, q = x.split("-", 1)
            return self.label[p] - self.label[q]
        return int(x, 0) & U32

    def run(self):
        """up to each barrier"""
        signed = lambda u: u - (1 << 32) if u & 0x80000000 else u  # noqa: E731
        mt, (M, N, K), lds = self.mt, self.shape, self.lds
        per_tile, k, steps = 2 * (K // 64), 0, 0
        while k < len(self.text):
            ln = self.text[k]
            k, steps = k + 1, steps + 1
            assert steps < 200000
            if ln.endswith(":") or ln.startswith(";"):
                continue
            op, _, rest = ln.partition(" ")
            a = [x.strip() for x in re.split(r",(?![^\[]*\])", rest)]
            if op == "s_barrier":
                assert not self.flying, ln                    # its reads are done
                self.barriers += 1
                yield
            elif op == "s_getpc_b64":
                self.s[int(a[0][2:].split(":")[0])], self.s[int(a[0][2:].split(":")[0]) + 1] = k, 0
            elif op == "s_setpc_b64":
                k = self.val(a[0])
                assert self.text[k].endswith(":")
            elif op == "s_branch" or (op == "s_cbranch_scc1" and self.scc):
                k = self.label[a[0]]
            elif op.startswith("s_cmp_"):
                x, y = self.val(a[0]), self.val(a[1])
                self.scc = int({"eq": x == y, "lg": x != y, "lt": x < y, "ge": x >= y}[op.split("_")[2]])
            elif op == "s_and_b64":
                self.exec = self.val(a[1]) & self.val(a[2])
            elif op == "s_mov_b64":
                assert a == ["exec", "-1"]
                self.exec = np.ones(64, bool)
            elif op.startswith("s_") and op not in ("s_nop", "s_waitcnt", "s_cbranch_scc1"):
                x = self.val(a[1])
                y = self.val(a[2]) if len(a) > 2 else None
                if op in ("s_add_u32", "s_addc_u32"):
                    r = x + y + (self.scc if op == "s_addc_u32" else 0)
                    self.scc = r >> 32
                elif op in ("s_sub_u32", "s_subb_u32"):
                    r = x - y - (self.scc if op == "s_subb_u32" else 0)
                    self.scc = int(r < 0)
                else:
                    r = {"s_mov_b32": lambda: x, "s_mul_i32": lambda: x * y, "s_mul_hi_u32": lambda: (x * y) >> 32, "s_sub_i32": lambda: x - y,
                         "s_lshl_b32": lambda: x << y, "s_lshr_b32": lambda: x >> y, "s_min_u32": lambda: min(x, y), "s_and_b32": lambda: x & y,
                         "s_cselect_b32": lambda: x if self.scc else y}[op]()
                if a[0] == "m0":
                    self.m0 = r & U32
                else:
                    self.s[int(a[0][1:])] = r & U32
            elif op == "s_waitcnt":
                m = re.search(r"vmcnt\((\d+)\)", ln)
                if m:                                        # in order, loads and stores alike; what is behind may fly on
                    keep = int(m.group(1))
                    self.queue = self.queue[len(self.queue) - keep:] if keep else []
                m = re.search(r"lgkmcnt\((\d+)\)", ln)
                if m:
                    self.flying = self.flying[len(self.flying) - int(m.group(1)):] if int(m.group(1)) else []
            elif op == "v_readlane_b32":
                at = self.val(a[2])
                assert at < len(self.tiles)
                self.s[int(a[0][1:])] = int(self.val(a[1])[at])
            elif op == "v_cmp_gt_i32":
                r = np.broadcast_to(signed(self.val(a[1])) > self.val(a[2]), 64)
                self.s["vcc" if a[0] == "vcc" else int(a[0][2:].split(":")[0])] = r
            elif op == "global_load_lds_dwordx4":
                base, off = self.val(a[1]), self.val(a[0])
                assert (off >= 0).all() and (off < 1 << 31).all()
                addr, at = base + off, (self.m0 + 16 * np.arange(64)) // 16
                kind = int(base >= W_AT)
                rel, ld = addr - (W_AT if kind else X_AT), self.ldw if kind else self.ldx
                row, byte = rel // ld, rel % ld
                assert (rel >= 0).all() and (row < (N if kind else M)).all() and (byte + 16 <= 2 * K).all() and (byte % 16 == 0).all()
                assert (lds.read_at[at] < self.barriers).all()      # nobody reads what was there any more
                lds.row[at], lds.chunk[at], lds.op[at], lds.visible[at] = row, byte // 16, kind, False
                self.queue.append(at)
            elif op == "global_store_dwordx4":
                data = int(a[1][2:].split(":")[0])
                row0 = int(a[0][2:].split(":")[0])
                addr = self.v[row0] + (self.v[row0 + 1] << 32) + int(re.search(r"offset:(\d+)", ln).group(1)) - Y_AT
                for lane in np.flatnonzero(self.exec):
                    m, n = int(addr[lane]) // self.ldy, int(addr[lane]) % self.ldy // 2
                    assert m < M and n + 8 <= N and n % 8 == 0
                    for e in range(8):
                        from_lane, pair = self.v[data + e // 2][lane]
                        _, tile, acc, count = pair[e % 2]
                        assert count == per_tile and tile == self.tile - (self.tiles_done(acc))
                        ti, tj, r = acc // 4 // mt, acc // 4 % mt, acc % 4
                        tm, tn = self.tiles[tile]
                        # A rows of sub-tile 2 c + b are 32 c + 8 g + 4 b + r, B rows 16 tj + lane % 16
                        want_n = 256 * tn + (self.wave >> 1) * 128 + 32 * (ti // 2) + 8 * (from_lane >> 4) + 4 * (ti % 2) + r
                        want_m = 32 * mt * tm + (self.wave & 1) * 16 * mt + 16 * tj + (from_lane & 15)
                        assert (m, n + e) == (want_m, want_n)
                    assert (m, n) not in self.written
                    self.written[m, n] = True
                how = ln.split()[-1] if not ln.split()[-1].startswith("offset") else ""
                assert self.forms.setdefault(self.a[0][0], how) == how
                self.queue.append(np.zeros(0, int))
            elif op == "ds_read_b128":
                reg, imm = int(a[0][2:].split(":")[0]), int(re.search(r"offset:(\d+)", ln).group(1))
                at = (self.val(a[1].split()[0]) + imm) // 16
                assert lds.visible[at].all(), (ln, steps)
                assert reg not in self.flying
                # no two of 16 lanes in one 16-byte column of 256 bytes
                for g in range(4):
                    assert len(set((at[16 * g:16 * g + 16] % 16).tolist())) == 16
                lds.read_at[at] = np.maximum(lds.read_at[at], self.barriers)
                self.held[reg] = (lds.op[at].copy(), lds.row[at].copy(), lds.chunk[at].copy())
                self.flying.append(reg)
            elif op.startswith("v_mfma"):
                acc, fa, fb = (int(x[2:].split(":")[0]) for x in a[:3])
                assert a[3] == a[0] and fa not in self.flying and fb not in self.flying
                tile, count = self.a[acc]
                tm, tn = self.tiles[tile]
                ti, tj = acc // 4 // mt, acc // 4 % mt
                lane = np.arange(64)
                chunk = (count // 2) * 8 + (count % 2) * 4 + (lane >> 4)
                n = 256 * tn + (self.wave >> 1) * 128 + 32 * (ti // 2) + 8 * ((lane & 15) >> 2) + 4 * (ti % 2) + (lane & 3)
                m = 32 * mt * tm + (self.wave & 1) * 16 * mt + 16 * tj + (lane & 15)
                for frag, kind, want in ((fa, 1, np.minimum(n, N - 1)), (fb, 0, np.minimum(m, M - 1))):
                    o, row, ch = self.held[frag]
                    assert (o == kind).all() and (row == want).all() and (ch == chunk).all(), (ln, tile, count)
                for r in range(4):
                    self.a[acc + r] = (tile, count + 1)
            elif op == "v_accvgpr_write_b32":
                acc = int(a[0][1:])
                done = self.a.get(acc)
                assert a[1] == "0" and (done is None or done[1] == per_tile)
                self.a[acc] = (0 if done is None else done[0] + 1, 0)
            elif op == "v_accvgpr_read_b32":
                acc = int(a[1][1:])
                self.held.pop(int(a[0][1:]) & ~3, None)      # (no fragment any more)
                self.v[int(a[0][1:])] = ("sum", self.a[acc][0], acc, self.a[acc][1])
            elif op == "v_cvt_pk_bf16_f32":
                lo, hi = self.v[int(a[1][1:])], self.v[int(a[2][1:])]
                assert lo[0] == hi[0] == "sum"
                self.held.pop(int(a[0][1:]) & ~3, None)
                self.v[int(a[0][1:])] = [(lane, (lo, hi)) for lane in range(64)]
                self.written_at[int(a[0][1:])] = steps
            elif op == "v_mov_b32_dpp":                      # lane i of 16 takes that of lane (i + 8) % 16 where its bank of four is in the mask
                d, (x, *how) = int(a[0][1:]), a[1].split()
                mask = int(re.search(r"bank_mask:(0x\w+)", ln).group(1), 16)
                assert how[:2] == ["row_ror:8", "row_mask:0xf"] and steps - self.written_at[int(x[1:])] > 2
                old, new = self.v[int(x[1:])], list(self.v[d])
                for lane in range(64):
                    if mask >> (lane % 16 // 4) & 1:
                        new[lane] = old[lane & 48 | (lane + 8) & 15]
                self.v[d], self.written_at[d] = new, steps
            elif op == "v_mov_b32" and isinstance(self.v.get(int(a[1][1:]) if a[1][0] == "v" else -1), list):
                self.v[int(a[0][1:])], self.written_at[int(a[0][1:])] = self.v[int(a[1][1:])], steps
            elif op == "v_mad_u32_u24":
                x, y, z = (self.val(q) for q in a[1:])
                assert (np.asarray(x) < 1 << 24).all() and y < 1 << 24
                self.put(a[0], x * y + z)
            elif op == "v_add_co_u32":
                r = np.asarray(self.val(a[2]), dtype=np.int64) + self.val(a[3])
                self.put(a[0], r)
                self.s["vcc"] = np.broadcast_to(r >> 32, 64)
            elif op == "v_addc_co_u32":
                self.put(a[0], np.asarray(self.val(a[2]), dtype=np.int64) + self.val(a[3]) + self.s["vcc"])
            elif op in ("v_mov_b32", "v_add_u32", "v_xor_b32", "v_min_u32"):
                x = np.asarray(self.val(a[1]), dtype=np.int64)
                y = self.val(a[2]) if len(a) > 2 else None
                self.put(a[0], {"v_mov_b32": lambda: x, "v_add_u32": lambda: x + y, "v_xor_b32": lambda: x ^ y, "v_min_u32": lambda: np.minimum(x, y)}[op]())
            else:
                assert op in ("s_nop", "s_cbranch_scc1"), ln
        assert not any(len(at) for at in self.queue)          # no load is on its way when the wave ends

    def tiles_done(self, acc):
        return self.tile - self.a[acc][0]

    def put(self, d, x):
        n = int(d[1:])
        assert n not in self.held or n >= rows.ADDRW         # scalars of a lane never land in a fragment that is still to be used
        self.v[n] = np.broadcast_to(np.asarray(x, dtype=np.int64) & U32, 64).copy()


@pytest.mark.parametrize("form", [0, 4, 10])
@pytest.mark.parametrize("mt,shape,tiles,pad", [
    (8, (300, 520, 128), [(0, 0), (1, 2), (0, 1), (1, 0)], 1), (8, (513, 264, 384), [(2, 1), (0, 0)], 0), (8, (256, 768, 128), [(0, 0), (0, 1), (0, 2)], 3),
    (6, (200, 512, 256), [(0, 0), (0, 1), (1, 0)], 0), (6, (193, 8, 128), [(1, 0)], 1), (4, (129, 776, 128), [(1, 3), (0, 0), (0, 1), (1, 0)], 2),
    (4, (1, 256, 896), [(0, 0)], 0)])
def test_rows_loop_over_tiles(mt, shape, tiles, pad, form):
    """Four waves in step from barrier to barrier: every load lies inside its operand and goes where nobody reads any more, every product
    takes the rows and the 16 bytes of k of its tile, stage and k-step from registers that have them, every sum is complete
    when it leaves, and each element of the tiles is stored once, where it belongs."""
    text = [p for ln in rows.generate(mt) for p in ln.split("\n")]
    lds = _Lds()
    waves = [_Wave(mt, w, text, lds, shape, tiles, pad, form) for w in range(4)]
    going = [w.run() for w in waves]
    while going:
        ends = [next(g, "end") for g in going]
        assert len(set(ends)) == 1
        if ends[0] == "end":
            break
        pending = np.zeros(len(lds.row), bool)
        for w in waves:
            for at in w.queue:
                pending[at] = True
        lds.visible = (lds.row >= 0) & ~pending
    M, N, _ = shape
    want = {(m, n) for tm, tn in tiles for m in range(32 * mt * tm, min(32 * mt * (tm + 1), M)) for n in range(256 * tn, min(256 * (tn + 1), N), 8)}
    got = [k for w in waves for k in w.written]
    assert len(got) == len(want) and set(got) == want
    assert all(w.forms == {t: rows.FORMS[form >> 2 if t == len(tiles) - 1 else form & 3].strip() for t in range(len(tiles))} for w in waves)
    # hazards: a load to LDS stays off the M0 write before it; each stage's MFMAs are those of both k-steps on an accumulator in a row
    for k, ln in enumerate(text):
        if ln.startswith("global_load_lds"):
            assert " m0," not in text[k - 1]
    for P in range(rows.PERIOD):
        accs = [re.match(r"v_mfma\S+ (a\[\d+:\d+\])", m).group(1) for m, _ in rows.build_stage(P, mt)]
        assert accs[::2] == accs[1::2] and len(set(accs)) == 8 * mt


# --------------------------------------------------------------------------- which tiles a workgroup takes

def _share(left):
    """last_round_share"""
    return 16 if 0 < left <= 64 else (left + 7) >> 3


@pytest.mark.parametrize("tiles_m,tiles_n", [(1, 1), (1, 63), (64, 1), (13, 5), (17, 15), (32, 8), (257, 1), (9, 29), (40, 13), (127, 129), (128, 128), (16385, 1),
                                             (5, 3277), (255, 64), (33, 993), (8, 4097), (1, 49157)])
def test_every_tile_goes_to_one_workgroup(tiles_m, tiles_n):
    """gemm_rows_kernel's lists over the grid that enqueue_gemm_rows launches: rounds that end inside a group of 256 workgroups, lists of 63
    to 65 tiles, several groups."""
    total, rounds = tiles_m * tiles_n, -(-tiles_m * tiles_n // 256)
    workgroups = 8 * _share(total) if total < 256 else 256 * -(-rounds // 64)
    full, left = divmod(total, 256)
    share, taken = _share(left), []
    for b in range(workgroups):
        xcd, j, first = b & 7, b >> 3 & 31, (b >> 8) * 64
        mine = full + (j < share and xcd * share + j < left)
        for r in range(first, first + max(0, min(mine - first, 64))):
            nth = r * 256 + xcd * 32 + j if r < full else full * 256 + xcd * share + j
            band, in_band = divmod(nth, 8 * tiles_n)                 # tile_at
            height = min(8, tiles_m - band * 8)
            taken.append((band * 8 + in_band % height, in_band // height))
    assert len(taken) == total and set(taken) == {(m, n) for m in range(tiles_m) for n in range(tiles_n)}


# --------------------------------------------------------------------------- which kernel, and what it computes

# kernel, rows, columns, k, columns of Y's rows: one to three rounds, last row tiles of one row, last column tiles of eight columns, the
# shortest walk; rows of Y that are whole lines (a multiple of 64 columns) and rows that share them
CASES = [(256, 769, 13064, 128, 13064), (256, 769, 13064, 128, 13120), (256, 4097, 3592, 768, 3648), (256, 6145, 6920, 128, 6920), (256, 6145, 6920, 128, 6976),
         (192, 2881, 2824, 384, 2824), (192, 1537, 4872, 128, 4928), (192, 5761, 3080, 384, 3080), (128, 513, 11016, 128, 11016), (128, 4993, 4616, 256, 4672),
         (128, 2305, 2056, 640, 2112), ("kTile256x128", 4680, 1544, 384, 1544), ("kTile128", 2050, 1160, 128, 1160), ("kTile64", 1100, 1400, 256, 1400),
         ("kTile64Wide", 129, 200, 768, 200)]


def test_every_kernel_has_a_case():
    """... which is the one that the dispatch takes for it (in the names of the GPU tests' products too)."""
    from tests import test_gpu_edges as E
    assert [Hn.linear_kernel(*c[1:4]) for c in CASES] == [c[0] for c in CASES]
    assert [Hn.linear_kernel(*c[1:]) for c in E.LINEAR_TILES] == [c[0] for c in E.LINEAR_TILES]
    names, model, heights = Hn._gemm_models()
    kernels = {h[0] for h in heights} | {n for n, m in zip(names, model) if m[6]}
    assert {c[0] for c in CASES} == {c[0] for c in E.LINEAR_TILES} == kernels == {256, 192, 128, "kTile256x128", "kTile128", "kTile64", "kTile64Wide"}


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,M,N,K,ldy", CASES)
def test_products(kernel, M, N, K, ldy):
    """Against fp64, and nothing outside the result is written; X and W with rows longer than k."""
    import torch
    from paper_2511_20426_amd.runner import linear
    x, w = W.draw_linear(M, N, K, seed=M + N)
    xt, wt = (torch.full((t.shape[0] + 1, K + 16), 3.0, dtype=torch.bfloat16, device="cuda:0") for t in (x, w))
    xt[:M, :K], wt[:N, :K] = Hn.to_torch(x, "bf16"), Hn.to_torch(w, "bf16")
    yt = torch.full((M + 2, ldy), 7.0, dtype=torch.bfloat16, device="cuda:0")
    print(f"product {kernel} {M}x{N}x{K} ldy={ldy}", flush=True)
    linear(xt[:M, :K], wt[:N, :K], out=yt[:M, :N])
    torch.cuda.synchronize()
    got = Hn.from_torch(yt, "bf16")
    assert (got[M:] == 7.0).all() and (got[:, N:] == 7.0).all()
    # one rounding to bf16 and fp32 accumulation: half an ulp is 2^-9 relative, 2^-8 and 1e-5 of sum |x||w| allowed
    rows_ = np.unique(np.concatenate([np.arange(0, M, max(1, M // 300)), [M - 1]]))
    xf, wf = W.to_f64(x[rows_]), W.to_f64(w)
    ref = orc.layer_linear(xf, wf)
    bound = np.abs(ref) * 2.0 ** -8 + 1e-5 * orc.layer_linear(np.abs(xf), np.abs(wf)) + 1e-30
    assert (np.abs(got[rows_, :N].astype(np.float64) - ref) <= bound).all(), f"{M}x{N}x{K}"


@pytest.mark.gpu
def test_lists_of_more_than_64_tiles():
    """A second group of workgroups (more than 64 rounds of 256 tiles): every element against the product in fp32."""
    import torch
    from paper_2511_20426_amd.runner import linear
    M, N, K = 256 * 256 * 64 + 256 + 1, 256, 128
    assert Hn.linear_kernel(M, N, K) == 256
    gen = torch.Generator(device="cuda:0").manual_seed(8)
    x, w = (torch.randn((n, K), generator=gen, device="cuda:0", dtype=torch.bfloat16) for n in (M, N))
    y = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device="cuda:0")
    print(f"product {M}x{N}x{K}", flush=True)
    linear(x, w, out=y[:M])
    torch.cuda.synchronize()
    assert (y[M] == 7.0).all()
    wf = w.float()
    for at in range(0, M, 1 << 18):
        xf, got = x[at:at + (1 << 18)].float(), y[at:min(M, at + (1 << 18))].float()
        ref = xf @ wf.T
        # one rounding to bf16 (2^-9 relative) and the order of 128 products in fp32 on both sides
        assert ((got - ref).abs() <= ref.abs() * 2.0 ** -8 + 2e-5 * (xf.abs() @ wf.abs().T) + 1e-30).all(), at
