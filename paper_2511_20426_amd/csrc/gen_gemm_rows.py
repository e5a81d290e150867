#!/usr/bin/env python3
"""Emits gemm_rows{256,192,128}_gfx950.inc: the whole life of a workgroup of the plain linear map Y = X . W^T, which takes
one tile of 256, 192 or 128 rows by 256 columns after the other (MT = 8, 6, 4 sub-tiles of 16 rows to a wave).

Tile, waves, stages of 64 k, rings in LDS and barriers are those of gen_gemm_core.py, which says why they are so.  Here a
workgroup does not end with its tile: the stream of stages goes on with the next tile's, so that nothing is requested twice
and nothing waited for between tiles, and the results leave straight from registers, without LDS, which the next tile's
stages are filling by then.  What a tile of 256 rows costs outside its products went from 11 us (set-up, first fill, transposition
through LDS, two barriers) to 5.1, by the cost models fitted to either (rows_tile in gemm_bf16.hip).

Results from registers.  With W as the A operand a lane ends up with four consecutive rows of W, that is four columns of one
row of Y.  The 16 rows of W that sub-tile ti = 2 c + b multiplies are picked as 32 c + 8 g + 4 b + r (lane group g, accumulator
r), so that a lane's two sub-tiles of a pair hold eight consecutive columns: 16 bytes, and its lane groups 64 bytes of a row.  Lanes 0..7 and 8..15 of a
group then exchange one of two such pieces, so that a store writes eight rows of 128 bytes, whole lines, not 16 of half of one.
W's rows lie in LDS with their chunks at c ^ s(row), s = (row >> 1 & 1) | (row >> 3 & 3) << 1, which makes these reads free
of bank conflicts (X's rows as in gen_gemm_core.py).

Order of the products.  Both k-steps of a stage follow one another on an accumulator, and the tiles go two rows at a time,
forth and back: an accumulator that stays in the pipe and an operand that stays put save power.  An MFMA-only loop over
random operands, TFLOP/s: rows of tiles one after the other 2110, two rows forth and back 2169, with both k-steps
2243.  For that X's fragments of a whole stage are held in registers (two sets, the next stage's is read behind the
barrier) and W's of two rows of tiles (three sets in turn).

Register map:
  a[0:32 MT - 1]   accumulators, sub-tile (ti over n, tj over m) at a[4 (MT ti + tj) ..]
  v[0:127]    X fragments: stage parity p, k-step kk, sub-tile tj at v[64 p + 32 kk + 4 tj ..]; set 1 is scratch between tiles
  v[128:175]  W fragments: set b, row i of two, k-step kk at v[128 + 16 b + 8 i + 4 kk ..]
  v176..v181  LDS read addresses of W: v[176 + 2 ring slot + kk];  v182..v185 of X
  v186..v193, v194..v201  lane's byte offset from the stage's global base for W / X loads 0..7
  v202..v205  address of the lane's row of Y, temporaries
"""
from __future__ import annotations

import os
import sys

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gen_gemm_core import CAP, NW, NX, PART, PERIOD, XBASE, A, V, tile_order  # noqa: E402
from issue_sched import Atom, quanta, schedule  # noqa: E402

ADDRW, ADDRX = 176, 182  # + 2*ring slot + kk
OFFW, OFFX = 186, 194    # +i
YROW, VT = 202, 204      # address of the lane's row (two registers), temporaries (two)
LAST_VGPR = 205

S_BW, S_BX = 36, 38      # global bases of the W / X stage being loaded (64-bit each)
S_WSTEP, S_XSTEP = 40, 41  # bytes from one stage to the next: 128, 0 behind the last tile
S_TRIPS, S_HALF, S_NST, S_M0B, S_M0X = 42, 43, 44, 45, 46
S_WT, S_XT, S_YT = 47, 48, 49                 # number, in this workgroup's list, of the tile loaded and multiplied
S_WL = 50                # pairs of stages until the next tile's W is due
S_WLIM, S_XLIM = 51, 52  # last valid row of the tile being loaded
S_RET = 54               # 54,55: where out-of-line code returns to
S_T = 56                 # 56..63 temporaries
S_COLS = 64              # 64..67: lanes whose columns exist, of the first 64 and the others
S_ROWS, S_NCOL = 68, 69  # rows and columns of the tile that exist


def xfrag(p, kk, tj):
    return 64 * p + 32 * kk + 4 * tj


def wfrag(buf, i, kk):
    return 128 + 16 * (buf % 3) + 8 * i + 4 * kk


def mfma(P, ti, tj, kk, mt):
    acc = A(4 * (mt * ti + tj), 4)
    return f"v_mfma_f32_16x16x32_bf16 {acc}, {V(wfrag(P + ti // 2, ti % 2, kk), 4)}, {V(xfrag(P % 2, kk, tj), 4)}, {acc}"


def read_w(stage, ti, kk):
    """rows 32 c + 4 b .. of the wave's 128 (lane part in the address register) for sub-tile ti = 2 c + b"""
    return f"ds_read_b128 {V(wfrag(stage + ti // 2, ti % 2, kk), 4)}, {V(ADDRW + 2 * (stage % NW) + kk)} offset:{4096 * (ti // 2) + 512 * (ti % 2)}"


def read_x(stage, tj, kk):
    return f"ds_read_b128 {V(xfrag(stage % 2, kk, tj), 4)}, {V(ADDRX + 2 * (stage % NX) + kk)} offset:{2048 * tj}"


def load_lines(op, stage, i, mt):
    """as gen_gemm_core's"""
    ring = (stage % NW) * PART if op == 0 else XBASE + (stage % NX) * PART * mt // 8
    base, off, m0b = (S_BW, OFFW, S_M0B) if op == 0 else (S_BX, OFFX, S_M0X)
    return [f"s_add_u32 m0, s{m0b}, {ring + 1024 * i}",
            f"global_load_lds_dwordx4 {V(off + i)}, s[{base}:{base + 1}]"]


def call_lines(to, back, tag):
    """out-of-line code common to several places: `to` is entered with the address of `back` (which lies before) in S_RET"""
    return [f"s_getpc_b64 s[{S_RET}:{S_RET + 1}]", f"PC{tag}_%=:", f"s_sub_u32 s{S_RET}, s{S_RET}, PC{tag}_%=-{back}",
            f"s_subb_u32 s{S_RET + 1}, s{S_RET + 1}, 0", f"s_branch {to}"]


def advance_lines(op):
    """on to the next stage to load"""
    base, step = (S_BW, S_WSTEP) if op == 0 else (S_BX, S_XSTEP)
    return [f"s_add_u32 s{base}, s{base}, s{step}", f"s_addc_u32 s{base + 1}, s{base + 1}, 0"]


def w_due_lines(tag, cold):
    """out of line to the next tile's W when it is due (behind an even number of stages, so that every other stage looks)"""
    go, back = f"NEXTW{tag}_%=", f"BACKW{tag}_%="
    cold += [f"{go}:"] + call_lines("TILEW_%=", back, f"W{tag}")
    return [f"s_sub_u32 s{S_WL}, s{S_WL}, 1", f"s_cmp_eq_u32 s{S_WL}, 0", "s_nop 0", f"s_cbranch_scc1 {go}", f"{back}:"]


def next_tile_lines(op, mt):
    """The tile whose stages are requested next: its base, less a step, and the lanes' offsets if it has another number of
    rows than the one before (rows past the end re-read the last one).  Behind the last tile its last stage is requested
    over and over, into buffers that nothing reads."""
    name = "W" if op == 0 else "X"
    base, step, t, lim, off = (S_BW, S_WSTEP, S_WT, S_WLIM, OFFW) if op == 0 else (S_BX, S_XSTEP, S_XT, S_XLIM, OFFX)
    rows, total, stride, ld, n, first, chunk = ((256, "%[N]", "%[tile_w]", "%[ldw2]", 8, "%[roww]", "%[chunkw]") if op == 0 else
                                                (32 * mt, "%[M]", "%[tile_x]", "%[ldx2]", mt, "%[rowx]", "%[chunkx]"))
    a = S_T
    out = [f"s_mov_b32 s{S_WL}, s{S_HALF}"] if op == 0 else []
    out += [f"s_add_u32 s{t}, s{t}, 1", f"s_cmp_ge_u32 s{t}, %[tiles]", "s_nop 0", f"s_cbranch_scc1 LAST{name}_%=",
            f"v_readlane_b32 s{a}, %[list_{'n' if op == 0 else 'm'}], s{t}", "s_nop 3",
            f"s_mul_i32 s{base}, s{a}, {stride}", f"s_mul_hi_u32 s{base + 1}, s{a}, {stride}",
            f"s_add_u32 s{base}, s{base}, %[{name.lower()}_lo]", f"s_addc_u32 s{base + 1}, s{base + 1}, %[{name.lower()}_hi]",
            f"s_sub_u32 s{base}, s{base}, s{step}", f"s_subb_u32 s{base + 1}, s{base + 1}, 0",
            f"s_mul_i32 s{a + 1}, s{a}, {rows}", f"s_sub_u32 s{a + 1}, {total}, s{a + 1}", f"s_min_u32 s{a + 1}, s{a + 1}, {rows}",
            f"s_sub_u32 s{a + 1}, s{a + 1}, 1",
            f"s_cmp_eq_u32 s{a + 1}, s{lim}", "s_nop 0", f"s_cbranch_scc1 SAME{name}_%=", f"s_mov_b32 s{lim}, s{a + 1}"]
    for i in range(n):
        out += [f"v_add_u32 {V(VT)}, {8 * i}, {first}", f"v_min_u32 {V(VT)}, s{lim}, {V(VT)}",
                f"v_xor_b32 {V(VT + 1)}, {((i & 3) << 5) if op == 0 else ((i & 1) << 6)}, {chunk}",
                f"v_mad_u32_u24 {V(off + i)}, {V(VT)}, {ld}, {V(VT + 1)}"]
    return out + [f"SAME{name}_%=:", f"s_setpc_b64 s[{S_RET}:{S_RET + 1}]",
                  f"LAST{name}_%=:", f"s_mov_b32 s{step}, 0", f"s_setpc_b64 s[{S_RET}:{S_RET + 1}]"]


FORMS = ("", " sc1", " nt")     # how results are written: left in L2, written through it, past the caches


def result_lines(mt):
    """A tile's sums leave, rounded to bf16, 16 bytes of a row to a lane, in the form that %[form] has for the last tile of the
    workgroup or for the others, and start from zero again if there is a next tile.  (Between a vector instruction that writes VCC
    or a scalar register and one that reads it stand two wait states, as the compiler has it for gfx950.)"""
    a = S_T
    out = ["s_nop 15", "s_nop 15",                         # the last MFMAs have written back
           f"v_readlane_b32 s{a}, %[list_m], s{S_YT}", f"v_readlane_b32 s{a + 1}, %[list_n], s{S_YT}", "s_nop 3",
           # y + tm * (rows of a tile) + tn * 512 bytes
           f"s_mul_i32 s{a + 2}, s{a}, %[tile_y_lo]", f"s_mul_hi_u32 s{a + 3}, s{a}, %[tile_y_lo]", f"s_mul_i32 s{a + 4}, s{a}, %[tile_y_hi]",
           f"s_add_u32 s{a + 3}, s{a + 3}, s{a + 4}", f"s_add_u32 s{a + 2}, s{a + 2}, %[y_lo]", f"s_addc_u32 s{a + 3}, s{a + 3}, %[y_hi]",
           f"s_lshl_b32 s{a + 4}, s{a + 1}, 9", f"s_add_u32 s{a + 2}, s{a + 2}, s{a + 4}", f"s_addc_u32 s{a + 3}, s{a + 3}, 0",
           f"v_add_co_u32 {V(YROW)}, vcc, s{a + 2}, %[ylane_lo]", f"v_mov_b32 {V(VT)}, s{a + 3}", "s_nop 0",
           f"v_addc_co_u32 {V(YROW + 1)}, vcc, {V(VT)}, %[ylane_hi], vcc",
           # what exists of the tile
           f"s_mul_i32 s{a + 4}, s{a}, {32 * mt}", f"s_sub_u32 s{S_ROWS}, %[M], s{a + 4}",
           f"s_lshl_b32 s{a + 4}, s{a + 1}, 8", f"s_sub_u32 s{S_NCOL}, %[N], s{a + 4}"]
    for c in range(2):
        out += [f"s_sub_i32 s{a + 4}, s{S_NCOL}, {64 * c}", f"v_cmp_gt_i32 s[{S_COLS + 2 * c}:{S_COLS + 2 * c + 1}], s{a + 4}, %[col]"]
    out += [f"s_add_u32 s{S_YT}, s{S_YT}, 1", f"s_and_b32 s{a + 5}, %[form], 3", f"s_lshr_b32 s{a + 6}, %[form], 2",
            f"s_cmp_lt_u32 s{S_YT}, %[tiles]", f"s_cselect_b32 s{a + 5}, s{a + 5}, s{a + 6}"]
    for k in (1, 2):
        out += [f"s_cmp_eq_u32 s{a + 5}, {k}", "s_nop 0", f"s_cbranch_scc1 FORM{k}_%="]
    for k, form in enumerate(FORMS):
        out.append(f"FORM{k}_%=:")
        for tj in range(mt):
            pack = 96 + 16 * (tj % 2)
            for c in range(4):
                acc = 64 + 8 * (c % 2)
                for i in range(8):                         # sub-tiles 2 c and 2 c + 1
                    out.append(f"v_accvgpr_read_b32 {V(acc + i)}, {A(4 * (mt * (2 * c + i // 4) + tj) + i % 4)}")
                for i in range(4):
                    out.append(f"v_cvt_pk_bf16_f32 {V(pack + 4 * c + i)}, {V(acc + 2 * i)}, {V(acc + 2 * i + 1)}")
            # whole lines: of two pairs of sub-tiles, lanes 0..7 and 8..15 of a group exchange the one they do not keep (a register
            # is read across lanes two or more instructions after it was written)
            for c in (0, 2):
                kept, other, t = pack + 4 * c, pack + 4 * c + 4, 80 + 2 * c
                out += [f"v_mov_b32 {V(t + i)}, {V(other + i)}" for i in range(4)]
                out += [f"v_mov_b32_dpp {V(other + i)}, {V(kept + i)} row_ror:8 row_mask:0xf bank_mask:0x3" for i in range(4)]
                out += [f"v_mov_b32_dpp {V(kept + i)}, {V(t + i)} row_ror:8 row_mask:0xf bank_mask:0xc" for i in range(4)]
            for half in range(2):                          # rows 0..7 of the sixteen, then the others
                out += [f"s_sub_i32 s{a + 4}, s{S_ROWS}, {16 * tj + 8 * half}", f"v_cmp_gt_i32 vcc, s{a + 4}, %[row]", "s_nop 1"]
                for c in range(2):
                    out += [f"s_and_b64 exec, vcc, s[{S_COLS + 2 * c}:{S_COLS + 2 * c + 1}]",
                            f"global_store_dwordx4 {V(YROW, 2)}, {V(pack + 8 * c + 4 * half, 4)}, off offset:{128 * c}{form}"]
                out.append("s_mov_b64 exec, -1")
                if tj < mt - 1 or half == 0:
                    out += [f"v_add_co_u32 {V(YROW)}, vcc, %[row8_lo], {V(YROW)}", f"v_mov_b32 {V(VT)}, %[row8_hi]", "s_nop 0",
                            f"v_addc_co_u32 {V(YROW + 1)}, vcc, {V(VT)}, {V(YROW + 1)}, vcc"]
        if k < 2:
            out.append("s_branch LEFT_%=")
    out += ["LEFT_%=:", f"s_mov_b32 s{S_TRIPS}, s{S_HALF}", f"s_cmp_lt_u32 s{S_YT}, %[tiles]", "s_nop 0", "s_cbranch_scc1 CLEAR_%=",
            f"s_waitcnt vmcnt({4 * mt})",                  # the last tile: every load has landed; the results need not have
            "s_branch DONE_%=", "CLEAR_%=:"]
    return (out + [f"v_accvgpr_write_b32 {A(r)}, 0" for r in range(32 * mt)] +
            ["s_nop 7", f"s_cmp_eq_u32 s{S_HALF}, 1", "s_nop 0", "s_cbranch_scc1 TILEX_%=", f"s_setpc_b64 s[{S_RET}:{S_RET + 1}]"])


def build_stage(P, mt=8, cold=None):
    """Stage P (mod PERIOD) of the steady state: 16 mt slots of (MFMA, lines issued after it)."""
    cold = [] if cold is None else cold
    slots, x_by, pair = 16 * mt, 5 * mt, 4 * mt             # pair: slots of two rows of tiles
    half = slots // 2
    mf = [mfma(P, ti, tj, kk, mt) for ti, tj in tile_order(mt) for kk in range(2)]
    tail = [[] for _ in range(slots)]
    # in front of the barrier: this stage's last fragments are in registers, everything but the W loads issued last has landed (and the
    # results of a tile that left at the start of this stage); behind it this stage's buffers are free
    tail[half - 1] += ["s_waitcnt vmcnt(@VM@) lgkmcnt(0)", "s_barrier"]
    tail[pair - 1] += ["s_waitcnt lgkmcnt(4)"]             # the second two rows' fragments; the third's may be on their way
    tail[slots - 1] += ["s_waitcnt lgkmcnt(0)"]
    atoms = []

    def reads(lines, first, last, hard):
        prev = None
        for k, ln in enumerate(lines):
            at = first + (k * (last - first)) // len(lines)
            prev = Atom([ln], at, at, [prev] if prev else [], 0, hard=hard)
            atoms.append(prev)
    rows = lambda stage, b: [read_w(stage, 2 * b + i, kk) for i in range(2) for kk in range(2)]  # noqa: E731
    reads(rows(P, 1), 0, pair // 3, pair - 9)
    reads(rows(P, 2), pair // 2, pair - 1, pair - 1)
    reads(rows(P, 3), pair, half - 8, half - 6)             # (set of the first two rows, done with by then)
    # behind the barrier: the next stage's X, its first two rows of W; what is used first comes first
    order = []
    for ti, tj in tile_order(mt):
        for kk in range(2):
            order += [ln for ln in ([read_w(P + 1, ti, kk)] if ti < 2 else []) + [read_x(P + 1, tj, kk)] if ln not in order]
    reads(order, half + 1, slots - 14, slots - 6)
    prev = None
    for grp in [advance_lines(1)] + ([w_due_lines(P, cold)] if P % 2 else []) + [advance_lines(0)]:
        prev = Atom(grp, half, half, [prev] if prev else [], 0, hard=half + 8)
        atoms.append(prev)
    # behind the barrier: X of stage P+2 first (it is needed one stage on), then W of stage P+3 (M0 is written in an earlier slot than
    # its load, so that an MFMA stands between, and behind the load before)
    last, w_gap = prev, (half - 14) / 8 if mt < 8 else 6.5
    for op, stage, i, at, hard in ([(1, P + 2, i, half + 5 + (i * x_by) // mt, min(half + x_by + 8, slots - 11)) for i in range(mt)] +
                                   [(0, P + 3, i, half + 7 + int(w_gap * i), slots - 2 - (7 - i)) for i in range(8)]):
        m0, load = load_lines(op, stage, i, mt)
        write = Atom([m0], at - 1, at - 1, [last], 0, hard=hard - 1)
        last = Atom([load], at, at, [write], 1, hard=hard)
        atoms += [write, last]
    fixed = [2.0 + sum(quanta(ln) for ln in tail[i]) for i in range(slots)]
    placed = schedule(fixed, atoms, CAP)
    out = [(mf[i], [ln for a in placed[i] for ln in a.lines] + tail[i]) for i in range(slots)]
    # Loads complete in order.  At the next barrier the X loads issued here must have landed (and with them every older load): as
    # many may still fly as were issued behind the last X load.
    kinds = ["x" if f"s[{S_BX}:" in ln else "w" for _, lines in out for ln in lines if ln.startswith("global_load_lds")]
    behind = len(kinds) - 1 - max(k for k, x in enumerate(kinds) if x == "x")
    out = [(m, [ln.replace("@VM@", str(behind)) for ln in lines]) for m, lines in out]
    return out


def generate(mt=8):
    L, cold = [], []
    e = L.append
    e(f"s_mov_b32 s{S_NST}, %[n_stages]")
    e(f"s_lshr_b32 s{S_HALF}, s{S_NST}, 1")
    e(f"s_mov_b32 s{S_TRIPS}, s{S_HALF}")
    e(f"s_lshl_b32 s{S_M0B}, %[wave], 13")
    e(f"s_add_u32 s{S_M0B}, s{S_M0B}, %[lds0]")
    e(f"s_mul_i32 s{S_M0X}, %[wave], {1024 * mt}")
    e(f"s_add_u32 s{S_M0X}, s{S_M0X}, %[lds0]")
    for r in (S_WT, S_XT, S_WLIM, S_XLIM):
        e(f"s_mov_b32 s{r}, -1")
    for r in (S_WSTEP, S_XSTEP):
        e(f"s_mov_b32 s{r}, 128")
    e(f"s_mov_b32 s{S_YT}, 0")
    # the first tile, stage 0 first, then what the steady state would have requested, in its order: X of stage 1, W of 1 and 2
    for op, name in ((0, "W"), (1, "X")):
        e(f"s_branch FIRST{name}_%=")
        e(f"GOT{name}_%=:")
        cold += [f"FIRST{name}_%=:"] + call_lines(f"TILE{name}_%=", f"GOT{name}_%=", f"F{name}")
    for op, st in ((0, 0), (1, 0), (1, 1), (0, 1), (0, 2)):
        if (op, st) == (0, 2):
            L.extend(w_due_lines("P", cold))
        L.extend(advance_lines(op))
        for i in range(mt if op else 8):
            m0, load = load_lines(op, st, i, mt)
            L.extend([m0, "s_nop 0", load])
    e(f"s_cmp_eq_u32 s{S_TRIPS}, 1")                      # X of stage 2 is the next tile's
    e("s_nop 0")
    e("s_cbranch_scc1 NEXTX_%=")
    e("BACKX_%=:")
    cold += ["NEXTX_%=:"] + call_lines("TILEX_%=", "BACKX_%=", "X")
    # (meanwhile: read addresses, accumulators)
    for arg, areg, depth, ring0, part in (("aw0", ADDRW, NW, 0, PART), ("ax0", ADDRX, NX, XBASE, PART * mt // 8)):
        for slot in range(depth):
            for kk in range(2):                           # chunk index of k-step 1 = that of 0, xor 4
                r = areg + 2 * slot + kk
                e(f"v_xor_b32 {V(r)}, {kk << 6}, %[{arg}]")
                e(f"v_add_u32 {V(r)}, %[lds0], {V(r)}")
                e(f"v_add_u32 {V(r)}, {ring0 + slot * part}, {V(r)}")
    for r in range(32 * mt):
        e(f"v_accvgpr_write_b32 {A(r)}, 0")
    e(f"s_waitcnt vmcnt({mt + 16})")                      # stage 0 has landed
    e("s_barrier")
    for i in range(2):
        for kk in range(2):
            e(read_w(0, i, kk))
    for tj in range(mt):
        for kk in range(2):
            e(read_x(0, tj, kk))
    e("s_waitcnt lgkmcnt(0)")
    # a tile may end every two stages; a loop trip is PERIOD stages
    e("LOOP_%=:")
    for P in range(PERIOD):
        e(f"; ---- stage {P}")
        for m, lines in build_stage(P, mt, cold):
            e(m)
            L.extend(lines)
        if P % 2 == 1:
            e(f"s_sub_u32 s{S_TRIPS}, s{S_TRIPS}, 1")
            e(f"s_cmp_lt_u32 s{S_TRIPS}, 2")
            e("s_nop 0")
            e(f"s_cbranch_scc1 END{P}_%=")
            e(f"ON{P}_%=:")
            cold += [f"END{P}_%=:"] + call_lines("PAIR_%=", f"ON{P}_%=", f"E{P}")
    e("s_branch LOOP_%=")
    L += cold
    L += ["TILEW_%=:"] + next_tile_lines(0, mt) + ["TILEX_%=:"] + next_tile_lines(1, mt)
    # a tile ends, or its last two stages begin: X of those behind them is the next tile's
    L += ["PAIR_%=:", f"s_cmp_eq_u32 s{S_TRIPS}, 1", "s_nop 0", "s_cbranch_scc1 TILEX_%="] + result_lines(mt)
    e("DONE_%=:")
    return L


def main(out_path):
    by = "// Generated by gen_gemm_rows.py -- do not edit.\n"
    clobbers = by
    for mt in (8, 6, 4):
        path = out_path.replace("gemm_rows_", f"gemm_rows{32 * mt}_")
        lines = generate(mt)
        with open(path, "w") as f:
            f.write(by)
            for ln in lines:
                f.write('"' + ln + '\\n"\n')
        print(f"{path}: {len(lines)} lines")
        clob = [f"v{i}" for i in range(LAST_VGPR + 1)] + [f"a{i}" for i in range(32 * mt)] + [f"s{i}" for i in range(36, S_NCOL + 1)]
        clobbers += f"#define CA_GEMM_ROWS_CLOBBERS{32 * mt} \\\n"
        for i in range(0, len(clob), 12):
            chunk = ", ".join(f'"{c}"' for c in clob[i:i + 12])
            clobbers += "  " + chunk + (", \\\n" if i + 12 < len(clob) else "\n")
    with open(out_path.replace("gemm_rows_gfx950.inc", "gemm_rows_clobbers.inc"), "w") as f:
        f.write(clobbers)


if __name__ == "__main__":
    main(sys.argv[1] if len(sys.argv) > 1 else "gemm_rows_gfx950.inc")
