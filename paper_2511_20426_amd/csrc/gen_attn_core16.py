#!/usr/bin/env python3
"""Emits attn_core16_gfx950.inc: the main loop of gen_attn_core.py on the 16x16x32 matrix instruction, for launches that
fill the chip.  Walk, page traffic, barriers and scalar registers are that generator's.

Why 16x16x32 and not 32x32x16: a launch that fills the chip is limited by power, and per flop the smaller
shape moves half as many accumulator registers.  An MFMA-only loop over random operands (mfma_peak.hip) reaches 2118..2203
TFLOP/s with it, four consecutive MFMAs on one accumulator as QK has them below, against 1784..1876 with 32x32x16 in the same sessions.  The
price is issue room (64 MFMAs a step for 32): a slot is dealt out by its own model (schedule16), and by it a step takes 1096
cycles, 1024 of them of the matrix pipe: what is left over is vector work that finds no room.  14B step of five blocks 16.45 ->
15.6 ms, 1.3B one block 688 -> 643 us, one device's share 2.91 -> 2.8 ms.  (Row sums taken by the matrix pipe, ones x P, would
be 1 to 1.5 % faster, but of probabilities already rounded to bf16: a row with one heavy key was then off by up to 2.5e-3 as a whole.)

Pipeline (a "step" is 32 keys, a page is 4 steps; t counts steps):
    QK(t+1): 32 MFMAs  S_next = K_frag x Q                      (K fragments from LDS)
    SM(t)  : p = exp2(S_cur), bf16 pack, row sums                (VALU; S_cur already holds
             s*c - m_ref: Q is pre-scaled by c = log2(e)/sqrt(D) and QK starts from -m_ref)
    PV(t-1): 32 MFMAs  O^T   += V_frag x P_prev                  (V fragments from LDS)

Keys in the accumulators.  A 16x16 accumulator tile gives lane group g (of 16 lanes) its rows 4g..4g+3.  A 32-key
step has two such tiles; their 16 rows are keys 0..7 and 16..23 (second tile: 8..15 and 24..31), so that what a
lane group holds in both, keys 16 (g/2) + 4 (g%2) + {0..3, 8..11}, is one 16-byte chunk of a V row and P goes from accumulator
to operand without movement.  The K rows a read touches then meet in pairs in an LDS bank; LDS has the room
(33 % busy, a third of that for these conflicts).

The exponent reference m_ref of a row is lazy: it starts as the maximum of the row's first tile
and moves only when it has to.  No maximum is taken in the loop; instead the 8 probabilities of a row that a
lane forms in a step are summed on their own, and a sum above 2^16 (or inf: exp2 against a stale
reference may overflow) sends the wave to an out-of-line block at the end of the step, which
takes the tile's maximum, forms the step's probabilities again from the S tile (still in
registers) against the raised reference and rescales what earlier steps left.  The same branch
serves the rare step whose S tile needs its ragged tail masked.

Register map (fixed):
  a[0:127]    O^T accumulators, (dt, qt) at a[16 dt + 4 qt ..]: dims 16 dt + 4 (lane/16) + i of query lane%16 of tile qt
  a[128:191]  Q fragments, (qt, ks) at a[128 + 4*(4*qt+ks) ..]
  v[0:31]     S tile A, (kt, qt) at v[16 kt + 4 qt ..]     v[32:63]  S tile B
  v[64:79]    P^T tile A, qt at v[64 + 4 qt ..]      v[80:95]  P^T tile B
  v[96:127]   ring of 8 operand fragments
  v[128:131]  LDS address in the K ring for chunks 4j.., v[132:135] in the V ring for 32-key step j of a page
  v[148:151]  running row sums of this lane's keys, per query tile
  v[152:155]  row sums of the current step
  v156..v175  temporaries of the out-of-line blocks
  v[184:199]  -m_ref per query tile, replicated 4 times: the C operand of the
              first MFMA of every S tile, so a tile comes out of the matrix pipe as s*c - m_ref
  v[216:223]  lane's byte offset inside a page for page load i = 0..7
  v[224:255]  the 32 probabilities of the step before they are packed
  v177,v178   address of page 0 of each KV block for this head (lane i = block i), low / high word
  v179        first key this lane holds in a step: 16 (g/2) + 4 (g%2)
  v180, v181  4*(lane ^ 16), 4*(lane ^ 32): ds_bpermute addresses of the lanes that share this query
"""
from __future__ import annotations

import os
import sys

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import gen_attn_core as base  # noqa: E402
from gen_attn_core import (A, FR, P_TILE, PAGE, S_LDS0, S_NLEFT, S_P, S_PGCUR, S_PGNEXT, S_PM1, S_RG, S_T, S_TILE,  # noqa: E402
                           S_VLAST, S_VLP, V, VRING, Emitter, page_advance_lines, page_load_atoms, page_load_lines, v_address_lines,
                           barriers, emit_pages_with_tails, last_step_atoms)
from issue_sched import Atom, is_vector, schedule16, split_cost  # noqa: E402

QT = 4               # query tiles of 16 per wave
SLOTS = 64           # MFMAs of a step: 32 QK, 32 PV

XOK, XOV = 128, 132
XOVL, XOV_STRIDE = 136, 1      # with short pages: LDS address in the V ring for the last step walked; registers of a step's
LACC = 148           # 148..151: running row sums per query tile
TS = [152, 153, 154, 155]      # row sums of the current step
NT = [184 + 4 * qt for qt in range(QT)]      # -m_ref of the tile's query, four times: C operand of a tile's first MFMA
MX = [156, 157, 158, 159]
PX = 224             # 224..255: the 32 probabilities of the step, before packing
RT = list(range(160, 176))     # rare-path temporaries
KIDX, XL16, XL32 = 179, 180, 181


def s_reg(s_base, kt, qt, i=0):
    return s_base + 16 * kt + 4 * qt + i


def o_reg(dt, qt, i=0):
    return 16 * dt + 4 * qt + i


def mfma_qk(s_base, kt, qt, ks, start=None):
    """start: what the sums begin with in place of -m_ref"""
    d = V(s_reg(s_base, kt, qt), 4)
    c = (start or V(NT[qt], 4)) if ks == 0 else d
    return f"v_mfma_f32_16x16x32_bf16 {d}, {V(FR + 4 * (4 * kt + ks), 4)}, {A(128 + 4 * (4 * qt + ks), 4)}, {c}"


def mfma_pv(dt, qt, p_base):
    o = A(o_reg(dt, qt), 4)
    return f"v_mfma_f32_16x16x32_bf16 {o}, {V(FR + 4 * dt, 4)}, {V(p_base + 4 * qt, 4)}, {o}"


def pv_order(p_base):
    """the query tiles forth and back, so that where a V fragment ends the next MFMA keeps its P operand: 2178 TFLOP/s in a loop of
    nothing but these MFMAs and QK's, 2148 with the tiles always in one order; whole steps gain under 1 %, which the noise of a
    run hides at the 14B shape"""
    return [mfma_pv(dt, qt if dt % 2 == 0 else QT - 1 - qt, p_base) for dt in range(8) for qt in range(QT)]


def qk_order():
    """the four k-steps of a tile back to back: an accumulator that stays in the pipe costs less power"""
    return [(kt, qt, ks) for kt in range(2) for qt in range(QT) for ks in range(4)]


def k_source(page_sub, par, f):
    """(address register, immediate) of K fragment f = 4 kt + ks of a 32-key step of a page."""
    kt, ks = f >> 2, f & 3
    return XOK + (ks ^ (2 * kt)), par * PAGE + page_sub * 8192 + kt * 2048


def frag_source(R, par, f, tails=False, short=False):
    """(address register, immediate) of operand fragment f of step (R, par): 0..7 K, 8..15 V."""
    if f < 8:                                   # K fragment of step t+1
        return k_source(R + 1, par, f) if R < 3 else k_source(0, 1 - par, f)   # (first step of page q+1)
    dt = f - 8
    if R == 0 and tails:                        # V of the last step of page q-1, whichever that was
        return XOVL, (1 - par) * PAGE + dt * 4096
    if short:                                   # the step after a short page's first
        return XOV, par * PAGE + dt * 4096
    if R == 0:                                  # V of the last step of page q-1
        return XOV + 3, (1 - par) * PAGE + dt * 4096
    return XOV + R - 1, par * PAGE + dt * 4096


def ds_read_frag(f, src):
    reg, imm = src
    return f"ds_read_b128 {V(FR + 4 * (f % 8), 4)}, {V(reg)} offset:{imm}"


def row_max_lines(m, regs):
    """m = max over eight registers"""
    return [f"v_max3_f32 {m}, {V(regs[0])}, {V(regs[1])}, {V(regs[2])}",
            f"v_max3_f32 {m}, {m}, {V(regs[3])}, {V(regs[4])}",
            f"v_max3_f32 {m}, {m}, {V(regs[5])}, {V(regs[6])}",
            f"v_max_f32 {m}, {m}, {V(regs[7])}"]


def row_regs(s_base, qt):
    """the eight scores of a query of tile qt that a lane holds"""
    return [s_reg(s_base, kt, qt, i) for kt in range(2) for i in range(4)]


def across_lanes_lines(m, other):
    """m = its maximum over the four lanes that share a query"""
    out = []
    for x in (XL16, XL32):
        out += [f"ds_bpermute_b32 {other}, {V(x)}, {m}", "s_waitcnt lgkmcnt(0)", f"v_max_f32 {m}, {m}, {other}"]
    return out


def tile_max_ops(s_base):
    """ops leaving the maximum over a lane's eight scores of each query tile in MX[qt]."""
    return [ln for qt in range(QT) for ln in row_max_lines(V(MX[qt]), row_regs(s_base, qt))]


def emit_mask(E, s_base, valid_sreg):
    """Scores of keys at or past `valid` (keys of this 32-key step) become -inf, all query tiles."""
    E.e(f"v_mov_b32 {V(RT[0])}, 0xff800000")
    for kt in range(2):
        for i in range(4):
            E.e(f"s_sub_i32 s{S_T}, s{valid_sreg}, {8 * kt + i}")
            E.e(f"v_cmp_lt_i32 vcc, {V(KIDX)}, s{S_T}")             # key row < valid
            E.e("s_nop 1")                                          # (vcc is read by a vector instruction)
            for qt in range(QT):
                r = V(s_reg(s_base, kt, qt, i))
                E.e(f"v_cndmask_b32 {r}, {V(RT[0])}, {r}, vcc")


def emit_first_reference(E, s_base):
    """The exponent reference of a row starts as the maximum of its first tile (at s_base, its
    per-lane maxima in MX): the tile moves by it and -m_ref becomes known.  Nothing has been
    accumulated yet, so there is nothing to rescale."""
    E.e("s_nop 15\ns_nop 15\ns_nop 15")                   # every MFMA issued so far has written back
    for qt in range(QT):
        m = V(MX[qt])
        for ln in across_lanes_lines(m, V(RT[3])) + base.finite_reference_lines(m, V(RT[3])):
            E.e(ln)
        for i in range(4):
            E.e(f"v_sub_f32 {V(NT[qt] + i)}, 0, {m}")
        for r in row_regs(s_base, qt):
            E.e(f"v_sub_f32 {V(r)}, {V(r)}, {m}")


def emit_mask_check(E, s_base, pg_sreg, sub):
    """If the tile at s_base is the ragged tail of a block's last page: mask it and redo its max."""
    cold, back = E.label("MASK"), E.label("MBACK")
    E.e(f"s_cmp_eq_u32 s{pg_sreg}, s{S_PM1}")
    E.e(f"s_cselect_b32 s{S_T + 8}, s{S_VLAST + sub}, 32")
    E.e(f"s_cmp_lt_u32 s{S_T + 8}, 32")
    E.e(f"s_cbranch_scc1 {cold}")
    E.e(f"{back}:")
    sub_e = Emitter()
    emit_mask(sub_e, s_base, S_T + 8)
    E.cold.append(f"{cold}:")
    E.cold.append("s_nop 15\ns_nop 15\ns_nop 15")
    E.cold.extend(sub_e.lines)
    E.cold.extend(tile_max_ops(s_base))
    E.cold.append(f"s_branch {back}")


def p_word(p_base, j):
    """VGPR of the packed pair that ends at element j (odd) of the tile being exponentiated; element
    16 kt + 4 qt + i."""
    return p_base + 4 * ((j & 15) >> 2) + 2 * (j >> 4) + ((j & 3) >> 1)


CAP = 4.0            # issue quanta per MFMA slot the scheduler may fill
E_SPREAD = 48        # the 32 exponentials of a step are due by this slot
E_HARD = 56          # ... and issue by this one
THRESH = "0x47800000"     # 2^16: a step's sum of 8 probabilities above this moves the reference
K_BARRIER_SLOT = 32  # step 2: K(q+1) visible, slot of K(q) free
N_KLOADS_R2 = 3      # of the 8 loads of K(q+2), how many issue in step 2 (the rest in step 3)

# Operand reads: fragment -> slot it is read in.  Fragment f goes to registers FR + 4 (f % 8): V's take the place of
# K's as those have been multiplied, and the next step's K's the place of V's; K fragment 7 of a step
# is read in its own slot 1.
V_READS = {8 + i: 16 + 2 * i for i in range(4)} | {12: 32, 13: 34, 14: 36, 15: 37}
K_READS = {0: 38, 1: 41, 2: 45, 3: 48, 4: 53, 5: 56, 6: 60}
# lgkmcnt of the waits before the slots that first use a fragment: what was read later may still be on its way
WAITS = {15: 0, 31: 0, 47: 3, 63: 3}


def build_step(R, par, tails=False, short=False):
    """One 32-key step as a list of SLOTS slots: (MFMA line, [lines issued after it]).  short: steps 0 and 3 of a short page."""
    cur, nxt = ("A", "B") if R % 2 == 0 else ("B", "A")
    s_cur, s_next = S_TILE[cur], S_TILE[nxt]
    p_prev, p_cur = (P_TILE["B"], P_TILE["A"]) if R % 2 == 0 else (P_TILE["A"], P_TILE["B"])
    nR, npar = ((R + 1) & 3, par if R < 3 else 1 - par)
    if short and R == 0:
        nR, npar = 3, par
    of = "S" if short else ""
    cold, back = f"COLD{of}_{R}_{par}_%=", f"BACK{of}_{R}_{par}_%="

    head, tail = [[] for _ in range(SLOTS)], [[] for _ in range(SLOTS)]
    mfma = [mfma_qk(s_next, *x) for x in qk_order()] + pv_order(p_prev)
    head[1].append(ds_read_frag(7, frag_source(R, par, 7)))
    for f, at in V_READS.items():
        head[at].append(ds_read_frag(f, frag_source(R, par, f, tails, short and R == 3)))
    for f, at in K_READS.items():
        head[at].append(ds_read_frag(f, frag_source(nR, npar, f)))
    for at, n in WAITS.items():
        tail[at].append(f"s_waitcnt lgkmcnt({n})")
    barriers(R, short, tail, K_BARRIER_SLOT)

    atoms = []
    # row sums of the previous step join the running sums; this step's start afresh
    lacc = [Atom([f"v_add_f32 {V(LACC + qt)}, {V(LACC + qt)}, {V(TS[qt])}"], 0, qt, hard=6) for qt in range(QT)]
    atoms += lacc
    exps = [Atom([f"v_exp_f32 {V(PX + e)}, {V(s_cur + e)}"], 0, (e * E_SPREAD) // 32, hard=E_HARD) for e in range(32)]
    atoms += exps
    last_sum = [None] * QT
    for j in range(1, 32, 2):                              # the pair (j - 1, j) of query tile qt
        qt, deps, dl = (j & 15) >> 2, [exps[j - 1], exps[j]], (j * E_SPREAD) // 32 + 6
        atoms.append(Atom([f"v_cvt_pk_bf16_f32 {V(p_word(p_cur, j))}, {V(PX + j - 1)}, {V(PX + j)}"], 0, dl, deps, 2, hard=E_HARD + 4))
        if last_sum[qt] is None:
            sums = [Atom([f"v_add_f32 {V(TS[qt])}, {V(PX + j - 1)}, {V(PX + j)}"], 0, dl + 2, deps, 2, hard=E_HARD + 4)]
            sums[0].after.append((lacc[qt], 0))
        else:
            sums = [Atom([f"v_add_f32 {V(TS[qt])}, {V(TS[qt])}, {V(PX + k)}"], 0, dl + 2, deps, 2, hard=E_HARD + 4) for k in (j - 1, j)]
            sums[0].after.append((last_sum[qt], 0))
            sums[1].after.append((sums[0], 0))
        atoms += sums
        last_sum[qt] = sums[-1]
    # is the tile just produced the ragged tail of a block's last page?
    pg, sub = (S_PGCUR, R + 1) if R < 3 else (S_PGNEXT, 0)
    rag = Atom([f"s_cmp_eq_u32 s{pg}, s{S_PM1}",
                f"s_cselect_b64 s[{S_RG}:{S_RG + 1}], s[{S_VLP + 2 * sub}:{S_VLP + 2 * sub + 1}], 0"], 0, 12, hard=44)
    top = V(RT[1])
    det = Atom([f"v_max3_f32 {top}, {V(TS[0])}, {V(TS[1])}, {V(TS[2])}", f"v_max_f32 {top}, {top}, {V(TS[3])}",
                f"v_cmp_lt_f32 vcc, {THRESH}, {top}"], 0, E_HARD + 5, last_sum, 0, hard=E_HARD + 5)
    # scc travels from here to the branch after the last MFMA: nothing that writes scc may
    # issue behind it (every such atom has hard <= 55)
    orr = Atom([f"s_or_b64 s[{S_T + 8}:{S_T + 9}], vcc, s[{S_RG}:{S_RG + 1}]"], 62, 62, [det, rag], 1, hard=62)
    atoms += [rag, det, orr]
    tail[SLOTS - 1].insert(0, f"{back}:")
    tail[SLOTS - 1].insert(0, f"s_cbranch_scc1 {cold}")
    # page traffic
    if R == 0:                                             # address of V(q+1), then of K(q+2)
        prev = None
        for k, grp in enumerate(v_address_lines() + page_advance_lines()):
            prev = Atom(grp, 4, 12 + 6 * k, [prev] if prev else [], 1, hard=55)
            atoms.append(prev)
    if R == 1:                                             # V(q+1) into the slot V(q-1) left
        atoms += page_load_atoms([(page_load_lines(i, VRING + (1 - par) * PAGE, 1), 3 + (i * 52) // 8) for i in range(8)], 0, 55)
    if R == 2:                                             # K(q+2) into the slot K(q) left
        atoms += page_load_atoms([(page_load_lines(i, par * PAGE, 0), K_BARRIER_SLOT + 4 + (i * (52 - K_BARRIER_SLOT)) // N_KLOADS_R2)
                                  for i in range(N_KLOADS_R2)], K_BARRIER_SLOT, 55)
    if R == 3:
        n = 8 - N_KLOADS_R2
        if short:                                          # V(q+1), then K(q+2)
            atoms += page_load_atoms([(page_load_lines(i % 8, par * PAGE if i >= 8 else VRING + (1 - par) * PAGE, i < 8), 4 + (i * 50) // 16)
                                      for i in range(16)], 0, 55, tight=True)
        else:
            atoms += page_load_atoms([(page_load_lines(N_KLOADS_R2 + i, par * PAGE, 0), 4 + (i * 52) // n) for i in range(n)], 0, 55)
        # page-in-block counters of pages q and q+1 move on; one page less to go
        pe = Atom([f"s_mov_b32 s{S_PGCUR}, s{S_PGNEXT}", f"s_add_u32 s{S_T}, s{S_PGNEXT}, 1",
                   f"s_cmp_eq_u32 s{S_T}, s{S_P}", f"s_cselect_b32 s{S_PGNEXT}, 0, s{S_T}",
                   f"s_sub_u32 s{S_NLEFT}, s{S_NLEFT}, 1"], 0, 40, [rag], 1, hard=55)
        atoms.append(pe)
        if tails:
            atoms += last_step_atoms(sys.modules[__name__], pe, 1 if short else 3, 55)

    fixed = [split_cost(head[i] + tail[i]) for i in range(SLOTS)]
    placed = schedule16(fixed, atoms, CAP)
    for i in range(62, SLOTS):
        for a in placed[i]:
            assert not any(l.split()[0].startswith(("s_add", "s_sub", "s_cmp", "s_and", "s_mul")) for l in a.lines), a.lines
    slots = []
    for i in range(SLOTS):
        # what is not vector work goes first; nothing of the step may stand behind the branch at its end
        atom_lines = [[l for a in placed[i] for l in a.lines if is_vector(l) == vec] for vec in (False, True)]
        if i == SLOTS - 1:
            lines = atom_lines[0] + atom_lines[1] + tail[i]
        else:
            lines = tail[i] + head[i] + atom_lines[0] + atom_lines[1]
        slots.append((mfma[i], lines))
    return slots, (s_cur, s_next, p_cur, cold, back, (S_VLAST + (R + 1 if R < 3 else 0)))


def rescale_lines(s_cur, s_next, p_cur):
    """As gen_attn_core's: the reference moves, the step's probabilities are formed again, what earlier steps left is scaled."""
    c = []
    for qt in range(QT):
        m, delta, alpha = V(MX[qt]), V(MX[qt]), V(RT[6])
        regs = row_regs(s_cur, qt)
        c += row_max_lines(m, regs)
        c += across_lanes_lines(m, V(RT[3]))
        c.append(f"v_max_f32 {delta}, 0, {delta}")                  # the reference never moves down
        c.append(f"v_exp_f32_e64 {alpha}, -{delta}")
        c.append("s_nop 3")                              # a trans result is not forwarded to the next VALU op
        c.append(f"v_mul_f32 {V(LACC + qt)}, {V(LACC + qt)}, {alpha}")
        for dt in range(8):
            for i in range(4):
                acc = A(o_reg(dt, qt, i))
                tmp = V(RT[8 + (4 * dt + i) % 8])
                c.append(f"v_accvgpr_read_b32 {tmp}, {acc}")
                c.append(f"v_mul_f32 {tmp}, {tmp}, {alpha}")
                c.append(f"v_accvgpr_write_b32 {acc}, {tmp}")
        for r in regs:                                   # the step's probabilities again
            c.append(f"v_sub_f32 {V(r)}, {V(r)}, {delta}")
        es = [r - s_cur for r in regs]
        for e in es:
            c.append(f"v_exp_f32 {V(PX + e)}, {V(s_cur + e)}")
        c.append("s_nop 3")
        c.append(f"v_add_f32 {V(TS[qt])}, {V(PX + es[0])}, {V(PX + es[1])}")
        for e in es[2:]:
            c.append(f"v_add_f32 {V(TS[qt])}, {V(TS[qt])}, {V(PX + e)}")
        for j in es[1::2]:
            c.append(f"v_cvt_pk_bf16_f32 {V(p_word(p_cur, j))}, {V(PX + j - 1)}, {V(PX + j)}")
        for i in range(4):                               # -m_ref operand and the tile just produced
            c.append(f"v_sub_f32 {V(NT[qt] + i)}, {V(NT[qt] + i)}, {delta}")
        for r in row_regs(s_next, qt):
            c.append(f"v_sub_f32 {V(r)}, {V(r)}, {delta}")
    return c


def emit_drain(E, par_last, tails=False):
    """PV of the final step: V page (parity par_last), keys 96..127 (or of the last step walked), P tile B."""
    for qt in range(QT):                                  # row sums of the final step
        E.e(f"v_add_f32 {V(LACC + qt)}, {V(LACC + qt)}, {V(TS[qt])}")
    for dt in range(8):
        E.e(f"ds_read_b128 {V(FR + 4 * dt, 4)}, {V(XOVL if tails else XOV + 3)} offset:{par_last * PAGE + dt * 4096}")
    E.e("s_waitcnt lgkmcnt(0)")
    for ln in pv_order(P_TILE["B"]):
        E.e(ln)


def emit_idle(E, done, vmcnt, tails=False):
    """A wave without a single query row (the last tile of a segment has up to three) only takes its part in
    moving pages: the lines of a step that do so, and the barriers, in a loop of their own.  Its matrix
    work would cost power that the others can use (half-size 1.3B grid, five blocks: one wave in twenty)."""
    idle = E.label("IDLE")
    E.e("s_cmp_ge_i32 %[idle], 0")
    E.e("s_nop 0")
    E.e(f"s_cbranch_scc1 {idle}")

    def page(F, par, short):
        c = F.lines
        for R in (0, 3) if short else range(4):
            for _, lines in build_step(R, par, tails, short)[0]:
                for ln in lines:
                    if ln.startswith(("global_load", "v_readlane", "s_")) and not ln.startswith(("s_cbranch", "s_or", "s_waitcnt lgkmcnt")):
                        if ln.startswith("global_load") and " m0," in c[-1]:
                            c.append("s_nop 0")           # (what stands between in a working wave is left out here)
                        c.append(ln.replace("@VMCNT_V@", str(vmcnt[0])).replace("@VMCNT_K@", str(vmcnt[1])))

    F = Emitter(E)
    F.e(f"{idle}:")
    if tails:
        emit_pages_with_tails(F, "I", page, (done, done))
    else:
        for par in range(2):
            page(F, par, False)
            F.e(f"s_cmp_eq_u32 s{S_NLEFT}, 0")
            F.e("s_nop 0")
            F.e(f"s_cbranch_scc1 {done}")
        F.e(f"s_branch {idle}")
    E.cold += F.lines + F.cold


def emit_operand_setup(E):
    E.e(f"v_mov_b32 {V(KIDX)}, %[kidx]")
    E.e(f"v_mov_b32 {V(XL16)}, %[xl16]")
    E.e(f"v_mov_b32 {V(XL32)}, %[xl32]")
    for j in range(4):
        E.e(f"v_xor_b32 {V(XOK + j)}, {j << 6}, %[xk0]")
        E.e(f"v_add_u32 {V(XOK + j)}, s{S_LDS0}, {V(XOK + j)}")
        E.e(f"v_xor_b32 {V(XOV + j)}, {j << 6}, %[xv0]")
        E.e(f"v_add_u32 {V(XOV + j)}, s{S_LDS0}, {V(XOV + j)}")
        E.e(f"v_add_u32 {V(XOV + j)}, {VRING}, {V(XOV + j)}")


def emit_clear(E):
    for qt in range(QT):
        E.e(f"v_mov_b32 {V(LACC + qt)}, 0")
        E.e(f"v_mov_b32 {V(TS[qt])}, 0")


def emit_first_tile(E):
    """S tile of step 0 into tile A, its mask, max and reference"""
    for f in range(8):
        E.e(ds_read_frag(f, k_source(0, 0, f)))
    E.e("s_waitcnt lgkmcnt(0)")
    clear = base.clear_accumulator_lines(32)
    for x in qk_order():
        E.e(mfma_qk(S_TILE["A"], *x, "0"))
        E.lines += next(clear)
    E.e("s_nop 15\ns_nop 15\ns_nop 15")
    for op in tile_max_ops(S_TILE["A"]):
        E.e(op)
    emit_mask_check(E, S_TILE["A"], S_PGCUR, 0)
    emit_first_reference(E, S_TILE["A"])


def emit_first_reads(E):
    """first operand fragments of step (R=0, parity 0)"""
    for f in K_READS:
        E.e(ds_read_frag(f, frag_source(0, 0, f)))
    E.e(f"s_waitcnt lgkmcnt({WAITS[SLOTS - 1]})")


emit_results = base.emit_results


def generate(tails=False):
    return base.generate(sys.modules[__name__], tails)


def main(out_path):
    # registers the block uses beyond its operands (v148..v151 and NT are outputs)
    clob = [f"v{i}" for i in range(128, 256) if not 148 <= i <= 151 and i not in NT]
    clob += [f"a{i}" for i in range(0, 128)] + [f"s{i}" for i in range(36, 96)]
    base.write_include(out_path, generate(), clob, "CA_CORE16_CLOBBERS")
    base.write_lines(out_path.replace("_gfx950", "_tails_gfx950"), generate(tails=True))


if __name__ == "__main__":
    main(sys.argv[1] if len(sys.argv) > 1 else "attn_core16_gfx950.inc")
