"""CPU tests of the code generators of the hand-scheduled kernels: the list scheduler honours its
constraints, and the emitted instruction streams keep the invariants the kernels rely on (hazard
distances, condition-code lifetimes, load / barrier / wait bookkeeping).  Nothing is assembled or
run here; the GPU parity tests cover what the code computes."""
import importlib.util
import os
import re
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_20426_amd", "csrc")


def _load(name):
    spec = importlib.util.spec_from_file_location(name, os.path.join(CSRC, name + ".py"))
    mod = sys.modules[name] = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


sched = _load("issue_sched")
attn = _load("gen_attn_core")
attn16 = _load("gen_attn_core16")
gemm = _load("gen_gemm_core")

SCC_WRITERS = ("s_add", "s_sub", "s_cmp", "s_and", "s_or", "s_mul", "s_lsh", "s_min", "s_max")


def _m0_writes(text):
    """Lines that write M0, by place, after checking that writes and loads to LDS alternate and that a load never follows its
    write directly: it takes M0 one wait state after a scalar instruction wrote it."""
    writes, open_write = {}, None
    for k, ln in enumerate(text):
        if " m0," in ln:
            assert open_write is None, (k, ln)
            writes[k] = ln
            open_write = k
        elif ln.startswith("global_load_lds"):
            assert open_write is not None and k >= open_write + 2, (k, ln)
            open_write = None
    assert open_write is None
    return writes


def test_loads_to_lds_keep_their_distance_from_the_m0_write():
    for gen, n in ((attn, 8 + 2 * 16), (attn16, 8 + 2 * 2 * 16), (gemm, 40 + 16 * gemm.PERIOD)):
        assert len(_m0_writes([p for ln in gen.generate() for p in ln.split("\n")])) == n
    # the inline assembly of the kernels around the loops
    found = 0
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".hip", ".hpp")):
            with open(os.path.join(CSRC, name)) as f:
                for body in re.findall(r'asm volatile\("((?:[^"\\]|\\.)*)"', f.read()):
                    lines = [x.strip() for x in body.replace("\\t", "").split("\\n")]
                    found += len(_m0_writes(lines))
    assert found == 3


def test_scheduler_respects_ready_order_gaps_and_hard_deadlines():
    rng = np.random.default_rng(7)
    for trial in range(20):
        n = 32
        atoms = []
        for k in range(40):
            after = [atoms[j] for j in rng.choice(len(atoms), size=min(len(atoms), int(rng.integers(0, 3))), replace=False)] if atoms else []
            ready = int(rng.integers(0, 20))
            atoms.append(sched.Atom(["v_add_f32 v0, v0, v0"] * int(rng.integers(1, 3)), ready, int(rng.integers(ready, n)),
                                    after, int(rng.integers(0, 3)), hard=n - 1))
        placed = sched.schedule([2.0] * n, atoms, 8.0)
        assert sorted(id(a) for s in placed for a in s) == sorted(id(a) for a in atoms)     # each exactly once
        pos = {id(a): (i, k) for i, s in enumerate(placed) for k, a in enumerate(s)}
        for a in atoms:
            assert a.slot == pos[id(a)][0] and a.slot >= a.ready
            for dep, gap in a.after:
                assert a.slot >= dep.slot + gap
                assert pos[id(a)] > pos[id(dep)]                                             # issue order too
        for i, s in enumerate(placed):                                                         # no overflow: all of it fits
            assert 2.0 + sum(a.cost for a in s) <= 8.0 + 1e-9 or any(a.hard <= i for a in s)
    # an atom larger than any slot takes the first one that holds nothing else; one that finds no
    # room before its hard deadline is placed there regardless
    big = sched.Atom(["v_exp_f32 v1, v2"] * 5, 2, 3, hard=5)
    small = [sched.Atom(["v_add_f32 v0, v0, v0"] * 6, 0, 0, hard=7) for _ in range(3)]
    placed = sched.schedule([2.0] * 8, small + [big], 8.0)
    assert big.slot == 3 and [a.slot for a in small] == [0, 1, 2] and placed[3] == [big]
    late = sched.Atom(["v_add_f32 v0, v0, v0"] * 4, 0, 0, hard=1)
    placed = sched.schedule([2.0] * 4, [sched.Atom(["v_add_f32 v0, v0, v0"] * 6, 0, 0, hard=3) for _ in range(2)] + [late], 8.0)
    assert late.slot == 1


def test_quanta_model():
    q = sched.quanta
    assert q("v_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]") == 2.0
    assert q("v_exp_f32 v1, v2") == 2.0 and q("ds_read_b128 v[0:3], v4 offset:16") == 2.2
    assert q("global_load_lds_dwordx4 v1, s[2:3]") == 2.7 and q("s_cbranch_scc1 X") == 2.5
    assert q("s_waitcnt lgkmcnt(0)") == 1.0 and q("LABEL_1:") == 0.0 and q("; comment") == 0.0


def _steps():
    return [(R, par, attn.build_step(R, par)) for par in range(2) for R in range(4)]


def test_attention_step_invariants():
    exp_re = re.compile(r"v_exp_f32 (v\d+), (v\d+)")
    for R, par, (slots, cold) in _steps():
        assert len(slots) == 32 and all(m.startswith("v_mfma_f32_32x32x16_bf16") for m, _ in slots)
        flat = [(i, ln) for i, (m, lines) in enumerate(slots) for ln in [m] + lines]
        text = [ln for _, ln in flat]
        # 32 exponentials, 16 packs, row-sum adds for every probability exactly once
        exps = {m.group(1): i for i, ln in flat for m in [exp_re.match(ln)] if m}
        assert len(exps) == 32
        packs = [(i, ln) for i, ln in flat if ln.startswith("v_cvt_pk_bf16_f32")]
        assert len(packs) == 16
        used = []
        for i, ln in flat:
            if ln.startswith(("v_cvt_pk_bf16_f32", "v_add_f32")):
                for reg in re.findall(r"v\d+", ln.split(",", 1)[1]):
                    if reg in exps:
                        assert i >= exps[reg] + 2, (R, ln)      # a trans result is consumed >= 2 slots later
                        used.append((ln.split()[0], reg))
        assert sorted(r for op, r in used if op == "v_cvt_pk_bf16_f32") == sorted(exps)
        assert sorted(r for op, r in used if op == "v_add_f32") == sorted(exps)
        # scc set by the s_or survives until the branch that ends the step
        k_or = max(k for k, ln in enumerate(text) if ln.startswith("s_or_b64"))
        k_br = max(k for k, ln in enumerate(text) if ln.startswith("s_cbranch_scc1"))
        assert k_br > k_or + 1                                  # not directly behind the s_or
        assert not any(ln.split()[0].startswith(SCC_WRITERS) for ln in text[k_or + 1:k_br])
        # the compare that feeds it sits at least a slot before
        i_cmp = max(i for i, ln in flat if ln.startswith("v_cmp_lt_f32 vcc"))
        i_or = max(i for i, ln in flat if ln.startswith("s_or_b64"))
        assert i_or >= i_cmp + 1
        # scc producer / consumer pairs are adjacent (no other scc writer between)
        for k, ln in enumerate(text):
            if ln.split()[0] in ("s_cselect_b32", "s_cselect_b64", "s_addc_u32"):
                back = k - 1
                while text[back].split()[0] in ("s_cselect_b32", "s_cselect_b64"):
                    back -= 1
                assert text[back].split()[0].startswith(("s_cmp", "s_add_u32", "s_addc_u32")), (R, text[back], ln)
        assert _m0_writes(text) == {k: text[k] for k, ln in enumerate(text) if ln.startswith("s_add_u32 m0")}


def test_attention_page_traffic_bookkeeping():
    """16 loads per page pair (8 V after the V barrier, 8 K after the K barrier), two barriers per
    page, and the vmcnt operands equal the number of loads issued behind the page being awaited."""
    vm_v, vm_k = attn.wait_counts()
    events = []                                   # ("load", stream) | ("bar", which), in program order over one page
    for R in range(4):
        slots, _ = attn.build_step(R, 0)
        for m, lines in slots:
            for k, ln in enumerate(lines):
                if ln.startswith("global_load_lds"):
                    events.append(("load", "V" if "s[76:77]" in ln else "K"))
                if ln == "s_barrier":
                    wait = lines[k - 1]
                    events.append(("bar", "V" if "@VMCNT_V@" in wait else "K"))
    loads = [e[1] for e in events if e[0] == "load"]
    assert loads.count("V") == 8 and loads.count("K") == 8
    assert [e[1] for e in events if e[0] == "bar"] == ["V", "K"]           # V barrier ends step 0, K barrier in step 2
    two = events + events                         # two consecutive pages
    for which, vm in (("V", vm_v), ("K", vm_k)):
        bars = [k for k, e in enumerate(two) if e == ("bar", which)]
        b = bars[1]                               # a barrier in the second page: awaits the loads of the first
        first_page_last = max(k for k, e in enumerate(events) if e == ("load", which))
        # every load of that stream in the previous period has at most vm loads behind it
        behind = sum(1 for e in two[first_page_last + 1:b] if e[0] == "load")
        # loads of the awaited page issued after the previous barrier of the same kind are the ones meant
        assert behind == vm, (which, behind, vm)


def test_attention_cold_blocks_have_no_barrier_and_return():
    lines = attn.generate()
    text = [p for ln in lines for p in ln.split("\n")]
    n_bar = sum(1 for ln in text if ln == "s_barrier")
    assert n_bar == 1 + 2 * 2                     # prologue + two per page, two pages per loop trip
    colds = [k for k, ln in enumerate(text) if ln.startswith("COLD_")]
    assert len(colds) == 8
    for k in colds:
        j = k
        while not text[j].startswith("s_branch BACK_"):
            assert text[j] != "s_barrier"
            j += 1


def test_gemm_stage_invariants():
    for P in range(gemm.PERIOD):
        slots = gemm.build_stage(P)
        assert len(slots) == 128 and all(m.startswith("v_mfma_f32_16x16x32_bf16") for m, _ in slots)
        text = [ln for m, lines in slots for ln in [m] + lines]
        reads = [ln for ln in text if ln.startswith("ds_read_b128")]
        loads = [k for k, ln in enumerate(text) if ln.startswith("global_load_lds_dwordx4")]
        assert len(reads) == 32 and len(loads) == 16
        assert sum(1 for ln in text if ln == "s_barrier") == 1
        k_bar = text.index("s_barrier")
        # all loads sit behind the barrier that frees their buffers, each with an M0 write of its own;
        # W goes to ring slot (P+3) % 3, X to ring slot (P+2) % 2
        assert min(loads) > k_bar
        writes = _m0_writes(text)
        for k in loads:
            m0 = re.match(r"s_add_u32 m0, s\d+, (\d+)$", writes[max(w for w in writes if w < k)])
            assert m0
            off = int(m0.group(1))
            if f"s[{gemm.S_BX}:" in text[k]:
                assert gemm.XBASE + ((P + 2) % gemm.NX) * gemm.PART <= off < gemm.XBASE + ((P + 2) % gemm.NX + 1) * gemm.PART
            else:
                assert ((P + 3) % gemm.NW) * gemm.PART <= off < ((P + 3) % gemm.NW + 1) * gemm.PART
        # the wait at the barrier lets exactly the loads issued behind the last X load fly
        kinds = ["x" if f"s[{gemm.S_BX}:" in text[k] else "w" for k in loads]
        behind = len(kinds) - 1 - max(i for i, x in enumerate(kinds) if x == "x")
        assert text[k_bar - 1] == f"s_waitcnt vmcnt({behind}) lgkmcnt(0)"
        assert kinds.count("x") == 8 and kinds.count("w") == 8
        # fragment reads: first k-step reads this stage's ring slots, second the next stage's
        for ln in text[:k_bar]:
            if ln.startswith("ds_read_b128"):
                addr = int(re.search(r", v(\d+) offset", ln).group(1))
                assert addr in (gemm.ADDRW + 2 * (P % gemm.NW) + 1, gemm.ADDRX + 2 * (P % gemm.NX) + 1)
        for ln in text[k_bar:]:
            if ln.startswith("ds_read_b128"):
                addr = int(re.search(r", v(\d+) offset", ln).group(1))
                assert addr in (gemm.ADDRW + 2 * ((P + 1) % gemm.NW), gemm.ADDRX + 2 * ((P + 1) % gemm.NX))
        assert text[-1] == "s_waitcnt lgkmcnt(0)"
        # the two k-steps use different fragment buffers; every accumulator tile is hit once per k-step
        for kk in range(2):
            accs = [re.match(r"v_mfma\S+ (a\[\d+:\d+\])", m_).group(1) for m_, _ in slots[64 * kk:64 * kk + 64]]
            assert len(set(accs)) == 64


# ---- the loop on 16x16x32 matrix instructions, and what both attention loops share

def test_schedule16_respects_ready_order_gaps_and_room():
    rng = np.random.default_rng(11)
    kinds = ["v_add_f32 v0, v0, v0", "v_exp_f32 v1, v2", "s_add_u32 s0, s0, 1", "ds_read_b128 v[0:3], v4 offset:0"]
    for trial in range(20):
        n, atoms = 160, []
        for k in range(60):
            after = [atoms[j] for j in rng.choice(len(atoms), size=min(len(atoms), int(rng.integers(0, 3))), replace=False)] if atoms else []
            ready = int(rng.integers(0, 40))
            atoms.append(sched.Atom([kinds[int(rng.integers(0, 4))] for _ in range(int(rng.integers(1, 3)))], ready, int(rng.integers(ready, n)),
                                    after, int(rng.integers(0, 3)), hard=n - 1))
        fixed = [(1.0, 0.0) if i % 4 == 0 else (0.0, 0.0) for i in range(n)]
        placed = sched.schedule16(fixed, atoms, 4.0)
        assert sorted(id(a) for s in placed for a in s) == sorted(id(a) for a in atoms)
        pos = {id(a): (i, k) for i, s in enumerate(placed) for k, a in enumerate(s)}
        for a in atoms:
            assert a.slot == pos[id(a)][0] and a.slot >= a.ready
            for dep, gap in a.after:
                assert a.slot >= dep.slot + gap and pos[id(a)] > pos[id(dep)]
        for i, s in enumerate(placed):
            other, vector = sched.split_cost([ln for a in s for ln in a.lines])
            assert sched.slot_end(other + fixed[i][0], vector + fixed[i][1]) <= 4.0 or len(s) == 1 or any(a.hard <= i for a in s)
    late = sched.Atom(["v_exp_f32 v1, v2"], 0, 9, hard=1)
    placed = sched.schedule16([(0.0, 0.0)] * 4, [sched.Atom(["v_exp_f32 v3, v4"], 0, 0, hard=3) for _ in range(3)] + [late], 4.0)
    assert late.slot == 1                                   # due last, but its hard limit has come
    # a matrix instruction takes one quantum of four and keeps vector work out for two
    assert sched.slot_end(0, 0) == 1 and sched.slot_end(0, 2) == 4 and sched.slot_end(1, 2) == 4 and sched.slot_end(2, 2) == 5


def _regs(text, kind="v"):
    """register numbers named in a piece of an instruction"""
    out = set()
    for a, b in re.findall(rf"\b{kind}\[(\d+):(\d+)\]", text):
        out |= set(range(int(a), int(b) + 1))
    return out | {int(x) for x in re.findall(rf"\b{kind}(\d+)\b", text)}


def test_attention16_step_invariants():
    exp_re = re.compile(r"v_exp_f32 (v\d+), (v\d+)")
    for par in range(2):
        for R in range(4):
            slots, cold = attn16.build_step(R, par)
            s_cur, s_next, p_cur = cold[:3]
            assert len(slots) == 64 and all(m.startswith("v_mfma_f32_16x16x32_bf16") for m, _ in slots)
            flat = [(i, ln) for i, (m, lines) in enumerate(slots) for ln in [m] + lines]
            text = [ln for _, ln in flat]
            # 32 exponentials of the present tile; every one packed once and summed once, in fp32, at least two slots later
            exps = {m.group(1): i for i, ln in flat for m in [exp_re.match(ln)] if m}
            assert len(exps) == 32
            assert set().union(*(_regs(exp_re.match(ln).group(2)) for _, ln in flat if exp_re.match(ln))) == set(range(s_cur, s_cur + 32))
            used = []
            for i, ln in flat:
                if ln.startswith(("v_cvt_pk_bf16_f32", "v_add_f32")):
                    for reg in re.findall(r"v\d+", ln.split(",", 1)[1]):
                        if reg in exps:
                            assert i >= exps[reg] + 2, (R, ln)
                            used.append((ln.split()[0], reg))
            assert sorted(r for op, r in used if op == "v_cvt_pk_bf16_f32") == sorted(exps)
            assert sorted(r for op, r in used if op == "v_add_f32") == sorted(exps)
            # the pairs of a query tile land in its P words and its sum
            for i, ln in flat:
                if ln.startswith("v_cvt_pk_bf16_f32"):
                    dst, a, b = (int(x) for x in re.findall(r"v(\d+)", ln.split(None, 1)[1]))
                    e = a - attn16.PX
                    assert b == a + 1 and e % 2 == 0 and dst == p_cur + 4 * ((e % 16) // 4) + 2 * (e // 16) + (e % 4) // 2
                if ln.startswith("v_add_f32") and not ln.startswith(f"v_add_f32 v{attn16.LACC}") and exps.keys() & set(re.findall(r"v\d+", ln)):
                    dst, *src = (int(x) for x in re.findall(r"v(\d+)", ln.split(None, 1)[1]))
                    assert all(attn16.TS[((x - attn16.PX) % 16) // 4] == dst for x in src if x >= attn16.PX)
            # the running sums take the step before's before its registers start afresh
            for qt in range(4):
                ts, acc = attn16.TS[qt], attn16.LACC + qt
                k_acc = text.index(f"v_add_f32 v{acc}, v{acc}, v{ts}")
                assert k_acc < min(k for k, ln in enumerate(text) if ln.startswith(f"v_add_f32 v{ts},"))
            # QK writes the other tile, PV reads the other P; nothing of the vector work touches either
            for i, (m, _) in enumerate(slots):
                d, a, b, c = (x.strip() for x in re.split(r",(?![^\[]*\])", m.split(None, 1)[1]))
                if i < 32:
                    assert _regs(d) <= set(range(s_next, s_next + 32)) and (c == d or _regs(c) <= set(range(184, 200)))
                else:
                    assert d == c and not _regs(b) & set(range(p_cur, p_cur + 16))
            assert len({m.split()[1] for m, _ in slots[:32]}) == 8 and len({m.split()[1] for m, _ in slots[32:]}) == 32
            # what decides about the out-of-line block: sums -> vcc -> scc -> the branch that ends the step
            k_cmp, k_or = (max(k for k, ln in enumerate(text) if ln.startswith(x)) for x in ("v_cmp_lt_f32 vcc", "s_or_b64"))
            k_br = max(k for k, ln in enumerate(text) if ln.startswith("s_cbranch_scc1"))
            assert k_cmp > max(k for k, ln in enumerate(text) if ln.startswith(tuple(f"v_add_f32 v{t}," for t in attn16.TS)))
            assert flat[k_or][0] >= flat[k_cmp][0] + 1 and k_br > k_or + 1
            assert not any(ln.split()[0].startswith(SCC_WRITERS) for ln in text[k_or + 1:k_br])
            assert sum("vcc" in ln for ln in text) == 2
            for k, ln in enumerate(text):
                if ln.split()[0] in ("s_cselect_b32", "s_cselect_b64", "s_addc_u32"):
                    back = k - 1
                    while text[back].split()[0] in ("s_cselect_b32", "s_cselect_b64"):
                        back -= 1
                    assert text[back].split()[0].startswith(("s_cmp", "s_add_u32", "s_addc_u32")), (R, text[back], ln)
            assert len(_m0_writes(text)) == [0, 8, attn16.N_KLOADS_R2, 8 - attn16.N_KLOADS_R2][R]


def _loop_text(core):
    """the main loop in program order, one trip (two pages), without the out-of-line blocks"""
    text = [p for ln in attn.generate(core) for p in ln.split("\n")]
    start = next(k for k, ln in enumerate(text) if ln.startswith("LOOP_"))
    return text, text[start + 1:next(k for k, ln in enumerate(text) if ln.startswith("s_branch LOOP_"))]


@pytest.mark.parametrize("core", [attn.CORE, attn16], ids=["32x32x16", "16x16x32"])
def test_attention_operand_fragments_have_arrived(core):
    """Two trips of the loop: every matrix instruction finds the operand fragment it is meant to have in its registers, and a
    wait has covered the read (LDS answers a wave's reads in order)."""
    _, loop = _loop_text(core)
    want = []                                               # (address register, offset) per matrix instruction
    for par in range(2):
        for R in range(4):
            if core is attn16:
                # K of the next 32-key step of the walk, V of the one before
                kp, vp = (par if R < 3 else 1 - par) * attn.PAGE, (par if R > 0 else 1 - par) * attn.PAGE
                want += [(attn16.XOK + (ks ^ (2 * kt)), kp + ((R + 1) % 4) * 8192 + kt * 2048) for kt in range(2) for qt in range(4) for ks in range(4)]
                want += [(attn16.XOV + (R - 1) % 4, vp + dt * 4096) for dt in range(8) for qt in range(4)]
            else:
                want += [attn.frag_source(R, par, i >> 1) for i in range(32)]
    held, flying, n = {}, [], 0
    for trip in range(2):
        for ln in loop:
            if ln.startswith("ds_read_b128"):
                m = re.match(r"ds_read_b128 v\[(\d+):\d+\], v(\d+) offset:(\d+)", ln)
                reg, src = int(m.group(1)), (int(m.group(2)), int(m.group(3)))
                held[reg] = src
                flying.append(reg)
            elif ln.startswith("s_waitcnt") and "lgkmcnt" in ln:
                left = int(re.search(r"lgkmcnt\((\d+)\)", ln).group(1))
                flying = flying[len(flying) - left:] if left < len(flying) else flying
                if left == 0:
                    flying = []
            elif ln.startswith("v_mfma"):
                reg = int(re.findall(r"v\[(\d+):\d+\]", ln)[1 if ln.split()[1].startswith("v") else 0])
                if reg in held or trip:                     # (the very first operands were read ahead of the loop)
                    assert held[reg] == want[n % len(want)] and reg not in flying, (n, ln)
                n += 1
            elif ln == "s_barrier":
                assert not [r for r in flying if r not in held]
    assert n == 2 * len(want)


@pytest.mark.parametrize("core", [attn.CORE, attn16], ids=["32x32x16", "16x16x32"])
def test_attention_pages_are_there_when_read(core):
    """The page loop's loads, waits and barriers over eight pages: a read finds the page it is meant to have, published by a
    barrier behind a wait that covers the page's last load, and no load goes to a slot that a wave may still read."""
    _, loop = _loop_text(core)
    # K(0), V(0), K(1) requested ahead of the loop in this order, the first two published
    queue, published = [("K", 1)] * 8, {("K", 0), ("V", 0)}
    slot_of = {"K": {0: 0, 1: 1}, "V": {0: 0, 1: None}}      # page held (or on its way) per ring slot
    last_reads, n_load, m0 = {}, {"K": 16, "V": 8}, None
    barriers = 0
    for trip in range(4):
        step = mfma = 0
        for ln in loop:
            if " m0," in ln:
                m0 = int(ln.split()[-1])
            elif ln.startswith("global_load_lds"):
                which = "V" if f"s[{attn.S_ADDRV}:" in ln else "K"
                pg = n_load[which] // 8
                slot = (m0 - (attn.VRING if which == "V" else 0)) // attn.PAGE
                assert slot == pg % 2 and (m0 % attn.PAGE) // 4096 == n_load[which] % 8
                old = slot_of[which][slot]
                if old is not None and old != pg:           # the page that leaves: its last read lies before the last barrier
                    assert last_reads.get((which, old), -1) < barriers, (which, old, pg)
                slot_of[which][slot] = pg
                published.discard((which, old))
                queue.append((which, pg))
                n_load[which] += 1
            elif ln.startswith("s_waitcnt vmcnt"):
                left = int(re.search(r"vmcnt\((\d+)\)", ln).group(1))
                queue = queue[len(queue) - left:] if left < len(queue) else queue
            elif ln == "s_barrier":
                barriers += 1
                for which in "KV":
                    for slot, pg in slot_of[which].items():
                        if pg is not None and (which, pg) not in queue and n_load[which] >= 8 * (pg + 1):
                            published.add((which, pg))
            elif ln.startswith("ds_read_b128"):
                reg, imm = (int(x) for x in re.match(r"ds_read_b128 \S+ v(\d+) offset:(\d+)", ln).groups())
                is_v = reg >= core.XOV if core is attn16 else reg >= attn.XOV
                which, slot = ("V" if is_v else "K"), (imm // attn.PAGE) % 2
                pg = slot_of[which][slot]
                if which == "V" and pg is None:             # the all-zero P of the first step
                    assert trip == 0 and step == 0
                    continue
                assert (which, pg) in published, (which, pg, trip, step)
                last_reads[(which, pg)] = barriers
            elif ln.startswith("v_mfma"):
                mfma += 1
                step = mfma // core.SLOTS
    assert barriers == 16


def test_attention16_idle_waves_move_the_same_pages():
    """A wave without query rows: the same loads to the same places, waits for them and barriers, in the same order, and nothing else
    that another wave could see."""
    text, loop = _loop_text(attn16)
    start = next(k for k, ln in enumerate(text) if re.match(r"IDLE_\d+_%=:", ln))
    idle = text[start + 1:next(k for k, ln in enumerate(text) if ln.startswith("s_branch IDLE_"))]

    def traffic(lines):
        return [ln for ln in lines if ln.startswith(("global_load", "s_waitcnt vmcnt", "s_barrier", "v_readlane", "s_mul", "s_add", "s_sub",
                                                     "s_mov", "s_cmp", "s_cselect"))]
    assert traffic(idle) == traffic(loop)
    assert not any(ln.startswith(("ds_", "v_mfma", "global_store")) for ln in idle)
    assert len(_m0_writes(idle)) == 32
    assert sum(ln.startswith("s_cbranch_scc1 DONE_") for ln in idle) == 2       # it leaves after the same page
    for k, ln in enumerate(idle):
        if ln.startswith("s_cbranch"):
            assert idle[k - 2] == f"s_cmp_eq_u32 s{attn.S_NLEFT}, 0" and idle[k - 1] == "s_nop 0"


def test_attention16_cold_blocks_have_no_barrier_and_return():
    text, _ = _loop_text(attn16)
    assert sum(1 for ln in text if ln == "s_barrier") == 1 + 2 * 2 + 2 * 2       # prologue, the loop, the loop of idle waves
    colds = [k for k, ln in enumerate(text) if ln.startswith("COLD_")]
    assert len(colds) == 8
    for k in colds:
        j = k
        while not text[j].startswith("s_branch BACK_"):
            assert text[j] != "s_barrier" and not text[j].startswith(("global_load", "ds_read"))
            j += 1
        block = text[k:j]
        # the step's sums start again from the probabilities formed anew, the running ones are scaled
        for qt in range(4):
            ts = attn16.TS[qt]
            assert sum(ln.startswith(f"v_add_f32 v{ts},") for ln in block) == 7
            assert sum(ln.startswith(f"v_mul_f32 v{attn16.LACC + qt},") for ln in block) == 1


class _Walk:
    """Runs a generated attention loop for one wave on the CPU as far as control, page traffic and operands go: scalar instructions are
    interpreted, memory to LDS loads, barriers, waits and operand reads are followed with the page they concern, no row sum ever
    exceeds its limit.  Leaves the 32-key steps multiplied (K side and V side), the tiles masked, and the barriers met."""
    BLOCK = 1 << 20                                          # bytes from one KV block's first page to the next one's

    def __init__(self, core, text, n_pages, ppb, last_valid, n_kvb, kb0, pg0, idle=False):
        self.core, self.text = core, text
        self.stride = 2 * attn.PAGE
        self.label = {ln[:-1]: k for k, ln in enumerate(text) if ln.endswith(":")}
        self.s = {}
        self.arg = {"n_pages": n_pages, "ppb": ppb, "stride": self.stride, "n_kvb": n_kvb, "kb0": kb0, "pg0": pg0, "last_valid": last_valid,
                    "wave": 0, "lds0": 0, "idle": 0 if idle else -1}
        self.scc = 0
        self.moved = {}                                      # v_mov_b32 of one LDS address register to another
        self.queue, self.slot, self.ready, self.read_at = [], {}, set(), {}
        self.held, self.flying = {}, []
        self.barriers, self.k_tiles, self.v_steps, self.masked, self.n_mfma = 0, [], [], {}, {"K": 0, "V": 0}
        self.traffic = []
        for which in "KV":                                   # requested ahead of the block, oldest first
            self.slot[which, 0] = [(kb0, pg0), 8]
            self.queue += [(which, 0)] * 8
        self.run()

    def val(self, x):
        x = x.strip()
        if x.startswith("%["):
            return self.arg[x[2:-1]]
        if x == "vcc":
            return 0
        if x.startswith("s["):
            a = int(x[2:].split(":")[0])
            return self.s.get(a, 0) | self.s.get(a + 1, 0) << 32
        if re.fullmatch(r"s\d+", x):
            return self.s.get(int(x[1:]), 0)
        if x == "m0":
            return self.m0
        if "-" in x[1:]:                                     # a difference of labels
            a, b = x.split("-", 1)
            return self.label[a] - self.label[b]
        return int(x, 0) & 0xffffffff

    def put(self, d, v):
        d = d.strip()
        if d == "m0":
            self.m0 = v & 0xffffffff
        elif d.startswith("s["):
            a = int(d[2:].split(":")[0])
            self.s[a], self.s[a + 1] = v & 0xffffffff, (v >> 32) & 0xffffffff
        else:
            self.s[int(d[1:])] = v & 0xffffffff

    def page_at(self, addr):
        return addr // self.BLOCK, addr % self.BLOCK // self.stride, "V" if addr % self.stride >= attn.PAGE else "K"

    def run(self):
        signed = lambda v: v - (1 << 32) if v & 0x80000000 else v
        k, steps = 0, 0
        while k < len(self.text):
            ln = self.text[k]
            k, steps = k + 1, steps + 1
            assert steps < 400000
            if ln.endswith(":") or ln.startswith(";"):
                continue
            op, _, rest = ln.partition(" ")
            a = [x.strip() for x in re.split(r",(?![^\[]*\])", rest)]
            if op in ("s_mov_b32", "s_mul_i32", "s_mul_hi_u32", "s_lshl_b32", "s_add_u32", "s_addc_u32", "s_sub_u32", "s_subb_u32", "s_sub_i32",
                      "s_max_i32", "s_min_i32", "s_cselect_b32", "s_cselect_b64", "s_or_b64"):
                x, y = (self.val(v) for v in (a[1:3] if len(a) > 2 else (a[1], a[1])))
                if op == "s_mov_b32":
                    self.put(a[0], x)
                elif op == "s_mul_i32":
                    self.put(a[0], x * y)
                elif op == "s_mul_hi_u32":
                    self.put(a[0], (x * y) >> 32)
                elif op == "s_lshl_b32":
                    self.put(a[0], x << y)
                elif op in ("s_add_u32", "s_addc_u32"):
                    v = x + y + (self.scc if op == "s_addc_u32" else 0)
                    self.put(a[0], v)
                    self.scc = v >> 32
                elif op in ("s_sub_u32", "s_subb_u32"):
                    v = x - y - (self.scc if op == "s_subb_u32" else 0)
                    self.put(a[0], v)
                    self.scc = int(v < 0)
                elif op == "s_sub_i32":
                    self.put(a[0], x - y)
                elif op in ("s_max_i32", "s_min_i32"):
                    self.put(a[0], (max if op == "s_max_i32" else min)(signed(x), signed(y)))
                elif op == "s_or_b64":
                    self.put(a[0], x | y)
                    self.scc = int(x | y != 0)
                else:
                    self.put(a[0], x if self.scc else y)
            elif op.startswith("s_cmp_"):
                x, y = self.val(a[0]), self.val(a[1])
                if op.endswith("i32"):
                    x, y = signed(x), signed(y)
                self.scc = int({"eq": x == y, "lg": x != y, "lt": x < y, "le": x <= y, "ge": x >= y}[op.split("_")[2]])
            elif op == "s_getpc_b64":
                self.put(a[0], k)
            elif op == "s_setpc_b64":
                k = self.val(a[0])
                assert self.text[k].startswith("BACK")
            elif op == "s_branch" or (op == "s_cbranch_scc1" and self.scc) or (op == "s_cbranch_scc0" and not self.scc) or op == "s_cbranch_vccz":
                k = self.label[a[0]]
            elif op == "v_readlane_b32":
                kb = self.val(a[2])
                assert kb < self.arg["n_kvb"]
                self.put(a[0], kb * self.BLOCK if a[1] == f"v{attn.TBLLO}" else 0)
            elif op == "global_load_lds_dwordx4":
                kb, pg, which = self.page_at(self.val(a[1]))
                assert pg < self.arg["ppb"] and which == ("V" if a[1].startswith(f"s[{attn.S_ADDRV}:") else "K")
                key = (which, self.m0 % attn.VRING // attn.PAGE)
                assert (self.m0 >= attn.VRING) == (which == "V") and self.m0 % attn.PAGE == 4096 * (int(a[0][1:]) - attn.DMAOFF)
                old = self.slot.get(key)
                if old is None or old[1] == 8:               # the page that was there: its last read lies before the last barrier
                    assert self.read_at.get(key, -1) < self.barriers
                    self.ready.discard(key)
                    old = self.slot[key] = [(kb, pg), 0]
                assert old[0] == (kb, pg)
                old[1] += 1
                self.queue.append(key)
                self.traffic.append((which, kb, pg, self.m0))
            elif op == "s_waitcnt":
                m = re.search(r"vmcnt\((\d+)\)", ln)
                if m:
                    self.queue = self.queue[len(self.queue) - int(m.group(1)):] if int(m.group(1)) else []
                    self.traffic.append(ln)
                m = re.search(r"lgkmcnt\((\d+)\)", ln)
                if m:
                    self.flying = self.flying[len(self.flying) - int(m.group(1)):] if int(m.group(1)) else []
            elif op == "s_barrier":
                self.barriers += 1
                self.traffic.append(ln)
                self.ready |= {key for key, (_, n) in self.slot.items() if n == 8 and key not in self.queue}
            elif op == "v_mov_b32" and self.core.XOVL <= int(a[0][1:] if a[0][1:].isdigit() else -1) < self.core.XOVL + self.core.XOV_STRIDE:
                self.moved[int(a[0][1:])] = int(a[1][1:])
            elif op == "ds_read_b128":
                src, imm = (int(x) for x in re.match(r"v(\d+) offset:(\d+)", a[1]).groups())
                src = self.moved.get(src, src)
                xok, xov = (self.core.XOK, self.core.XOV) if self.core is attn16 else (attn.XOK, attn.XOV)
                which = "V" if src >= xov else "K"
                key = (which, imm // attn.PAGE)
                sub = (src - xov) // self.core.XOV_STRIDE if which == "V" else imm % attn.PAGE // 8192
                reg = int(re.match(r"v\[(\d+)", a[0]).group(1))
                if key in self.slot and not (which == "V" and not self.v_steps and not self.k_tiles[1:]):
                    assert key in self.ready, (ln, key, steps)
                    self.read_at[key] = self.barriers
                    self.held[reg] = (which, *self.slot[key][0], sub, (src, imm % attn.PAGE))
                else:                                        # the all-zero P of the first step
                    self.held[reg] = (which, None, None, None, (src, imm % attn.PAGE))
                self.flying.append(reg)
            elif op.startswith("v_mfma"):
                frag = int(re.match(r"v\[(\d+)", a[1]).group(1))
                assert frag not in self.flying
                which, kb, pg, sub, _ = self.held[frag]
                per = 16 if self.core is attn.CORE else 32
                out = self.k_tiles if a[0].startswith("v") else self.v_steps
                assert which == ("K" if a[0].startswith("v") else "V")
                if self.n_mfma[which] % per == 0:
                    out.append((kb, pg, sub))
                assert out[-1] == (kb, pg, sub), (ln, out[-1], self.held[frag])
                self.n_mfma[which] += 1
            elif op == "v_cmp_lt_i32":                       # a tile is masked: what it compares key 0's offset with
                tile = len(self.k_tiles) - 1
                valid = signed(self.val(a[2]))
                self.masked[tile] = max(self.masked.get(tile, -1 << 20), valid)
            else:
                assert op.startswith(("v_", "ds_bpermute", "s_nop")) or op in ("s_cbranch_scc0", "s_cbranch_scc1", "s_cbranch_vccnz"), ln


@pytest.mark.parametrize("tails", [False, True])
@pytest.mark.parametrize("core", [attn.CORE, attn16], ids=["32x32x16", "16x16x32"])
def test_attention_walks_every_step_of_its_pages(core, tails):
    """The steps multiplied are those of the pages of the walk, in order, on both sides, the ones with absent keys masked, and a wave
    without rows moves the same pages.  With short pages two steps are walked of a block's last page of up to 64 tokens."""
    text = [p for ln in attn.generate(None if core is attn.CORE else core, tails) for p in ln.split("\n")]
    core_ = attn.CORE if core is attn.CORE else attn16
    for ppb, n_kvb, last in ((1, 4, 64), (1, 1, 7), (2, 3, 1), (3, 3, 33), (4, 3, 128), (3, 2, 65), (5, 2, 64)):
        pages = [(kb, pg) for kb in range(n_kvb) for pg in range(ppb)]
        for lo, hi in ((0, len(pages)), (0, 1), (len(pages) - 1, len(pages)), (len(pages) // 2, len(pages)), (1 % len(pages), len(pages))):
            w = _Walk(core_, text, hi - lo, ppb, last, n_kvb, *pages[lo])
            want, valid = [], []
            for kb, pg in pages[lo:hi]:
                n = min(max(last - 0, 0), 128) if pg == ppb - 1 else 128
                for sub in range(2 if tails and n <= 64 else 4):
                    want.append((kb, pg, sub))
                    valid.append(min(max(n - 32 * sub, 0), 32))
            # one tile more is formed at the end (of a page that is there again, or the last one), and one of P = 0 at the start
            assert w.k_tiles[:-1] == want and len(w.k_tiles) == len(want) + 1, (ppb, n_kvb, last, lo, hi)
            assert w.v_steps[1:] == want, (ppb, n_kvb, last, lo, hi, w.v_steps)
            for i, n in enumerate(valid):
                assert (i in w.masked) == (n < 32) and (n == 32 or w.masked[i] == n), (i, n, w.masked.get(i))
            if core is attn16:
                idle = _Walk(core_, text, hi - lo, ppb, last, n_kvb, *pages[lo], idle=True)
                assert idle.traffic == w.traffic and not idle.k_tiles and not idle.v_steps


@pytest.mark.parametrize("mt", [8, 4])
@pytest.mark.parametrize("n_stages", [2, 4, 6, 14])
def test_gemm_loops_multiply_every_stage(mt, n_stages):
    """The whole program of a tile, followed on the CPU: every product takes the fragments of its stage and k-step, read from a ring slot whose
    loads have landed and been published, behind a wait for the read; no load goes to a slot before the barrier behind its last
    read; every accumulator gets every k-step once, in order."""
    text = [p for ln in gemm.generate(mt) for p in ln.split("\n")]
    label = {ln[:-1]: k for k, ln in enumerate(text) if ln.endswith(":")}
    trips, scc, m0 = n_stages // 2, 0, None
    queue, slot, ready, last_read, barriers = [], {}, set(), {}, 0
    count = {"w": 0, "x": 0}                                 # loads issued
    per = {"w": 8, "x": mt}
    part = {"w": gemm.PART, "x": gemm.PART * mt // 8}
    depth = {"w": gemm.NW, "x": gemm.NX}
    held, flying, steps = {}, [], {}
    k = 0
    while k < len(text):
        ln = text[k]
        k += 1
        if ln.startswith("s_sub_u32") and f"s{gemm.S_TRIPS}," in ln:
            trips -= 1
            scc = int(trips != 0)
        elif ln.startswith("s_cbranch_scc1") and scc or ln.startswith("s_cbranch_scc0") and not scc and "DONE" in ln:
            k = label[ln.split()[1]]
        elif " m0," in ln:
            base, off = re.match(r"s_add_u32 m0, s(\d+), (\d+)", ln).groups()
            m0 = (int(base), int(off))
        elif ln.startswith("global_load_lds"):
            op = "x" if f"s[{gemm.S_BX}:" in ln else "w"
            assert m0[0] == (gemm.S_M0X if op == "x" else gemm.S_M0B)
            st, i = divmod(count[op], per[op])
            key = (op, st % depth[op])
            assert m0[1] == (gemm.XBASE if op == "x" else 0) + key[1] * part[op] + 1024 * i
            assert int(re.search(r" v(\d+),", ln).group(1)) == (gemm.OFFX if op == "x" else gemm.OFFW) + i
            if i == 0:
                assert last_read.get(key, -1) < barriers, (op, st)
                ready.discard(key)
                slot[key] = st
            count[op] += 1
            queue.append(key)
        elif ln.startswith("s_waitcnt"):
            m = re.search(r"vmcnt\((\d+)\)", ln)
            if m:
                queue = queue[len(queue) - int(m.group(1)):] if int(m.group(1)) else []
            if "lgkmcnt(0)" in ln:
                flying = []
        elif ln == "s_barrier":
            barriers += 1
            ready |= {key for key, st in slot.items() if key not in queue and count[key[0]] >= per[key[0]] * (st + 1)}
        elif ln.startswith("ds_read_b128"):
            reg, addr, off = (int(x) for x in re.match(r"ds_read_b128 v\[(\d+):\d+\], v(\d+) offset:(\d+)", ln).groups())
            op = "x" if addr >= gemm.ADDRX else "w"
            s, kk = divmod(addr - (gemm.ADDRX if op == "x" else gemm.ADDRW), 2)
            assert (op, s) in ready
            last_read[op, s] = barriers
            held[reg] = (op, slot[op, s], kk, off // 2048)
            flying.append(reg)
        elif ln.startswith("v_mfma"):
            acc, a, b = (int(x) for x in re.match(r"v_mfma_f32_16x16x32_bf16 a\[(\d+):\d+\], v\[(\d+):\d+\], v\[(\d+):\d+\]", ln).groups())
            assert a not in flying and b not in flying
            ti, tj = divmod(acc // 4, mt)
            n = steps.get(acc, 0)
            assert held[a] == ("w", n // 2, n % 2, ti) and held[b] == ("x", n // 2, n % 2, tj), (ln, n, held[a], held[b])
            steps[acc] = n + 1
    assert len(steps) == 8 * mt and set(steps.values()) == {2 * n_stages} and not queue
