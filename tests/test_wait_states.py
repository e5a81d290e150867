"""Wait states in the generated assembly, which the compiler does not look into: a follower of every path of a program, for the distances
that hipcc keeps on gfx950 between two instructions of its own."""
import importlib.util
import os
import re
import sys

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_20426_amd", "csrc")


def _load(name):
    spec = importlib.util.spec_from_file_location(name, os.path.join(CSRC, name + ".py"))
    mod = sys.modules[name] = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


attn, attn16, gemm, rows = (_load(name) for name in ("gen_attn_core", "gen_attn_core16", "gen_gemm_core", "gen_gemm_rows"))
TRANS = ("v_exp", "v_log", "v_rcp", "v_rsq", "v_sqrt", "v_sin", "v_cos")


def _regs(tokens):
    out = set()
    for t in tokens:
        t = t.lstrip("-")
        m = re.fullmatch(r"([vsa])\[(\d+):(\d+)\]", t)
        if m:
            out |= {f"{m[1]}{i}" for i in range(int(m[2]), int(m[3]) + 1)}
        elif t in ("vcc", "exec") or re.fullmatch(r"[vsa]\d+", t):
            out.add(t)
    return out


class _Op:
    def __init__(self, line):
        self.line = line
        self.name, _, rest = line.partition(" ")
        self.args = [x.split()[0] for x in re.split(r",(?![^\[]*\])", rest) if x.strip()]
        n = 0 if self.name.startswith(("global_store", "ds_write", "s_cmp", "s_cbranch", "s_branch", "s_waitcnt", "s_nop")) else 1
        n += self.name.startswith(("v_add_co", "v_addc_co"))
        self.writes, self.reads = _regs(self.args[:n]), _regs(self.args[n:])
        self.states = int(self.args[0], 0) + 1 if self.name == "s_nop" else 1
        self.vector = self.name.startswith("v_")


def _needed(first, then):
    """Wait states between two instructions of which the first one is a vector instruction."""
    scalars = {r for r in first.writes if r[0] == "s" or r in ("vcc", "exec")}
    need = 0
    if then.vector and scalars & then.reads:
        need = 2
    if then.name.startswith("v_readlane"):
        need = max(need, 4 if scalars & then.reads else 1 if first.writes & then.reads else 0)
    if then.name.startswith(("global_", "ds_")) and scalars & then.reads:
        need = 5
    if "_dpp" in then.name and first.writes & _regs(then.args[1:2]):
        need = max(need, 2)
    if first.name.startswith(TRANS) and then.vector and not then.name.startswith(TRANS) and first.writes & (then.reads | then.writes):
        need = max(need, 1)
    return need


def too_close(text):
    """Pairs of lines that stand too close to each other on some path of the program."""
    text = [p.strip() for ln in text for p in ln.split("\n")]
    ops = [None if ln.startswith(";") or ln.endswith(":") else _Op(ln) for ln in text]
    label = {ln[:-1]: k for k, ln in enumerate(text) if ln.endswith(":")}

    def behind(k):
        op = ops[k]
        if op is None or not op.name.startswith(("s_branch", "s_cbranch", "s_setpc")):
            return [k + 1] if k + 1 < len(ops) else []
        return [] if op.name.startswith("s_setpc") else [label[op.args[0]]] + ([k + 1] if op.name != "s_branch" else [])

    found = []
    for k, first in enumerate(ops):
        if first is None or not first.vector or first.name.startswith("v_mfma"):
            continue
        todo, best = [(n, 0) for n in behind(k)], {}
        while todo:
            at, states = todo.pop()
            if states >= 5 or best.get(at, 5) <= states:
                continue
            best[at] = states
            then = ops[at]
            if then is not None:
                if states < _needed(first, then):
                    found.append((first.line, then.line, states))
                states += then.states
            todo += [(n, states) for n in behind(at)]
    return found


@pytest.mark.parametrize("gen,kw", [(attn, {}), (attn, {"tails": True}), (attn16, {}), (attn16, {"tails": True}), (gemm, {}), (gemm, {"mt": 4}),
                                    (rows, {}), (rows, {"mt": 6}), (rows, {"mt": 4})])
def test_generated_programs_keep_the_wait_states(gen, kw):
    assert too_close(gen.generate(**kw)) == []


def test_the_follower_sees_what_stands_too_close():
    for text, n in ((["v_add_co_u32 v0, vcc, v1, v2", "v_addc_co_u32 v3, vcc, v4, v5, vcc"], 1),
                    (["v_add_co_u32 v0, vcc, v1, v2", "s_nop 1", "v_addc_co_u32 v3, vcc, v4, v5, vcc"], 0),
                    (["v_cmp_gt_f32 vcc, 0, v1", "s_branch L", "v_mov_b32 v9, v9", "L:", "v_cndmask_b32 v1, v1, v2, vcc"], 1),
                    (["v_readlane_b32 s4, v0, s5", "s_nop 1", "v_mov_b32 v1, s4"], 0), (["v_mov_b32 v0, v1", "v_readlane_b32 s4, v0, s5"], 1),
                    (["v_mov_b32 v0, v1", "s_nop 0", "v_mov_b32_dpp v2, v0 row_ror:8"], 1), (["v_exp_f32 v0, v1", "v_add_f32 v2, v0, v0"], 1)):
        assert len(too_close(text)) == n, text
