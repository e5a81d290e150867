"""Performance cases of the cascaded-attention library: what a program built on it has it do.

A case is one pass through the public entry points (CascadePool, attention_layer, linear):

  step     one cascade iteration of one attention layer: K/V of the blocks in flight published, then
           attention on unrotated queries (bf16; the kernel rotates Q while loading)
  step_f32 the same in fp32: publish, rotate Q, attend (the exact path, small sizes)
  share    one device's part of a step when the blocks in flight are spread over devices: all K/V
           published, the queries of one block rotated and attended
  layer    a whole self-attention layer: QKV projection, publication, attention, output projection
  publish  the memory-bound part alone: K/V of the blocks in flight published, Q rotated
  linear   one projection

Every pass works on the same blocks, so that it can be repeated: a block in flight may be published
again at every timestep.  Sizes are the Wan shapes of `workloads` and the small geometries of the
tests and of the smoke run.
"""
import math

import torch

from paper_2511_20426_amd import binding as B
from paper_2511_20426_amd.runner import CascadePool, attention_layer, linear

DEVICE = "cuda:0"
FRAMES = 3                                        # latent frames per block
TIMESTEPS = [0, 250, 500, 750, 1000]              # oldest block in flight is the cleanest
ROPE_DIMS = {32: (12, 10, 10), 64: (24, 20, 20), 128: (44, 42, 42)}
MODES = {"bidirectional": B.CA_BIDIRECTIONAL, "block_causal": B.CA_BLOCK_CAUSAL}
WINDOW, MAX_INFLIGHT = 6, 5                       # clean window and cascade width of the Wan configurations


def _cascade(kind, heads, grid_h, grid_w, cached, inflight, mode, **more):
    c = {"kind": kind, "heads": heads, "head_dim": 128, "grid_h": grid_h, "grid_w": grid_w, "cached": cached,
         "inflight": inflight, "sink": 0, "mode": mode}
    c.update(more)
    return c


def listed():
    return [
        # the tiny fp32 configuration: a correctness run beside a new model, all latency
        dict(_cascade("step_f32", 2, 6, 8, 2, 1, "bidirectional", head_dim=64, page_tokens=48), name="f32_tiny"),
        # fp32 at the largest size one still checks with: full head width, a cascade, ragged pages
        dict(_cascade("step_f32", 4, 12, 16, 2, 3, "block_causal", page_tokens=100), name="f32_cascade"),
        # the smallest bf16 cascade, that of the smoke run: launches and latency
        dict(_cascade("step", 3, 10, 13, 2, 3, "bidirectional"), name="small_cascade"),
        # a preview at half the height and width of the 1.3B grid, block-causal
        dict(_cascade("step", 12, 15, 26, 6, 5, "block_causal"), name="half_grid_cascade"),
        # 1.3B, one block in flight: the sequential baseline
        dict(_cascade("step", 12, 30, 52, 6, 1, "bidirectional"), name="wan1p3b_seq"),
        # 1.3B, five blocks in flight, one sink block and a full window: the long rollout's steady state
        dict(_cascade("step", 12, 30, 52, 7, 5, "block_causal", sink=1), name="wan1p3b_rollout"),
        # 14B, five blocks in flight: the headline
        dict(_cascade("step", 40, 30, 52, 6, 5, "bidirectional"), name="wan14b_cascade5"),
        # 14B, the part of the middle one of five devices
        dict(_cascade("share", 40, 30, 52, 6, 5, "block_causal", share=2), name="wan14b_share"),
        # a whole layer of the 1.3B model on one block
        dict(_cascade("layer", 12, 30, 52, 6, 1, "bidirectional", publish=False), name="layer_wan1p3b_seq"),
        # a whole layer of the 14B model on five blocks, K/V published by the projection
        dict(_cascade("layer", 40, 30, 52, 6, 5, "bidirectional", publish=True), name="layer_wan14b_cascade5"),
        # K/V of five blocks published and Q rotated at the 14B width: memory traffic only
        dict(_cascade("publish", 40, 30, 52, 0, 5, "bidirectional"), name="publish_wan14b"),
        # a projection of a few hundred tokens with ragged rows
        {"name": "linear_small", "kind": "linear", "rows": 257, "n_out": 768, "k_in": 1024},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "layer", "layer", "share", "publish", "linear", "linear", "step_f32"])
    if kind == "linear":
        return {"kind": kind, "rows": _log_int(rng, 64, 23400), "n_out": 8 * _log_int(rng, 16, 1920),
                "k_in": 128 * _log_int(rng, 2, 40)}
    mode = rng.choice(sorted(MODES))
    if kind == "step_f32":
        return _cascade(kind, rng.randint(1, 4), _log_int(rng, 4, 12), _log_int(rng, 6, 16), rng.randint(0, 2),
                        rng.randint(1, 3), mode, head_dim=rng.choice([32, 64, 128]), page_tokens=rng.choice([16, 48, 100]))
    sink = rng.choice([0, 0, 1])
    c = _cascade(kind, rng.choice([2, 3, 6, 8, 12, 16, 24, 40]), _log_int(rng, 5, 30), _log_int(rng, 8, 52),
                 rng.randint(sink, WINDOW), rng.randint(1, MAX_INFLIGHT), mode, sink=sink)
    if kind == "share":
        c["share"] = rng.randrange(c["inflight"])
    if kind == "layer":
        c["heads"] += c["heads"] % 2              # the publishing projection takes an even number of heads
        c["publish"] = rng.random() < 0.5
    return c


def _tokens(c):
    return FRAMES * c["grid_h"] * c["grid_w"]


def _bf16(case):
    return case["kind"] != "step_f32"


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    kind = case["kind"]

    def normal(*shape, scale=1.0):
        return torch.randn(shape, generator=gen, device=DEVICE) * scale

    if kind == "linear":
        m, n, k = case["rows"], case["n_out"], case["k_in"]
        return {"case": case, "x": normal(m, k).to(torch.bfloat16), "w": normal(n, k, scale=k ** -0.5).to(torch.bfloat16),
                "y": torch.empty((m, n), dtype=torch.bfloat16, device=DEVICE)}
    L, H, D, C, nc = _tokens(case), case["heads"], case["head_dim"], case["inflight"], case["cached"]
    dtype = torch.bfloat16 if _bf16(case) else torch.float32
    pool = CascadePool(heads=H, head_dim=D, frames_per_block=FRAMES, grid_h=case["grid_h"], grid_w=case["grid_w"],
                       rope_dims=ROPE_DIMS[D], rope_theta=10000.0, sink_blocks=case["sink"], window_blocks=WINDOW,
                       max_inflight=MAX_INFLIGHT, page_tokens=case.get("page_tokens", 128),
                       dtype="bf16" if _bf16(case) else "f32", device=DEVICE)

    def qkv(n):
        return normal(n, H, D, scale=0.5 if _bf16(case) else 1.0).to(dtype)

    for g in range(nc):                           # the clean cache
        pool.append(g, 0, 0, qkv(L), qkv(L))
        pool.ctx.kv_cache_promote(g)
    ids = list(range(nc, nc + C))
    # the pages of the blocks in flight: consecutive slots of the pool
    per_block = -(-L // pool.cfg.page_tokens) * H * 2 * pool.cfg.page_tokens * D
    pages = pool.pool[nc * per_block * dtype.itemsize:(nc + C) * per_block * dtype.itemsize].view(dtype)
    s = {"case": case, "pool": pool, "ids": ids, "timesteps": TIMESTEPS[:C], "mode": MODES[case["mode"]], "pages": pages}
    if kind == "layer":
        width = H * D
        s["x"] = normal(C * L, width).to(torch.bfloat16)
        s["w_qkv"] = normal(3 * width, width, scale=width ** -0.5).to(torch.bfloat16)
        s["w_out"] = normal(width, width, scale=width ** -0.5).to(torch.bfloat16)
        return s
    s["k"], s["v"] = [qkv(L) for _ in range(C)], [qkv(L) for _ in range(C)]
    s["q"] = qkv(L if kind == "share" else C * L)
    s["first_frame"] = FRAMES * (nc + case.get("share", 0))
    s["q_rot"], s["o"] = torch.empty_like(s["q"]), torch.empty_like(s["q"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "linear":
        return linear(s["x"], s["w"], out=s["y"])
    pool, ids = s["pool"], s["ids"]
    if kind == "layer":
        y = attention_layer(pool, s["x"], s["w_qkv"], s["w_out"], ids, s["timesteps"], 0, s["mode"],
                            publish_in_projection=case["publish"])
        return {"y": y, "pages": s["pages"]}
    pool.append_batch(ids, s["timesteps"], 0, s["k"], s["v"])
    if kind == "step":
        return {"o": pool.forward_rope(s["q"], ids, s["mode"], out=s["o"]), "pages": s["pages"]}
    pool.rope(s["q"], s["first_frame"], out=s["q_rot"])
    if kind == "publish":
        return {"q": s["q_rot"], "pages": s["pages"]}
    share = (case["share"], 1) if kind == "share" else None
    return {"o": pool.forward(s["q_rot"], ids, s["mode"], out=s["o"], share=share), "pages": s["pages"]}


def work(case):
    kind = case["kind"]
    if kind == "linear":
        m, n, k = case["rows"], case["n_out"], case["k_in"]
        return {"bytes": 2 * (m * k + n * k + m * n), "flops": 2 * m * n * k}
    L, H, D, C, nc = _tokens(case), case["heads"], case["head_dim"], case["inflight"], case["cached"]
    one = L * H * D * (2 if _bf16(case) else 4)   # K, V, Q or O of one block
    first, count = (case["share"], 1) if kind == "share" else (0, C)
    if kind == "publish":
        return {"bytes": (4 * C + 2 * C) * one, "flops": 3 * 2 * C * L * H * D}
    visible = sum(nc + (C if case["mode"] == "bidirectional" else i + 1) for i in range(first, first + count))
    flops = 4 * D * H * L * L * visible
    if kind == "layer":
        width = H * D
        return {"bytes": 2 * C * one + 2 * nc * one + 2 * C * one + 2 * 4 * width * width,
                "flops": flops + 2 * C * L * 4 * width * width}
    # K and V of the blocks in flight read and their pages written, the cache's pages read, Q read, O written
    return {"bytes": 4 * C * one + 2 * nc * one + 2 * count * one, "flops": flops}


# Relative error against the same path in fp64 (2-norm), measured over the listed and some drawn cases, times four.
_MEASURED = {"step": 2.5e-3, "share": 2.5e-3, "layer": 4.6e-3, "publish": 1.6e-3, "linear": 1.7e-3, "step_f32": 1.2e-6}


def tolerance(case):
    return {"rel": 4 * _MEASURED[case["kind"]]}
