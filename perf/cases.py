"""The work that a user of canon has it do, as timed cases: canonical GEMMs, norm rows, the loss head, decoder blocks,
the int8 quantised projection, the optimizer update and whole replayed steps, each through canon's entry points.

Sizes are those of the workloads that bench.py and the tests name (the 1B-shaped decoder: d 2048, 16 x 128 heads, FFN
8192, vocab 50304, sequence 2048; the paper's own architecture: FFN 5632, 16/4 heads, sequence 4096, window 512; the
small decoders of the tests), and ragged ones between.  Every result is defined bit for bit by the canonical order, so
outputs are compared exactly.
"""
from __future__ import annotations

import math

import torch

import paper_2609_17380_amd.canon as C
import paper_2609_17380_amd.inputs as I

EPS = 1e-5


def listed():
    return [
        # the smallest GEMM workload (128 x 128 x 256): launch and chain latency
        {"name": "gemm_small", "kind": "gemm", "m": 128, "n": 128, "k": 256, "layout": "fwd"},
        # the fused q/k/v projection over one microbatch of 8192 tokens
        {"name": "gemm_qkv", "kind": "gemm", "m": 8192, "n": 6144, "k": 2048, "layout": "fwd"},
        # a weight gradient with no aligned dimension (a trimmed batch, an odd head)
        {"name": "gemm_wgrad_ragged", "kind": "gemm", "m": 2047, "n": 1001, "k": 3001, "layout": "wgrad"},
        # RMSNorm forward and backward over a microbatch
        {"name": "norm", "kind": "norm", "rows": 8192, "cols": 2048},
        # softmax cross-entropy and its gradient over the 1B vocabulary
        {"name": "loss_head", "kind": "loss", "rows": 8192, "vocab": 50304, "z_loss": 0.0},
        # one decoder block, forward and backward: a test-sized one, the 1B block, the paper's block in int8
        {"name": "block_small", "kind": "block", "batch": 2, "seq": 192, "heads": 4, "kv_heads": 4, "head_dim": 64,
         "ffn": 704, "variant": "plain", "dy_std": 1.0},
        {"name": "block_1b", "kind": "block", "batch": 1, "seq": 2048, "heads": 16, "kv_heads": 16, "head_dim": 128,
         "ffn": 8192, "variant": "plain", "dy_std": 1.0},
        {"name": "block_paper_int8", "kind": "block", "batch": 1, "seq": 4096, "heads": 16, "kv_heads": 4,
         "head_dim": 128, "ffn": 5632, "variant": "int8", "dy_std": 1.0 / 4096},
        # the int8 gate/up projection of the paper's decoder: quantise, multiply, rotated backward, step gradient
        {"name": "qlinear", "kind": "qlinear", "tokens": 8192, "out": 11264, "in": 2048},
        # 8 microbatch gradients through the plan, global-norm clip and AdamW for a 110M-parameter decoder
        {"name": "update", "kind": "update", "layers": 8, "d": 768, "ffn": 2048, "vocab": 32000, "ranks": 8},
        # whole replayed steps from a saved state, with clip and audit hash: a test-sized decoder, and two
        # full-width layers of the 1B decoder
        {"name": "step_small", "kind": "step", "layers": 2, "heads": 4, "kv_heads": 4, "head_dim": 64, "ffn": 768,
         "vocab": 2000, "seq": 128, "micro_seqs": 2, "shards": 2, "variant": "plain"},
        {"name": "step_wide", "kind": "step", "layers": 2, "heads": 16, "kv_heads": 16, "head_dim": 128, "ffn": 8192,
         "vocab": 50304, "seq": 2048, "micro_seqs": 1, "shards": 2, "variant": "plain"},
    ]


# ---- drawn cases: the same kinds over their whole ranges ------------------------------------------------------

def _log(rng, lo, hi, grain=None):
    """An integer of [lo, hi], even over its logarithm; a multiple of 128, of 8, or any, as often each."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    g = rng.choice((128, 8, 1)) if grain is None else grain
    return max(g, min(hi // g * g, (v + g // 2) // g * g))


def draw(rng):
    kind = rng.choice(("gemm", "gemm", "gemm", "norm", "loss", "block", "block", "block", "qlinear", "update", "step",
                       "step"))
    while True:
        case = globals()["_draw_" + kind](rng)
        if case is not None:
            return case


def _draw_gemm(rng):
    m, n, k = _log(rng, 64, 8192), _log(rng, 64, 16384), _log(rng, 32, 8192)
    if m * n * k > 8192 * 6144 * 2048:
        return None
    return {"kind": "gemm", "m": m, "n": n, "k": k, "layout": rng.choice(("fwd", "dgrad", "wgrad"))}


def _draw_norm(rng):
    return {"kind": "norm", "rows": _log(rng, 64, 16384), "cols": _log(rng, 256, 4096)}


def _draw_loss(rng):
    rows, vocab = _log(rng, 128, 8192), _log(rng, 1000, 128256)
    if rows * vocab > 8192 * 50304:
        return None
    return {"kind": "loss", "rows": rows, "vocab": vocab, "z_loss": rng.choice((0.0, 1e-4))}


def _draw_heads(rng, small):
    head_dim = rng.choice((32, 64, 128))
    heads = rng.choice((2, 4, 8) if small else (4, 8, 16))
    return heads, head_dim


def _draw_block(rng):
    variant = rng.choice(("plain", "paper", "int8"))
    heads, head_dim = _draw_heads(rng, False)
    kv = heads if variant == "plain" else heads // rng.choice((1, 2, 4))
    batch, seq = rng.choice((1, 2, 4)), _log(rng, 64, 4096)
    d = heads * head_dim
    ffn = _log(rng, d, 4 * d)
    if variant == "int8":  # whole rotation blocks of 256 along tokens and widths
        seq, ffn = max(256, seq // 256 * 256), max(256, ffn // 256 * 256)
        if d % 256 or (d + 2 * kv * head_dim) % 256:
            return None
    case = {"kind": "block", "batch": batch, "seq": seq, "heads": heads, "kv_heads": kv, "head_dim": head_dim,
            "ffn": ffn, "variant": variant, "dy_std": rng.choice((1.0, 1.0 / (batch * seq)))}
    return case if batch * seq <= 8192 and _block_flops(case) <= 1.5e12 else None


def _draw_qlinear(rng):
    t, n, k = _log(rng, 256, 8192, 256), _log(rng, 256, 16384, 256), _log(rng, 128, 8192)
    if t * n * k > 8192 * 11264 * 2048:
        return None
    return {"kind": "qlinear", "tokens": t, "out": n, "in": k}


def _draw_update(rng):
    case = {"kind": "update", "layers": rng.randint(1, 16), "d": _log(rng, 64, 1024), "ffn": _log(rng, 128, 4096),
            "vocab": _log(rng, 500, 50304), "ranks": rng.randint(1, 8)}
    return case if _count(_model_shapes(case)) * case["ranks"] <= 9e8 else None


def _draw_step(rng):
    variant = rng.choice(("plain", "paper", "int8"))
    heads, head_dim = _draw_heads(rng, True)
    kv = heads if variant == "plain" else heads // rng.choice((1, 2))
    d = heads * head_dim
    case = {"kind": "step", "layers": rng.randint(1, 4), "heads": heads, "kv_heads": kv, "head_dim": head_dim,
            "ffn": _log(rng, d, 4 * d), "vocab": _log(rng, 500, 32000), "seq": _log(rng, 64, 1024),
            "micro_seqs": rng.choice((1, 2)), "shards": rng.choice((1, 2, 4)), "variant": variant}
    if variant == "int8":
        case["seq"], case["ffn"] = max(256, case["seq"] // 256 * 256), max(256, case["ffn"] // 256 * 256)
        if d % 256 or (d + 2 * kv * head_dim) % 256:
            return None
    return case if _step_flops(case) <= 2e12 else None


# ---- what a case cannot do without ----------------------------------------------------------------------------

def _pairs(seq, window):
    """Visible (query, key) pairs of a head."""
    if not window or window >= seq:
        return seq * (seq + 1) // 2
    return window * (window + 1) // 2 + (seq - window) * window


def _window(case):
    return 0 if case["variant"] == "plain" else 512


def _block_flops(case):
    t, d = case["batch"] * case["seq"], case["heads"] * case["head_dim"]
    n = d + 2 * case["kv_heads"] * case["head_dim"]
    pairs = case["batch"] * case["heads"] * _pairs(case["seq"], _window(case))
    return 6 * t * (d * n + d * d + 3 * d * case["ffn"]) + pairs * 12 * case["head_dim"]


def _model_shapes(case):
    kind = case["kind"]
    d = case["d"] if kind == "update" else case["heads"] * case["head_dim"]
    kv = d if kind == "update" else case["kv_heads"] * case["head_dim"]
    variant = case.get("variant", "plain")
    return I.model_param_shapes(case["layers"], d, case["ffn"], case["vocab"], kv_dim=kv,
                                embed_norm=variant != "plain", int8_linear=variant == "int8")


def _count(shapes):
    return sum(math.prod(s[1]) for s in shapes)


def _step_flops(case):
    t, ranks = case["micro_seqs"] * case["seq"], case["shards"]
    d = case["heads"] * case["head_dim"]
    layer = _block_flops(dict(case, batch=case["micro_seqs"]))
    return ranks * (case["layers"] * layer + 6 * t * d * case["vocab"])


def work(case):
    kind = case["kind"]
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 2 * (m * k + k * n) + 4 * m * n, "flops": 2 * m * n * k}
    if kind == "norm":  # forward: x in, y out; backward: x and dy in, dx out
        r, c = case["rows"], case["cols"]
        return {"bytes": r * c * (4 + 2 + 8 + 4) + 2 * c + 4 * c + 8 * r, "flops": 14 * r * c}
    if kind == "loss":
        r, v = case["rows"], case["vocab"]
        return {"bytes": 4 * r * v + 8 * r, "flops": 40 * r * v}
    if kind == "block":
        t, d = case["batch"] * case["seq"], case["heads"] * case["head_dim"]
        n = d + 2 * case["kv_heads"] * case["head_dim"]
        weights = d * n + d * d + 3 * d * case["ffn"] + 2 * d
        return {"bytes": 16 * t * d + 6 * weights, "flops": _block_flops(case)}
    if kind == "qlinear":
        t, n, k = case["tokens"], case["out"], case["in"]
        return {"bytes": n * k * (2 + 1 + 4) + t * k * (2 + 1 + 4) + t * n * 8, "flops": 6 * t * n * k}
    if kind == "update":  # each microbatch gradient in; gradient out; parameter and moments in and out
        p = _count(_model_shapes(case))
        return {"bytes": p * (4 * case["ranks"] + 4 + 4 + 16), "flops": p * (2 * case["ranks"] + 20)}
    p = _count(_model_shapes(case))  # step: state in and out, its hash's input, the gradient
    return {"bytes": p * (2 + 2 + 8 + 8 + 4), "flops": _step_flops(case)}


def tolerance(case):
    # the canonical order fixes every rounding: another correct implementation gives the same bits
    return "exact"


# ---- inputs, plans and workspaces a user's program holds --------------------------------------------------------

class _Gen:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed) & (2 ** 62 - 1))

    def f32(self, *shape, std=1.0):
        return torch.randn(shape, generator=self.g, device="cuda").mul_(std)

    def bf16(self, *shape, std=1.0):
        return self.f32(*shape, std=std).to(torch.bfloat16)

    def ints(self, high, *shape):
        return torch.randint(0, high, shape, generator=self.g, device="cuda", dtype=torch.int32)


def _bytes(n):
    return torch.empty(max(1, int(n)), dtype=torch.uint8, device="cuda")


def _empty(*shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device="cuda")


def _cfg(case, layers, vocab, micro_seqs):
    paper, int8 = case["variant"] != "plain", case["variant"] == "int8"
    return C.ModelCfg(layers, case["heads"] * case["head_dim"], case["heads"], case["head_dim"], case["ffn"], vocab,
                      case["seq"], micro_seqs, EPS, case["kv_heads"], int(paper), int(paper), _window(case),
                      5 if paper else 0, 1e-4 if paper else 0.0, int(int8), 40 if int8 else 0, int(int8))


def _rope(case):
    return [torch.from_numpy(t).cuda() for t in I.rope_tables(case["seq"], case["head_dim"])]


def _param(gen, shape, init):
    """A bf16 parameter as a fresh model holds it: N(0, init), a gain of 1, or an activation step."""
    if isinstance(init, tuple):
        return torch.full(shape, init[1], dtype=torch.bfloat16, device="cuda")
    if init is None:
        return torch.ones(shape, dtype=torch.bfloat16, device="cuda")
    return gen.bf16(*shape, std=init)


def _flat(shapes, dtype):
    """One zeroed buffer for a model's tensors (each at a 256-byte boundary) and the tensors as views of it."""
    at, spans = 0, []
    for s in shapes:
        spans.append((at, math.prod(s[1])))
        at += -(-spans[-1][1] // 128) * 128
    flat = torch.zeros(at, dtype=dtype, device="cuda")
    return flat, [flat[o:o + n].view(s[1]) for (o, n), s in zip(spans, shapes)]


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, _Gen(seed))


def run(state):
    return globals()["_run_" + state["kind"]](state)


def _prepare_gemm(case, gen):
    m, n, k = case["m"], case["n"], case["k"]
    ta, tb = {"fwd": (0, 1), "dgrad": (0, 0), "wgrad": (1, 0)}[case["layout"]]
    a = gen.bf16(*((k, m) if ta else (m, k)))  # activations, or an upstream gradient
    b = gen.bf16(*((n, k) if tb else (k, n)), std=1.0 if ta else 0.02)  # weights (activations for a weight gradient)
    return {"kind": "gemm", "mnk": (m, n, k), "ta": ta, "tb": tb, "a": a, "b": b, "c": _empty(m, n)}


def _run_gemm(s):
    m, n, k = s["mnk"]
    C.gemm(m, n, k, s["a"], m if s["ta"] else k, s["b"], k if s["tb"] else n, s["c"], n, trans_a=s["ta"],
           trans_b=s["tb"])
    return s["c"]


def _prepare_norm(case, gen):
    r, c = case["rows"], case["cols"]
    return {"kind": "norm", "rc": (r, c), "x": gen.f32(r, c), "gain": gen.f32(c, std=0.1).add_(1).to(torch.bfloat16),
            "dy": gen.f32(r, c, std=1.0 / r), "y": _empty(r, c, dtype=torch.bfloat16), "rstd": _empty(r),
            "dx": _empty(r, c), "dgain": _empty(c)}


def _run_norm(s):
    r, c = s["rc"]
    C.rownorm(C.FWD, r, c, s["x"], s["gain"], EPS, y=s["y"], rstd=s["rstd"])
    C.rownorm(C.BWD, r, c, s["x"], s["gain"], EPS, rstd=s["rstd"], dy=s["dy"], dx=s["dx"], dgain=s["dgain"])
    return s["y"], s["rstd"], s["dx"], s["dgain"]


def _prepare_loss(case, gen):
    r, v = case["rows"], case["vocab"]
    return {"kind": "loss", "rv": (r, v), "z": case["z_loss"], "logits": gen.bf16(r, v, std=2.0),
            "targets": gen.ints(v, r), "dlogits": _empty(r, v, dtype=torch.bfloat16), "rows": _empty(r),
            "mean": _empty(1)}


def _run_loss(s):
    r, v = s["rv"]
    C.softmax_xent(C.XENT, r, v, s["logits"], s["dlogits"], targets=s["targets"], inv_tokens=1.0 / r,
                   row_loss=s["rows"], mean_loss=s["mean"], z_loss=s["z"])
    return s["dlogits"], s["rows"], s["mean"]


def _prepare_block(case, gen):
    b, t, d = case["batch"], case["batch"] * case["seq"], case["heads"] * case["head_dim"]
    cfg = _cfg(case, 1, 32, b)
    model = dict(case, kind="step", layers=1, vocab=32)
    shapes = [s for s in _model_shapes(model) if s[0].startswith("l0.")]
    w = [_param(gen, s[1], s[2]) for s in shapes]
    cos, sin = _rope(case)
    return {"kind": "block", "cfg": cfg, "batch": b, "x": gen.f32(t, d), "dy": gen.f32(t, d, std=case["dy_std"]),
            "w": w, "cos": cos, "sin": sin, "y": _empty(t, d), "dx": _empty(t, d),
            "dw": [_empty(*s[1]) for s in shapes], "ws": _bytes(C.block_workspace_bytes(cfg, b))}


def _run_block(s):
    C.block_fwd_bwd(s["cfg"], s["batch"], s["x"], s["dy"], s["w"], s["cos"], s["sin"], s["y"], s["dx"], s["dw"],
                    s["ws"])
    return s["y"], s["dx"], s["dw"]


def _prepare_qlinear(case, gen):
    t, n, k = case["tokens"], case["out"], case["in"]
    return {"kind": "qlinear", "tnk": (t, n, k), "w": gen.bf16(n, k, std=0.02), "x": gen.bf16(t, k),
            "sx": torch.full((1,), I.ACT_STEPS["sx_gate_up"], device="cuda"), "dy": gen.f32(t, n, std=1.0 / t),
            "sw": _empty(n), "qw": _empty(n, k, dtype=torch.int8), "qx": _empty(t, k, dtype=torch.int8),
            "y": _empty(t, n), "dx": _empty(t, k), "dw": _empty(n, k), "ds": _empty(1),
            "ws": _bytes(C.qlinear_bwd_workspace_bytes(t, n, k)), "ls": _bytes(C.lsq_step_grad_workspace_bytes(t, k))}


def _run_qlinear(s):
    t, n, k = s["tnk"]
    C.quant_scales(n, k, s["w"], s["sw"])
    C.quantize(n, k, s["w"], s["sw"], 1, s["qw"])
    C.quantize(t, k, s["x"], s["sx"], 0, s["qx"])
    C.gemm_i8(t, n, k, s["qx"], k, s["qw"], k, y=s["y"], sa=s["sx"], sb=s["sw"])
    C.qlinear_bwd(t, n, k, s["dy"], s["qx"], s["sx"], s["qw"], s["sw"], s["dx"], s["dw"], s["ws"])
    C.lsq_step_grad(t, k, s["x"], s["sx"], s["dx"], s["ds"], s["ls"])
    return s["qw"], s["qx"], s["y"], s["dx"], s["dw"], s["ds"]


def _prepare_update(case, gen):
    shapes, ranks = _model_shapes(case), case["ranks"]
    pf, p = _flat(shapes, torch.bfloat16)
    mf, m = _flat(shapes, torch.float32)
    vf, v = _flat(shapes, torch.float32)
    gf, g = _flat(shapes, torch.float32)
    for t, s in zip(p, shapes):
        t.copy_(_param(gen, s[1], s[2]))
    # microbatch gradients whose mean has a norm of about 2: the clip at 1 acts
    std = 2.0 * math.sqrt(ranks / gf.numel())
    norm = _empty(1)
    return {"kind": "update", "plan": C.DPPlan(1, ranks, 1), "p": p, "m": m, "v": v, "g": g, "pf": pf, "mf": mf,
            "vf": vf, "gf": gf, "micro": [gen.f32(gf.numel(), std=std) for _ in range(ranks)], "norm": norm,
            "clip": C.make_clip(1.0, math.inf, 0, norm), "ws": _bytes(C.clip_grad_norm_workspace_bytes(g)),
            "decay": [s[3] for s in shapes], "consts": C.AdamWConsts(*I.adamw_constants())}


def _run_update(s):
    C.grad_accum(s["plan"], s["gf"].numel(), s["micro"], s["gf"])
    C.clip_grad_norm(s["g"], s["clip"], s["ws"])
    C.adamw(s["p"], s["m"], s["v"], s["g"], s["decay"], s["consts"])
    return s["pf"], s["mf"], s["vf"], s["gf"], s["norm"]


def _prepare_step(case, gen):
    cfg, plan = _cfg(case, case["layers"], case["vocab"], case["micro_seqs"]), C.DPPlan(1, case["shards"], 1)
    shapes = _model_shapes(case)
    pf, p = _flat(shapes, torch.bfloat16)
    mf, m = _flat(shapes, torch.float32)
    vf, v = _flat(shapes, torch.float32)
    gf, g = _flat(shapes, torch.float32)
    for t, s in zip(p, shapes):
        t.copy_(_param(gen, s[1], s[2]))
    cos, sin = _rope(case)
    norm = _empty(1)
    return {"kind": "step", "cfg": cfg, "plan": plan, "p": p, "m": m, "v": v, "g": g, "pf": pf, "mf": mf, "vf": vf,
            "gf": gf, "saved": pf.clone(), "cos": cos, "sin": sin, "norm": norm,
            "windows": gen.ints(case["vocab"], case["shards"] * case["micro_seqs"], case["seq"] + 1),
            "consts": C.AdamWConsts(*I.adamw_constants()), "clip": C.make_clip(1.0, math.inf, 0, norm),
            "loss": _empty(1), "digest": torch.zeros(32, dtype=torch.uint8, device="cuda"),
            "ws": _bytes(C.step_workspace_bytes(cfg, plan))}


def _run_step(s):
    # a replay: the saved state back in place, then the step
    s["pf"].copy_(s["saved"])
    s["mf"].zero_()
    s["vf"].zero_()
    C.step(s["cfg"], s["plan"], s["p"], s["m"], s["v"], s["windows"], s["cos"], s["sin"], s["consts"], s["ws"],
           s["loss"], grads_out=s["g"], clip=s["clip"], state_digest=s["digest"])
    return s["loss"], s["norm"], s["pf"], s["mf"], s["vf"], s["gf"], s["digest"]


# ---- the same results in 64 bits, in plain torch ----------------------------------------------------------------

def exact(case, seed):
    fn = globals().get("_exact_" + case["kind"])
    return None if fn is None else fn(case, prepare(case, seed))


def _exact_gemm(case, s):
    a, b = s["a"].double(), s["b"].double()
    return (a.t() if s["ta"] else a) @ (b.t() if s["tb"] else b)


def _norm64(x, gain, eps=float(torch.tensor(EPS, dtype=torch.float32))):
    r = torch.rsqrt(x.square().mean(-1, keepdim=True) + eps)
    return (x * r if gain is None else x * r * gain), r


def _exact_norm(case, s):
    x, g = s["x"].double().requires_grad_(), s["gain"].double().requires_grad_()
    y, r = _norm64(x, g)
    dx, dg = torch.autograd.grad(y, (x, g), s["dy"].double())
    return y.detach(), r.detach().view(-1), dx, dg


def _exact_loss(case, s):
    r, _ = s["rv"]
    dl, row = [], []
    for i in range(0, r, 1024):
        x, t = s["logits"][i:i + 1024].double(), s["targets"][i:i + 1024].long()
        lse = torch.logsumexp(x, 1, keepdim=True)
        row.append((lse - x.gather(1, t[:, None]) + s["z"] * lse.square()).view(-1))
        p = torch.exp(x - lse) * (1 + 2 * s["z"] * lse)
        p.scatter_add_(1, t[:, None], torch.full_like(t[:, None], -1.0, dtype=torch.float64))
        dl.append(p / r)
    row = torch.cat(row)
    return torch.cat(dl), row, row.mean().view(1)


def _rope64(x, cos, sin):
    a, b = x.chunk(2, -1)
    return torch.cat((a * cos - b * sin, b * cos + a * sin), -1)


def _exact_block(case, s):
    if case["variant"] == "int8":
        return None  # rounded codes: their straight-through gradients have no 64-bit value
    b, seq, h, kv, hd = case["batch"], case["seq"], case["heads"], case["kv_heads"], case["head_dim"]
    if b * h * seq * seq > 3e8:
        return None
    d, f = h * hd, case["ffn"]
    x = s["x"].double().requires_grad_()
    w = [t.double().requires_grad_() for t in s["w"]]
    qkv = _norm64(x, w[0])[0] @ w[1].t()
    q, k, v = (t.reshape(b, seq, -1, hd).transpose(1, 2) for t in qkv.split((d, kv * hd, kv * hd), 1))
    if case["variant"] != "plain":
        q, k = _norm64(q, None)[0], _norm64(k, None)[0]
    q, k = _rope64(q, s["cos"].double(), s["sin"].double()), _rope64(k, s["cos"].double(), s["sin"].double())
    k, v = k.repeat_interleave(h // kv, 1), v.repeat_interleave(h // kv, 1)
    i = torch.arange(seq, device="cuda")
    seen = i[None, :] <= i[:, None]
    if _window(case):
        seen &= i[None, :] > i[:, None] - _window(case)
    p = torch.softmax((q @ k.transpose(2, 3) / math.sqrt(hd)).masked_fill(~seen, -math.inf), -1)
    x2 = x + (p @ v).transpose(1, 2).reshape(b * seq, d) @ w[2].t()
    gate, up = (_norm64(x2, w[3])[0] @ w[4].t()).split(f, 1)
    y = x2 + (gate * torch.sigmoid(gate) * up) @ w[5].t()
    grads = torch.autograd.grad(y, [x] + w, s["dy"].double())
    return y.detach(), grads[0], list(grads[1:])


def _rotate(x):
    """Walsh-Hadamard rotation of blocks of 256 along the last dimension, scaled by 1/16."""
    v = x.reshape(*x.shape[:-1], x.shape[-1] // 256, 256)
    step = 1
    while step < 256:
        u = v.reshape(*v.shape[:-1], 256 // (2 * step), 2, step)
        v = torch.stack((u[..., 0, :] + u[..., 1, :], u[..., 0, :] - u[..., 1, :]), -2).reshape(*v.shape)
        step *= 2
    return (v / 16).reshape(x.shape)


def _codes(x, step):
    return torch.clamp(torch.round(x / step), -128, 127)


def _rotated_product(a, b):
    """a [I, M] and b [J, M]: both rotated along M and quantised with their absmax steps, then multiplied."""
    a, b = _rotate(a), _rotate(b)
    sa, sb = a.abs().max() / 127, b.abs().max() / 127
    return (_codes(a, sa) @ _codes(b, sb).t()) * (sa * sb)


def _exact_qlinear(case, s):
    t, n, k = s["tnk"]
    if t * n > 1e8:
        return None
    w, x, dy, sx = s["w"].double(), s["x"].double(), s["dy"].double(), s["sx"].double()
    sw = 2 * w.abs().mean(1, keepdim=True) / math.sqrt(127)
    qw, v = _codes(w, sw), x / sx
    qx = _codes(x, sx)
    y = (qx @ qw.t()) * sx * sw.t()
    dx = _rotated_product(dy, (sw * qw).t().contiguous())
    dw = _rotated_product(dy.t().contiguous(), (sx * qx).t().contiguous())
    delta = torch.where(v < -128, -128.0, torch.where(v > 127, 127.0, torch.round(v) - v))
    return None, None, y, dx, dw, ((dx * delta).sum() / math.sqrt(127 * k)).view(1)


def _exact_update(case, s):
    c = s["consts"]
    lr, b1, c1, b2, c2, ib1, ib2, eps, decay = (getattr(c, n) for n, _ in c._fields_)
    flat = sum(m.double() for m in s["micro"]) / case["ranks"]
    grads = [flat[t.storage_offset():t.storage_offset() + t.numel()] for t in s["g"]]
    norm = torch.sqrt(sum(g.square().sum() for g in grads))
    coef = min(1.0, float(1.0 / (norm + 1e-6)))
    out = [torch.zeros_like(s["gf"], dtype=torch.float64) for _ in range(3)]
    full = flat.clone()  # the padding between the tensors is not clipped
    for t, g, dec in zip(s["p"], grads, s["decay"]):
        at = slice(t.storage_offset(), t.storage_offset() + t.numel())
        g = g * coef
        full[at] = g
        m, v = c1 * g, c2 * g * g
        p = t.double().view(-1) * (decay if dec else 1.0)
        out[0][at], out[1][at], out[2][at] = p - lr * (m * ib1) / (torch.sqrt(v * ib2) + eps), m, v
    return out[0], out[1], out[2], full, norm.view(1)
