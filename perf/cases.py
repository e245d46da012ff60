"""The work that a user of this library has it do, as cases that can be timed and compared.

A denoising step of Latent Parallelism on one device is: cut the latent (lp_partition), run
the DiT blocks of every sub-latent (projection, attention, output projection), blend the
predictions and update the latent (lp_reconstruct or the guided step).  The cases are those
calls as a serving program makes them, from the smallest sub-latent of the tests to the
largest one of the configurations, always through the C-ABI binding.

Inputs are made on the device from the seed alone: latents and predictions N(0, 1) in
binary32; activations N(0, 1) in bf16; weights N(0, 1 / d_in) in bf16, so that a projection
of such activations is again O(1); bias 0.5 N(0, 1); gains 1 + 0.2 N(0, 1).
"""
import math

import torch

from paper_2512_07350_amd import binding as lp

EPS = 1e-6
GUIDANCE, COEF_Z, COEF_PRED = 5.0, 1.0, -0.02    # an Euler step of a flow-matching sampler
PATCH = (1, 2, 2)


def listed():
    return [
        # Attention of one sub-latent of the tiny configuration (5 x 8 x 5 patches): nothing but latency.
        dict(name="attention-tiny", kind="attention", n=200, heads=4, head_dim=64, batch=1, layout="token", scratch="workspace"),
        # A caller that keeps head-major tensors and cannot hand over scratch memory, head_dim 64, a length
        # that no tile divides.
        dict(name="attention-head-major-static", kind="attention", n=2999, heads=16, head_dim=64, batch=1, layout="head",
             scratch="static"),
        # The conditional and the unconditional pass of a guided step in one launch, the two items of a token
        # side by side: 49 frames at 480p cut in four along the width with overlap ratio 0.5 (13 x 30 x 19 patches).
        dict(name="attention-pair-480p", kind="attention", n=7410, heads=12, head_dim=128, batch=2, layout="side",
             scratch="workspace"),
        # The largest sub-latent of 81 frames at 720p cut in eight along the width (21 x 45 x 14 patches), 40 heads.
        dict(name="attention-720p", kind="attention", n=13230, heads=40, head_dim=128, batch=1, layout="token",
             scratch="workspace"),
        # One whole step of 33 frames at 480p along the height: cut, attend in every sub-latent, blend.
        dict(name="step-480p-33f", kind="step", channels=16, frames=9, height=60, width=104, parts=4, overlap=1, dim=1, heads=12,
             head_dim=128),
        # The block's attention path (projection with normalisation and rotation, attention, output projection)
        # on the tiny configuration's sub-latent.
        dict(name="block-tiny", kind="block", grid_t=5, grid_h=8, grid_w=5, heads=4, head_dim=64, bias=True),
        # The same on a sub-latent of 33 frames at 480p cut along the width, d_model 1536.
        dict(name="block-480p-33f", kind="block", grid_t=9, grid_h=30, grid_w=14, heads=12, head_dim=128, bias=True),
        # The same on the largest sub-latent of the 720p configuration, d_model 5120.
        dict(name="block-720p", kind="block", grid_t=21, grid_h=45, grid_w=14, heads=40, head_dim=128, bias=True),
        # A caller whose q, k and v are projected one by one: three plain products, normalisation and rotation in
        # place on q and k, attention, output projection; no bias.
        dict(name="own-projection", kind="own", grid_t=7, grid_h=17, grid_w=23, heads=16, head_dim=64, bias=False),
        # A linear layer with few tokens and a long reduction.
        dict(name="linear-ragged", kind="linear", n=520, d_in=5120, d_out=640, bias=True),
        # The latent side of three guided steps T -> H -> W of the 81-frame 480p loop, the latent carried in place.
        dict(name="guided-loop-480p", kind="guided", channels=16, frames=21, height=60, width=104, parts=4, overlap=2),
        # The latent side of one plain step at 720p along the width: cut in eight, blend.
        dict(name="latent-720p", kind="latent", channels=16, frames=21, height=90, width=160, parts=8, overlap=2, dim=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _latent_sizes(rng, widest):
    while True:
        c = dict(channels=rng.choice((4, 8, 16, 16, 16)), frames=_log_int(rng, 4, 41), height=2 * _log_int(rng, 8, 45),
                 width=2 * _log_int(rng, 8, 80), parts=rng.choice((2, 3, 4, 4, 8)), overlap=rng.choice((0, 1, 1, 2, 2)))
        # every dimension has to hold the cores: N >= K patches, and an overlap of O <= L (K - 1)
        if c["frames"] >= c["parts"] and c["channels"] * c["frames"] * c["height"] * c["width"] <= widest:
            return c


def draw(rng):
    """One more case of the same ranges; none costs more than the largest listed one."""
    kind = rng.choice(("attention", "attention", "attention", "step", "block", "block", "own", "linear", "guided", "latent"))
    most = work(dict(kind="block", grid_t=21, grid_h=45, grid_w=14, heads=40, head_dim=128, bias=True))["flops"]
    while True:
        if kind == "attention":
            c = dict(kind=kind, n=_log_int(rng, 96, 24000), heads=rng.choice((1, 3, 4, 8, 12, 12, 16, 24, 40)),
                     head_dim=rng.choice((64, 128, 128)), batch=rng.choice((1, 1, 2)), layout="token", scratch="workspace")
            if c["batch"] == 2:
                c["layout"] = rng.choice(("token", "side"))
            else:
                c["layout"] = rng.choice(("token", "token", "head"))
                c["scratch"] = rng.choice(("workspace", "workspace", "static", "none"))
        elif kind == "step":
            c = dict(kind=kind, **_latent_sizes(rng, 16 * 21 * 90 * 160), dim=rng.randrange(3), heads=rng.choice((4, 8, 12, 12)),
                     head_dim=rng.choice((64, 128, 128)))
        elif kind in ("block", "own"):
            c = dict(kind=kind, grid_t=_log_int(rng, 2, 41), grid_h=_log_int(rng, 4, 45), grid_w=_log_int(rng, 3, 52),
                     heads=rng.choice((4, 8, 12, 12, 16, 24, 40)), head_dim=rng.choice((64, 128, 128)), bias=rng.random() < 0.6)
        elif kind == "linear":
            c = dict(kind=kind, n=_log_int(rng, 33, 16000), d_in=64 * _log_int(rng, 4, 80), d_out=128 * _log_int(rng, 2, 40),
                     bias=rng.random() < 0.6)
        elif kind == "guided":
            c = dict(kind=kind, **_latent_sizes(rng, 16 * 21 * 90 * 160))
        else:
            c = dict(kind=kind, **_latent_sizes(rng, 16 * 41 * 90 * 160), dim=rng.randrange(3))
        if work(c)["flops"] <= most:
            return c


# ---- what each kind is made of

def _tokens(c):
    return c["grid_t"] * c["grid_h"] * c["grid_w"]


def _latent(c):
    return (c["channels"], c["frames"], c["height"], c["width"])


def _plan(c, dim):
    return lp.lp_plan_create(_latent(c), PATCH, c["parts"], dim, overlap_patches=c["overlap"])


class _Draws:
    """Tensors on the device from one seeded generator."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(seed)

    def f32(self, *shape):
        return torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.float32)

    def bf16(self, *shape):
        return torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.bfloat16)

    def weight(self, d_out, d_in):
        return (self.f32(d_out, d_in) * d_in ** -0.5).to(torch.bfloat16)


def _scratch(head_dim):
    size = lp.lp_attention_workspace_size(head_dim)
    return torch.empty(size, dtype=torch.uint8, device="cuda"), size


def prepare(case, seed):
    d = _Draws(seed)
    s = dict(case, stream=torch.cuda.current_stream().cuda_stream)
    kind = case["kind"]
    if kind == "attention":
        b, n, h, hd = case["batch"], case["n"], case["heads"], case["head_dim"]
        shape = {"token": (b, n, h, hd), "head": (h, n, hd), "side": (n, b, h, hd)}[case["layout"]]
        s["strides"] = {"token": (n * h * hd, h * hd, hd), "head": (0, hd, n * hd), "side": (h * hd, b * h * hd, hd)}[case["layout"]]
        s["q"], s["k"], s["v"] = d.bf16(*shape), d.bf16(*shape), d.bf16(*shape)
        s["o"] = torch.empty_like(s["q"])
        s["ws"] = _scratch(hd) if case["scratch"] == "workspace" else (None, 0)
    elif kind == "step":
        h, hd = case["heads"], case["head_dim"]
        s["plan"] = _plan(case, case["dim"])
        s["z"], s["preds"] = d.f32(*_latent(case)), d.f32(s["plan"].total_elems)
        s["subs"], s["out"] = torch.empty_like(s["preds"]), torch.empty_like(s["z"])
        s["tokens"] = [p.n_tokens for p in s["plan"].parts() if p.n_tokens]
        s["qkv"] = [(d.bf16(n, h, hd), d.bf16(n, h, hd), d.bf16(n, h, hd)) for n in s["tokens"]]
        s["o"] = [torch.empty_like(t[0]) for t in s["qkv"]]
        s["ws"] = _scratch(hd)
    elif kind in ("block", "own"):
        n, h, hd = _tokens(case), case["heads"], case["head_dim"]
        dm = h * hd
        s["n"], s["dm"] = n, dm
        s["x"], s["w_qkv"], s["w_o"] = d.bf16(n, dm), d.weight(3 * dm, dm), d.weight(dm, dm)
        s["b_qkv"] = 0.5 * d.f32(3 * dm) if case["bias"] else None
        if kind == "own":
            s["w_qkv"] = s["w_qkv"].split(dm)
            s["b_qkv"] = s["b_qkv"].split(dm) if case["bias"] else (None,) * 3
        s["b_o"] = 0.5 * d.f32(dm) if case["bias"] else None
        s["gain_q"], s["gain_k"] = 1.0 + 0.2 * d.f32(h, hd), 1.0 + 0.2 * d.f32(h, hd)
        s["rope"] = lp.make_rope((case["grid_t"], case["grid_h"], case["grid_w"]), head_dim=hd)
        empty = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda")  # noqa: E731
        s["q"], s["k"], s["v"], s["o"], s["y"] = (empty(n, h, hd) for _ in range(5))
        s["ws"] = _scratch(hd)
    elif kind == "linear":
        s["x"], s["w"] = d.bf16(case["n"], case["d_in"]), d.weight(case["d_out"], case["d_in"])
        s["b"] = 0.5 * d.f32(case["d_out"]) if case["bias"] else None
        s["y"] = torch.empty((case["n"], case["d_out"]), dtype=torch.bfloat16, device="cuda")
    elif kind == "guided":
        s["plans"] = [_plan(case, dim) for dim in range(3)]
        s["z"] = d.f32(*_latent(case))
        s["cond"] = [d.f32(p.total_elems) for p in s["plans"]]
        s["uncond"] = [d.f32(p.total_elems) for p in s["plans"]]
        s["subs"] = [torch.empty_like(t) for t in s["cond"]]
    elif kind == "latent":
        s["plan"] = _plan(case, case["dim"])
        s["z"], s["preds"] = d.f32(*_latent(case)), d.f32(s["plan"].total_elems)
        s["subs"], s["out"] = torch.empty_like(s["preds"]), torch.empty_like(s["z"])
    else:
        raise ValueError(kind)
    return s


def run(s):
    kind, st = s["kind"], s["stream"]
    if kind == "attention":
        n, h, hd, b = s["n"], s["heads"], s["head_dim"], s["batch"]
        stride_batch, stride_tok, stride_head = s["strides"]
        ws, size = s["ws"]
        if b > 1:
            lp.lp_attention_batch(s["q"], s["k"], s["v"], s["o"], b, n, h, hd, stride_batch, stride_tok, stride_head, 0.0, ws, size, st)
        elif s["scratch"] == "static":
            lp.lp_attention_static(s["q"], s["k"], s["v"], s["o"], n, h, hd, stride_tok, stride_head, 0.0, st)
        else:
            lp.lp_attention(s["q"], s["k"], s["v"], s["o"], n, h, hd, stride_tok, stride_head, 0.0, ws, size, st)
        return s["o"]
    if kind == "step":
        h, hd = s["heads"], s["head_dim"]
        ws, size = s["ws"]
        lp.lp_partition(s["plan"], s["z"], s["subs"], st)
        for n, (q, k, v), o in zip(s["tokens"], s["qkv"], s["o"]):
            lp.lp_attention(q, k, v, o, n, h, hd, h * hd, hd, 0.0, ws, size, st)
        lp.lp_reconstruct(s["plan"], s["preds"], s["out"], st)
        return {"subs": s["subs"], "o": s["o"], "out": s["out"]}
    if kind == "block":
        n, h, hd, dm = s["n"], s["heads"], s["head_dim"], s["dm"]
        ws, size = s["ws"]
        lp.lp_qkv_projection(s["x"], s["w_qkv"], s["b_qkv"], s["gain_q"], s["gain_k"], EPS, s["rope"], s["q"], s["k"], s["v"], n, h, hd, st)
        lp.lp_attention(s["q"], s["k"], s["v"], s["o"], n, h, hd, dm, hd, 0.0, ws, size, st)
        lp.lp_linear(s["o"], s["w_o"], s["b_o"], s["y"], n, dm, dm, st)
        return {"q": s["q"], "k": s["k"], "v": s["v"], "o": s["o"], "y": s["y"]}
    if kind == "own":
        n, h, hd, dm = s["n"], s["heads"], s["head_dim"], s["dm"]
        ws, size = s["ws"]
        for w, bias, out in zip(s["w_qkv"], s["b_qkv"], (s["q"], s["k"], s["v"])):
            lp.lp_linear(s["x"], w, bias, out, n, dm, dm, st)
        lp.lp_qk_norm_rope(s["q"], s["gain_q"], EPS, s["rope"], n, h, hd, dm, hd, st)
        lp.lp_qk_norm_rope(s["k"], s["gain_k"], EPS, s["rope"], n, h, hd, dm, hd, st)
        lp.lp_attention(s["q"], s["k"], s["v"], s["o"], n, h, hd, dm, hd, 0.0, ws, size, st)
        lp.lp_linear(s["o"], s["w_o"], s["b_o"], s["y"], n, dm, dm, st)
        return {"q": s["q"], "k": s["k"], "v": s["v"], "o": s["o"], "y": s["y"]}
    if kind == "linear":
        lp.lp_linear(s["x"], s["w"], s["b"], s["y"], s["n"], s["d_in"], s["d_out"], st)
        return s["y"]
    if kind == "guided":
        for dim in range(3):
            nxt = (dim + 1) % 3
            lp.lp_reconstruct_guided_step_partition(s["plans"][dim], s["cond"][dim], s["uncond"][dim], GUIDANCE, s["z"], COEF_Z,
                                                    COEF_PRED, s["z"], s["plans"][nxt], s["subs"][nxt], st)
        return {"z": s["z"], "subs": s["subs"]}
    lp.lp_partition(s["plan"], s["z"], s["subs"], st)
    lp.lp_reconstruct(s["plan"], s["preds"], s["out"], st)
    return {"subs": s["subs"], "out": s["out"]}


def work(case):
    kind = case["kind"]
    if kind == "attention":
        n, width, b = case["n"], case["heads"] * case["head_dim"], case["batch"]
        return {"bytes": 4 * n * width * 2 * b, "flops": 4 * n * n * width * b}
    if kind in ("step", "latent"):
        plan = _plan(case, case["dim"])
        sz, ext = plan.latent_elems * 4, plan.total_elems * 4
        w = {"bytes": 2 * ext + ext + sz, "flops": 2 * (sz + ext) // 4}
        if kind == "step":
            width = case["heads"] * case["head_dim"]
            for p in plan.parts():
                w["bytes"] += 4 * p.n_tokens * width * 2
                w["flops"] += 4 * p.n_tokens ** 2 * width
        return w
    if kind in ("block", "own"):
        n, dm = _tokens(case), case["heads"] * case["head_dim"]
        # the weights, x and y once, q, k, v and o once out and once in; own: q and k once more each way
        rows = 2 + 8 if kind == "block" else 2 + 8 + 4
        return {"bytes": 2 * (4 * dm * dm + rows * n * dm), "flops": 8 * n * dm * dm + 4 * n * n * dm}
    if kind == "linear":
        n, di, do = case["n"], case["d_in"], case["d_out"]
        return {"bytes": 2 * (n * di + di * do + n * do), "flops": 2 * n * di * do}
    total = 0
    plans = [_plan(case, dim) for dim in range(3)]
    for dim in range(3):
        total += (2 * plans[dim].total_elems + 2 * plans[dim].latent_elems + plans[(dim + 1) % 3].total_elems) * 4
    return {"bytes": total, "flops": sum(6 * p.total_elems + 4 * p.latent_elems for p in plans)}


def tolerance(case):
    """Latent operations are bit for bit.  Against binary64 a product of bf16 inputs with one rounding to bf16 on store is
    off by 1.7e-3 (the rounding alone), attention by 2.9e-3 to 3.3e-3 (pre-scaled q, probabilities and result are each
    rounded), a chain of them by 2.1e-3 to 4.8e-3: about four times the product's and attention's figures, for every kind."""
    kind = case["kind"]
    if kind in ("guided", "latent"):
        return "exact"
    if kind == "linear":
        return {"rel": 7e-3}
    return {"rel": 1.2e-2}
