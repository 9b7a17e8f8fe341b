"""What a training or serving program has the fused operators do, case by case, for timing and for checks.

A case is a dict of plain values.  `prepare` makes what such a program holds before the call, `run` makes one
pass through the package's public entry points, `work` says what a pass cannot do without, `tolerance` how far two
correct implementations may be apart, and `exact` gives the same outputs in float64 from plain torch.

Common keys:
  op        "infer"    lnmod.forward / forward_varlen: y and the statistics, no gradient (serving, sampling)
            "step"     functional.ln_modulate and its gradients (training)
            "gated"    functional.gated_ln_modulate and its gradients
            "qk"       functional.qk_norm and its gradients
  dtype     "bf16" (training and serving) or "f32" (debugging, small models)
  D         features of a row;  B, S: samples (op qk with a head's width: heads) and tokens of each;  segments, shortest, longest, lengths_seed: a
            packed batch instead (lengths spread over their logarithm), or mix = "video": the packed mixture of
            stills and clips that synth.py defines
  mod       "sample": one modulation row per sample or segment;  "token": one per token (step only)
  stats     False: only x is kept between the passes and the backward forms mean and rstd again (step only)
"""
import math
import random

import torch

from paper_2605_17923_amd import functional, lnmod, synth

EPS = 1e-6
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # The smallest step that is run at all: two short fp32 samples (a unit test, a toy model).  Latency,
        # launches and host work are all there is.
        dict(name="tiny_f32_step", op="step", dtype="f32", D=1536, B=2, S=256, mod="sample", stats=True),
        # Sampling one still picture with the 14B-shaped model: a single short forward.
        dict(name="image_infer", op="infer", dtype="bf16", D=5120, B=1, S=1560, mod="sample"),
        # Three ragged samples at a middle width: the ordinary fine-tuning step, no size a round number.
        dict(name="ragged_step", op="step", dtype="bf16", D=3072, B=3, S=4099, mod="sample", stats=True),
        # One clip through the 1.3B-shaped model.
        dict(name="clip_1536_step", op="step", dtype="bf16", D=1536, B=1, S=32760, mod="sample", stats=True),
        # One long clip through the 14B-shaped model: the headline training step.
        dict(name="clip_5120_step", op="step", dtype="bf16", D=5120, B=1, S=75600, mod="sample", stats=True),
        # The same model with activation checkpoints: no statistics kept.
        dict(name="recompute_step", op="step", dtype="bf16", D=5120, B=2, S=8190, mod="sample", stats=False),
        # A timestep per token (image-to-video, diffusion forcing): modulation rows streamed with x.
        dict(name="per_token_step", op="step", dtype="bf16", D=5120, B=2, S=32760, mod="token", stats=True),
        # The mixed bucket of stills and clips, packed: the largest call.
        dict(name="packed_video_step", op="step", dtype="bf16", D=5120, mix="video", mod="sample", stats=True),
        # Many stills of different sizes packed into one batch of the small model.
        dict(name="packed_images_step", op="step", dtype="bf16", D=1536, segments=96, shortest=64, longest=1560,
             lengths_seed=3, mod="sample", stats=True),
        # The residual update and the norm after it, two clips.
        dict(name="gated_step", op="gated", dtype="bf16", D=5120, B=2, S=16380, mod="sample"),
        # Query and key norm over the whole projection, and per attention head (12 heads of 128).
        dict(name="qk_wide_step", op="qk", dtype="bf16", D=5120, B=1, S=16380),
        dict(name="qk_head_step", op="qk", dtype="bf16", D=128, B=12, S=32760),
    ]


# A drawn case never moves more than this (the largest listed one moves about 6.3e9 bytes).
MOST_BYTES = 6.0e9


def _spread(rng, lo, hi):
    """An integer from [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["infer", "step", "step", "step", "gated", "qk"])
    c = dict(op=op, dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]))
    if op == "qk" and rng.random() < 0.5:
        c.update(D=rng.choice([64, 80, 96, 128]), B=rng.choice([8, 12, 16, 24, 40]), S=_spread(rng, 256, 75600))
    else:
        # widths that models have, or any that is allowed
        c["D"] = rng.choice([1152, 1536, 2048, 2560, 3072, 3584, 4096, 5120, 6144]) if rng.random() < 0.6 else \
            8 * _spread(rng, 64, 768)
        if op != "qk" and rng.random() < 0.35:
            c.update(segments=_spread(rng, 2, 256), shortest=rng.choice([1, 64, 257]),
                     longest=rng.choice([1560, 4095, 8190]), lengths_seed=rng.randrange(1 << 16))
        else:
            c.update(B=rng.choice([1, 1, 2, 3, 4]), S=_spread(rng, 256, 75600))
    if op != "qk":
        c["mod"] = "sample"
    if op == "step":
        kind = rng.random()
        c["stats"] = kind >= 0.2
        if kind > 0.8 and "segments" not in c:
            c["mod"] = "token"
    while work(c)["bytes"] > MOST_BYTES:
        if "segments" in c:
            c["segments"] = c["segments"] // 2 + 1
        else:
            c["S"] = c["S"] // 2 + 1
    return c


def _lengths(case):
    """Tokens of each sample or segment."""
    if case.get("mix") == "video":
        return list(synth.varlen_lengths()[0])
    if "segments" in case:
        rng = random.Random(case["lengths_seed"])
        return [_spread(rng, case["shortest"], case["longest"]) for _ in range(case["segments"])]
    return [case["S"]] * case["B"]


def _packed(case):
    return "segments" in case or "mix" in case


def prepare(case, seed):
    dt, D = DTYPES[case["dtype"]], case["D"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    lens = _lengths(case)
    n, T = len(lens), sum(lens)

    def normal(*shape, mean=0.0, std=1.0):
        return (torch.randn(*shape, generator=g, device="cuda") * std + mean).to(dt)

    def activations(*shape):
        # hidden states: off centre, wide, and one value in a thousand an outlier
        v = torch.randn(*shape, generator=g, device="cuda") * 2.0 + 0.5
        v *= torch.where(torch.rand(*shape, generator=g, device="cuda") < 1e-3, 50.0, 1.0)
        return v.to(dt)

    grad = case["op"] != "infer"
    rows = (T, D) if _packed(case) else (case["B"], case["S"], D)
    s = {"case": case}
    if case["op"] == "qk":
        s["q"], s["k"] = activations(*rows).requires_grad_(), normal(*rows).requires_grad_()
        s["wq"], s["wk"] = (normal(D, mean=1.0, std=0.1).requires_grad_() for _ in range(2))
        s["dq"], s["dk"] = normal(*rows), normal(*rows)
        return s
    mod = rows if case["mod"] == "token" else (n, D)
    s["x"] = activations(*rows).requires_grad_(grad)
    s["shift"], s["scale"] = (normal(*mod, std=0.1).requires_grad_(grad) for _ in range(2))
    if _packed(case):
        ends = [0]
        for v in lens:
            ends.append(ends[-1] + v)
        s["cu"] = torch.tensor(ends, dtype=torch.int32, device="cuda")
    else:
        s["cu"] = None
    if grad:
        s["dy"] = normal(*rows)
    if case["op"] == "gated":
        s["u"], s["gate"] = normal(*rows).requires_grad_(), normal(n, D, std=0.3).requires_grad_()
        s["dh"] = normal(*rows)
    return s


def run(s):
    case = s["case"]
    if case["op"] == "infer":
        if s["cu"] is not None:
            return lnmod.forward_varlen(s["x"], s["shift"], s["scale"], s["cu"], EPS)
        return lnmod.forward(s["x"], s["shift"], s["scale"], EPS)
    if case["op"] == "step":
        y = functional.ln_modulate(s["x"], s["shift"], s["scale"], EPS, s["cu"], case["stats"])
        return (y.detach(),) + torch.autograd.grad(y, (s["x"], s["shift"], s["scale"]), s["dy"])
    if case["op"] == "gated":
        h, y = functional.gated_ln_modulate(s["x"], s["u"], s["gate"], s["shift"], s["scale"], EPS, s["cu"])
        return (h.detach(), y.detach()) + torch.autograd.grad(
            (h, y), (s["x"], s["u"], s["gate"], s["shift"], s["scale"]), (s["dh"], s["dy"]))
    q, k = functional.qk_norm(s["q"], s["k"], s["wq"], s["wk"], EPS)
    return (q.detach(), k.detach()) + torch.autograd.grad(
        (q, k), (s["q"], s["k"], s["wq"], s["wk"]), (s["dq"], s["dk"]))


def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    n, T, D = len(_lengths(case)), sum(_lengths(case)), case["D"]
    row = T * D                      # elements of one token-by-feature tensor
    mod = (row if case.get("mod") == "token" else n * D) * e
    if case["op"] == "infer":        # x, shift, scale -> y, mean, rstd
        return {"bytes": 2 * row * e + 2 * mod + 8 * T, "flops": 8 * row}
    if case["op"] == "step":         # x, shift, scale, dy -> y, dx, dshift, dscale
        return {"bytes": 4 * row * e + 4 * mod, "flops": 23 * row}
    if case["op"] == "gated":        # x, u, gate, shift, scale, dh, dy -> h, y, dx, du, dgate, dshift, dscale
        return {"bytes": 8 * row * e + 6 * mod, "flops": 30 * row}
    return {"bytes": 8 * row * e + 4 * D * e, "flops": 2 * 17 * row}      # q, k, dq, dk -> the same four


def tolerance(case):
    # bf16: a result is rounded once to 8 bits of mantissa, 1.7e-3 against float64 and at most half a unit in the
    # last place; fp32: sums of up to 75 600 rows or 8192 features in another order
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 1e-5, "max": 1e-4}


def _ln_backward(dy, scale, xhat, rstd):
    g = dy * (1.0 + scale)
    return (g - g.mean(-1, keepdim=True) - xhat * (g * xhat).mean(-1, keepdim=True)) * rstd


def exact(case, seed):
    s = {k: v.detach() if isinstance(v, torch.Tensor) else v for k, v in prepare(case, seed).items()}
    D = case["D"]
    if case["op"] == "qk":
        outs, ins, ws = [], [], []
        for t, w, d in ((s["q"], s["wq"], s["dq"]), (s["k"], s["wk"], s["dk"])):
            t, w, d = t.double(), w.double(), d.double()
            rstd = (t.square().mean(-1, keepdim=True) + EPS).rsqrt()
            xhat = t * rstd
            g = d * w
            outs.append(xhat * w)
            ins.append((g - xhat * (g * xhat).mean(-1, keepdim=True)) * rstd)
            ws.append((d * xhat).reshape(-1, D).sum(0))
        return (*outs, *ins, *ws)
    shape, cut = s["x"].shape, _lengths(case)
    token = case["mod"] == "token"
    parts = {}
    x = s["x"].reshape(-1, D)
    at = 0
    for m, n in enumerate(cut):                       # one sample or segment at a time
        r = slice(at, at + n)
        at += n
        scale, shift = ((s[k].reshape(-1, D)[r] if token else s[k][m]).double() for k in ("scale", "shift"))
        v = x[r].double()
        got = {}
        if case["op"] == "gated":
            gate, u = s["gate"][m].double(), s["u"].reshape(-1, D)[r].double()
            # the residual stream is kept in the tensors' own type, and everything after it is of the kept values
            got["h"] = (v + gate * u).float().to(s["x"].dtype).double()
            v = got["h"]
        mean = v.mean(-1, keepdim=True)
        rstd = ((v - mean).square().mean(-1, keepdim=True) + EPS).rsqrt()
        xhat = (v - mean) * rstd
        got["y"] = xhat * (1.0 + scale) + shift
        if case["op"] == "infer":
            got["mean"], got["rstd"] = mean[:, 0], rstd[:, 0]
        else:
            dy = s["dy"].reshape(-1, D)[r].double()
            got["dx"] = _ln_backward(dy, scale, xhat, rstd)
            if case["op"] == "gated":
                got["dx"] += s["dh"].reshape(-1, D)[r].double()
                got["du"] = gate * got["dx"]
                got["dgate"] = (u * got["dx"]).sum(0, keepdim=True)
            if token:
                got["dshift"], got["dscale"] = dy, dy * xhat
            else:
                got["dshift"], got["dscale"] = dy.sum(0, keepdim=True), (dy * xhat).sum(0, keepdim=True)
        for k, t in got.items():
            parts.setdefault(k, []).append(t)
    whole = {k: torch.cat(v) for k, v in parts.items()}
    rows = {"h", "y", "dx", "du"} | ({"dshift", "dscale"} if token else set())
    whole = {k: v.view(shape) if k in rows else v for k, v in whole.items()}
    if case["op"] == "infer":
        like = (case["B"], case["S"]) if not _packed(case) else (-1,)
        return whole["y"], whole["mean"].view(like), whole["rstd"].view(like)
    keys = ("h", "y", "dx", "du", "dgate", "dshift", "dscale") if case["op"] == "gated" else \
        ("y", "dx", "dshift", "dscale")
    return tuple(whole[k] for k in keys)
