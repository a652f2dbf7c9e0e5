"""The work that users of this package have it do, as cases that can be timed.

``listed()`` names the cases, ``draw()`` gives others of the same ranges, ``prepare()`` makes what a
program holds before the call (inputs on the GPU, scales, the plan object and buffers that it keeps from
step to step, layers with their weights), ``run()`` is one pass through the public entry points.

Kinds:
  gemm       the calling sequence of a product A B^T: quantise both operands, plan, unpack, fused GEMM
  oneshot    ``exact_int_gemm``: the same in one call, integer product beside the fp32 one
  resident   the calling sequence with the second operand's integers and its unpacking resident
             (``Plan.keep_weights``): inference on fixed weights, prefill (many rows) and decode (few rows)
  linear     ``IMUnpackLinear``: forward and backward (or forward alone) of a layer
  attention  ``IMUnpackAttention``: forward and backward (or forward alone) over sequences and heads
  load       what loading a weight takes: the range estimate, the RTN step, quantisation and scan
"""
from __future__ import annotations

import torch

from paper_2403_07339_amd import attention, binding as imu, linear

STRATEGY = {"row": imu.ROW, "col": imu.COL, "both": imu.BOTH}
# largest listed product (2 n d h): no drawn case is larger
LARGEST = 2.0 * 4096 * 4096 * 11008


def listed():
    return [
        # one small product, all latency: 0.5 % scattered heavy hitters in both operands
        dict(name="tiny-256", kind="gemm", n=256, d=256, h=256, b=8, sa="both", sb="both", da="scattered", db="scattered", t=False, fp6=False),
        # forward of a ViT-B MLP up-projection (64 images x 197 tokens), few outlier channels
        dict(name="vit-fc1", kind="gemm", n=12608, d=768, h=3072, b=8, sa="row", sb="col", da="channels", db="clean", t=False, fp6=False),
        # LLaMA-7B up-projection, both operands quantised and unpacked on every step (the benchmark's workload)
        dict(name="llama-up", kind="gemm", n=4096, d=4096, h=11008, b=8, sa="both", sb="both", da="channels", db="sparse", t=False, fp6=False),
        # weight gradient dW = dY^T X: transposed views, heavy-tailed gradient, contraction over 8192 tokens
        dict(name="wgrad", kind="gemm", n=4096, d=8192, h=4096, b=8, sa="both", sb="both", da="heavy", db="channels", t=True, fp6=False),
        # low bit width, many digits per value, six-bit digit storage
        dict(name="lowbit-4096", kind="gemm", n=4096, d=4096, h=4096, b=4, sa="row", sb="col", da="channels", db="clean", t=False, fp6=True),
        # odd sizes through the one-call form, with the int64 product
        dict(name="ragged", kind="oneshot", n=1000, d=1031, h=777, b=6, sa="col", sb="row", da="channels", db="clean", t=False),
        # the up-projection on weights that stay resident: a prefill of 4096 tokens and a decode batch of 16
        dict(name="prefill-resident", kind="resident", n=4096, d=4096, h=11008, b=8, sa="both", sb="both", da="channels", db="sparse"),
        dict(name="decode-resident", kind="resident", n=16, d=4096, h=11008, b=8, sa="row", sb="both", da="channels", db="sparse"),
        # a training step of a layer: 8 images x 197 tokens through the ViT-B up-projection, all three products
        dict(name="linear-train", kind="linear", n=1576, d=768, h=3072, b=8, sa="row", sb="col", beta_x=31, beta_w=31, beta_g=255, backward=True),
        # self-attention, 12 heads of 64 over 197 tokens: a training step of two sequences, inference of four at b = 4
        dict(name="attn-train", kind="attention", seqs=2, heads=12, tokens=197, head_dim=64, b=8, sa="both", sb="both", beta_x=31, beta_g=255, backward=True),
        dict(name="attn-infer-b4", kind="attention", seqs=4, heads=12, tokens=197, head_dim=64, b=4, sa="row", sb="col", beta_x=31, beta_g=255, backward=False),
        # a weight being loaded: percentile, step, integers and heavy-hitter statistics with the OB list
        dict(name="load-weight", kind="load", n=11008, d=4096, b=8, beta=31),
    ]


def _log(rng, lo, hi, odd=0.35):
    """A size between lo and hi, even over the logarithm; most are multiples of 8, some are anything."""
    v = lo * (hi / lo) ** rng.random()
    v = int(round(v))
    return max(lo, v if v < 16 or rng.random() < odd else v // 8 * 8)


def draw(rng):
    kind = rng.choice(["gemm"] * 6 + ["oneshot"] * 2 + ["resident"] * 3 + ["linear"] * 3 + ["attention"] * 3 + ["load"])
    while True:
        c = dict(kind=kind)
        if kind in ("gemm", "oneshot", "resident"):
            # UnpackBoth (a greedy over the heavy hitters) is for operands with few of them: b = 8
            c["b"] = rng.choice([8, 8, 8, 8, 6, 5, 4, 4, 3])
            pick = ["row", "col", "both"] if c["b"] == 8 else ["row", "col"]
            c["n"], c["d"], c["h"] = _log(rng, 32, 12608), _log(rng, 64, 8192), _log(rng, 64, 11008)
            c["sa"], c["sb"] = rng.choice(pick), rng.choice(pick)
            c["da"] = rng.choice(["channels", "channels", "scattered", "clean", "heavy"])
            c["db"] = rng.choice(["sparse", "clean", "channels"])
            if kind == "resident":
                c["n"], c["sa"] = _log(rng, 1, 4096), "row"
            else:
                c["t"] = rng.random() < 0.25
            if kind == "gemm":
                c["fp6"] = c["b"] <= 4 and rng.random() < 0.5
            # every digit level multiplies the work
            ratio = {8: 1, 6: 2, 5: 3, 4: 6, 3: 12}[c["b"]]
            if 2.0 * c["n"] * c["d"] * c["h"] * ratio > LARGEST:
                continue
        elif kind == "linear":
            c.update(n=_log(rng, 32, 8192), d=_log(rng, 64, 4096), h=_log(rng, 64, 4096), b=rng.choice([8, 8, 5, 4]), sa=rng.choice(["row", "col"]),
                     sb=rng.choice(["row", "col"]), beta_x=rng.choice([15, 31]), beta_w=rng.choice([15, 31]), beta_g=255, backward=rng.random() < 0.6)
            if 2.0 * c["n"] * c["d"] * c["h"] > LARGEST / 16:
                continue
        elif kind == "attention":
            c["b"] = rng.choice([8, 8, 4])
            pick = ["row", "col", "both"] if c["b"] == 8 else ["row", "col"]
            c.update(seqs=_log(rng, 1, 4), heads=_log(rng, 1, 12), tokens=_log(rng, 17, 256), head_dim=rng.choice([32, 40, 64, 128]),
                     sa=rng.choice(pick), sb=rng.choice(pick), beta_x=31, beta_g=255, backward=rng.random() < 0.5)
        else:
            c.update(n=_log(rng, 64, 11008), d=_log(rng, 64, 4096), b=rng.choice([8, 6, 4]), beta=rng.choice([15, 31, 255]))
        return c


# ---- inputs ----------------------------------------------------------------------------------------
def _matrix(g, rows, cols, kind, std=1.0, factor=None):
    """fp32 rows x cols, heavy hitters over the contracted index as activations, weights and gradients show them."""
    x = torch.randn(rows, cols, generator=g, device="cuda") * std
    if kind == "channels":            # outlier channels: 0.5 % of the columns
        idx = torch.randperm(cols, generator=g, device="cuda")[:max(1, round(0.005 * cols))]
        x[:, idx] *= factor or 100.0
    elif kind in ("scattered", "sparse"):   # single entries: 0.5 % x 64 of an activation, 0.1 % x 20 of a weight
        share, f = (0.005, 64.0) if kind == "scattered" else (0.001, 20.0)
        x[torch.rand(rows, cols, generator=g, device="cuda") < share] *= factor or f
    elif kind == "heavy":             # Student-t with three degrees of freedom
        chi2 = sum(torch.randn(rows, cols, generator=g, device="cuda") ** 2 for _ in range(3))
        x = x / torch.sqrt(chi2 / 3.0)
    return x


def _scale(x):
    return float((4.0 * x.double().std(unbiased=False) / 127.0).float().item())


def _operand(g, rows, cols, kind, transposed, std=1.0):
    x = _matrix(g, rows, cols, kind, std)
    return x.t().contiguous().t() if transposed else x


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    st = {"case": c}
    kind = c["kind"]
    if kind in ("gemm", "oneshot", "resident"):
        n, d, h = c["n"], c["d"], c["h"]
        A = _operand(g, n, d, c["da"], c.get("t", False))
        B = _operand(g, h, d, c["db"], c.get("t", False), 0.02 if c["db"] in ("sparse", "clean") else 1.0)
        st.update(A=A, B=B, scale_a=_scale(A), scale_b=_scale(B), sa=STRATEGY[c["sa"]], sb=STRATEGY[c["sb"]], plan=imu.Plan())
        if kind == "oneshot":
            return st
        cap = imu.Stats.default_ob_cap
        st.update(Qa=torch.empty((n, d), dtype=torch.int32, device="cuda"), Qb=torch.empty((h, d), dtype=torch.int32, device="cuda"),
                  st_a=imu.Stats.empty(n, d, A.device, cap(n, d) if c["sa"] == "both" else 0),
                  st_b=imu.Stats.empty(h, d, A.device, cap(h, d) if c["sb"] == "both" else 0),
                  status=torch.zeros(2, dtype=torch.int32, device="cuda"), C=torch.empty((n, h), dtype=torch.float32, device="cuda"), A_ue=None, B_eu=None, ws=None, fp6=c.get("fp6", False))
        if kind == "resident":
            # the weights are quantised and unpacked when they are loaded, beside activations of an earlier batch
            # with the same outlier channels; from then on the plan keeps their unpacking
            imu.imunpack_quantize(B, st["scale_b"], c["b"], st["Qb"], st["st_b"], st["status"][1:2])
            st["fp6"] = c["b"] <= 4
            now, st["A"] = st["A"], A.flip(0).contiguous()
            run(st)
            st["plan"].keep_weights()
            run(st)
            st["A"] = now
        return st
    if kind == "linear":
        n, d, h = c["n"], c["d"], c["h"]
        cfg = linear.QuantConfig(beta_x=float(c["beta_x"]), beta_w=float(c["beta_w"]), beta_g=float(c["beta_g"]), b=c["b"], strategy_a=STRATEGY[c["sa"]], strategy_b=STRATEGY[c["sb"]])
        layer = linear.IMUnpackLinear(d, h, bias=True, cfg=cfg, device="cuda")
        with torch.no_grad():
            layer.weight.copy_(_matrix(g, h, d, "sparse", 0.02))
            layer.bias.copy_(torch.randn(h, generator=g, device="cuda") * 0.02)
        st.update(layer=layer, x=_matrix(g, n, d, "channels", factor=30.0).requires_grad_(c["backward"]))
        if c["backward"]:
            st["gy"] = _matrix(g, n, h, "scattered", 1e-3, factor=40.0)
        return st
    if kind == "attention":
        shape = (c["seqs"], c["heads"], c["tokens"], c["head_dim"])
        cfg = linear.QuantConfig(beta_x=float(c["beta_x"]), beta_g=float(c["beta_g"]), b=c["b"], strategy_a=STRATEGY[c["sa"]], strategy_b=STRATEGY[c["sb"]])
        st["attn"] = attention.IMUnpackAttention(cfg)
        q, k, v = (torch.randn(shape, generator=g, device="cuda") for _ in range(3))
        k[..., 5] *= 12.0             # an outlier channel in the keys
        st["qkv"] = [t.requires_grad_(c["backward"]) for t in (q, k, v)]
        if c["backward"]:
            go = torch.randn(shape, generator=g, device="cuda") * 1e-2
            go[torch.rand(shape, generator=g, device="cuda") < 0.01] *= 30.0
            st["go"] = go
        return st
    W = _matrix(g, c["n"], c["d"], "sparse", 0.02)
    st.update(W=W, stats=imu.Stats.empty(c["n"], c["d"], W.device, imu.Stats.default_ob_cap(c["n"], c["d"])))
    return st


# ---- one pass --------------------------------------------------------------------------------------
def _sequence(s):
    """quantise -> plan -> unpack -> fused GEMM, buffers kept and grown as a training or serving loop does."""
    c, plan = s["case"], s["plan"]
    if c["kind"] == "resident":
        imu.imunpack_quantize(s["A"], s["scale_a"], c["b"], s["Qa"], s["st_a"], s["status"][0:1])
    else:
        imu.imunpack_quantize_pair(s["A"], s["B"], s["scale_a"], s["scale_b"], c["b"], s["Qa"], s["Qb"], s["st_a"], s["st_b"], s["status"])
    imu.imunpack_plan(s["Qa"], s["Qb"], c["b"], s["sa"], s["sb"], s["st_a"], s["st_b"], plan)
    if s["fp6"] and plan.digits() != imu.DIGITS_FP6:
        plan.set_digits(imu.DIGITS_FP6)
    ba, bb, bw = plan.unpacked_bytes()
    if s["A_ue"] is None or s["A_ue"].numel() < ba:
        s["A_ue"] = torch.empty(ba, dtype=torch.int8, device="cuda")
    if s["B_eu"] is None or s["B_eu"].numel() < bb:
        s["B_eu"] = torch.empty(bb, dtype=torch.int8, device="cuda")
    imu.imunpack_unpack(plan, s["Qa"], s["Qb"], s["A_ue"], s["B_eu"])
    # the fused launch goes out before the host knows whether it is exact; if it was not, the call falls
    # back on the workspace, or says that it needs one
    try:
        imu.imunpack_gemm(plan, s["A_ue"], s["B_eu"], s["scale_a"], s["scale_b"], None, s["C"], s["ws"])
    except imu.ImunpackError as e:
        if e.code != imu.ERANGE:
            raise
        s["ws"] = torch.empty(bw // 8, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, s["A_ue"], s["B_eu"], s["scale_a"], s["scale_b"], None, s["C"], s["ws"])
    return s["C"]


def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind in ("gemm", "resident"):
        return _sequence(s)
    if kind == "oneshot":
        C_int, C_fp, _ = imu.exact_int_gemm(s["A"], s["B"], s["scale_a"], s["scale_b"], c["b"], s["sa"], s["sb"], plan=s["plan"])
        return {"C_int": C_int, "C_fp": C_fp}
    if kind == "linear":
        layer, x = s["layer"], s["x"]
        if not c["backward"]:
            with torch.no_grad():
                return layer(x)
        x.grad = layer.weight.grad = layer.bias.grad = None
        y = layer(x)
        y.backward(s["gy"])
        return {"y": y.detach(), "x": x.grad, "weight": layer.weight.grad, "bias": layer.bias.grad}
    if kind == "attention":
        if not c["backward"]:
            with torch.no_grad():
                return s["attn"](*s["qkv"])
        for t in s["qkv"]:
            t.grad = None
        o = s["attn"](*s["qkv"])
        o.backward(s["go"])
        return {"o": o.detach(), "q": s["qkv"][0].grad, "k": s["qkv"][1].grad, "v": s["qkv"][2].grad}
    alpha, _ = imu.imunpack_percentile(s["W"], 95.0)
    scale = float(alpha.item()) / (0.5 * c["beta"])      # the loader keeps the scale with the weight
    Q, stats, _ = imu.imunpack_quantize(s["W"], scale, c["b"], stats=s["stats"])
    return {"alpha": alpha, "Q": Q, "rowcnt": stats.rowcnt, "colcnt": stats.colcnt, "rowmax": stats.rowmax, "colmax": stats.colmax, "ob_count": stats.ob_count}


# ---- what a pass cannot do without -------------------------------------------------------------------
def work(case):
    c, kind = case, case["kind"]
    if kind in ("gemm", "oneshot", "resident"):
        n, d, h = c["n"], c["d"], c["h"]
        out = 12 if kind == "oneshot" else 4
        # resident weights are integers already: one byte per entry at least
        return {"bytes": 4.0 * n * d + (1.0 if kind == "resident" else 4.0) * h * d + out * n * h, "flops": 2.0 * n * d * h}
    if kind == "linear":
        n, d, h = c["n"], c["d"], c["h"]
        once = n * d + h * d + n * h + h
        return {"bytes": 4.0 * once * (2 if c["backward"] else 1), "flops": (6.0 if c["backward"] else 2.0) * n * d * h}
    if kind == "attention":
        items, t, e = c["seqs"] * c["heads"], c["tokens"], c["head_dim"]
        return {"bytes": 4.0 * items * t * e * (8 if c["backward"] else 4), "flops": (12.0 if c["backward"] else 4.0) * items * t * t * e}
    return {"bytes": 8.0 * c["n"] * c["d"], "flops": 1.0 * c["n"] * c["d"]}


def tolerance(case):
    """Integers, counts and positions are exact.  A product is an exact integer that is scaled and rounded to fp32:
    rounding the scale and the result in fp32 instead of once from binary64 measures 6e-8.  Attention puts fp32
    softmax arithmetic between the products: a last-bit difference there moves entries of the next operand over a
    rounding boundary (a whole step of the quantiser); with the softmax in binary64 instead the outputs differ by up to
    1e-4 (2-norm) and by 0.013 of their root mean square at one place.  The bias gradient is an fp32 sum (1e-7)."""
    if case["kind"] == "load":
        return "exact"
    if case["kind"] == "attention":
        return {"rel": 4e-4, "max": 0.05}
    if case["kind"] == "linear":
        return {"rel": 1e-6}
    return {"rel": 2.5e-7, "max": 1e-6}
