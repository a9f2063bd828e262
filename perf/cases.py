"""The calls that this library is timed on: sizes, inputs, one pass, the work it cannot do without, and how far
two correct implementations may differ.

A case is one call through the public entry points, as a denoising loop makes it at one place of a video U-Net:
a sliced transformer block (temporal or spatial), a Spatial ResBlock, its Up/DownSample, the Step Rehash
similarity test, and a block under Step Rehash that finds its cached output still good.

Inputs follow the repository's recipe: features and context ~ N(0,1), matrices and kernels ~ N(0, 0.02^2), norm
gains ~ N(1, 0.1^2), shifts and biases ~ N(0, 0.1^2); query and key projections are scaled to 1/sqrt(fan-in), so
that attention scores have unit variance and a softmax is neither flat nor one-hot.
"""
import math

import torch

import paper_2411_01171_amd as si

TEMPORAL, SPATIAL = "temporal", "spatial"
DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}


def _block(kind, C, F, H, W, heads, slice_len, *, B=2, dtype="bf16", pe=False, ctx=(0, 0), packed=False, rehash=False):
    return {"op": "rehash_step" if rehash else "block", "kind": kind, "dtype": dtype, "B": B, "C": C, "F": F, "H": H, "W": W,
            "heads": heads, "dim_head": C // heads, "pe": pe, "ctx_tokens": ctx[0], "ctx_dim": ctx[1],
            "slice_len": slice_len, "packed": packed}


def _resblock(C, F, H, W, slice_len, *, B=2, C_out=0, temb=1280):
    return {"op": "resblock", "dtype": "bf16", "B": B, "C": C, "C_out": C_out or C, "F": F, "H": H, "W": W, "temb": temb,
            "slice_len": slice_len}


def _resample(kind, C, F, H, W, slice_len, *, B=2):
    return {"op": "resample", "kind": kind, "dtype": "bf16", "B": B, "C": C, "F": F, "H": H, "W": W, "slice_len": slice_len}


def _check(C, F, H, W, *, B=2, dtype="bf16"):
    return {"op": "rehash_check", "dtype": dtype, "B": B, "C": C, "F": F, "H": H, "W": W}


def listed():
    return [dict(case, name=name) for name, case in (
        # the smallest block: an 8x8 map in single precision, as a numerics check of an integration runs it; all latency
        ("temporal_64_f32", _block(TEMPORAL, 64, 8, 8, 8, 1, 16, B=1, dtype="f32")),
        # motion module of a 512x512 16-frame model at the top level (64x64 latent, 8 heads of 40), four position windows
        ("temporal_320_d40", _block(TEMPORAL, 320, 16, 64, 64, 8, 1024, pe=True)),
        # the spatial block before it: same feature and heads, text context, one frame per slice
        ("spatial_320_d40", _block(SPATIAL, 320, 16, 64, 64, 8, 1, ctx=(77, 768))),
        # second level of such a model, heads of 64, one frame per slice
        ("spatial_640_d64", _block(SPATIAL, 640, 16, 32, 32, 10, 1, ctx=(77, 768))),
        # motion module of the second level at a ragged size: 8 heads of 80, 14 frames, 45x50 positions, windows of
        # 500 with a last one of 250, one batch entry (no guidance)
        ("temporal_640_d80_ragged", _block(TEMPORAL, 640, 14, 45, 50, 8, 500, B=1, pe=True)),
        # image-to-video model at 576x1024, 25 frames (72x128 latent), first level: the largest call
        ("spatial_320_d64", _block(SPATIAL, 320, 25, 72, 128, 5, 1, ctx=(1, 1024))),
        # the temporal block behind it, eight position windows
        ("temporal_320_d64", _block(TEMPORAL, 320, 25, 72, 128, 5, 1152)),
        # deepest level; weights stay re-laid-out in the workspace over the diffusion steps
        ("spatial_1280_d64", _block(SPATIAL, 1280, 16, 16, 16, 20, 4, ctx=(77, 768), packed=True)),
        # its temporal block, weights re-laid-out in the call
        ("temporal_1280_d64", _block(TEMPORAL, 1280, 16, 16, 16, 20, 64)),
        # first-level ResBlock of the image-to-video model, one frame per slice
        ("resblock_320", _resblock(320, 25, 72, 128, 1)),
        # its DownSample
        ("downsample_320", _resample("down", 320, 25, 72, 128, 1)),
        # Step Rehash: is the largest feature still the cached one?
        ("rehash_check_295mb", _check(320, 25, 72, 128)),
    )]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _map(rng, lo, hi):
    """Height and width of a latent map: square or 16:9, half of the time any size, else multiples of 8."""
    H = _log_int(rng, lo, hi)
    W = int(round(H * rng.choice((1.0, 1.0, 16 / 9, 1.1))))
    if rng.random() < 0.5:
        H, W = max(8, H // 8 * 8), max(8, W // 8 * 8)
    return H, W


# channels, heads (of 40, 64 and 80 channels), largest map height at that level
_LEVELS = ((320, 8, 72), (320, 5, 72), (640, 8, 36), (640, 10, 36), (1280, 20, 18))


def _class(case):
    """Cases of one class are bounded by the listed case of that class with the most work."""
    return (case["op"], case.get("kind") if case["op"] == "block" else "", case.get("dim_head", 0) % 64 == 0)


def _draw_one(rng):
    op = rng.choice((TEMPORAL,) * 6 + (SPATIAL,) * 6 + ("rehash_step", "f32") + ("resblock",) * 3 + ("down", "up") + ("check",) * 2)
    B, F = rng.choice((1, 2, 2)), rng.randint(6, 28)
    if op in (TEMPORAL, SPATIAL, "rehash_step", "f32"):
        C, heads, top = rng.choice(_LEVELS)
        kind = op if op in (TEMPORAL, SPATIAL) else rng.choice((TEMPORAL, SPATIAL))
        dtype = "bf16"
        if op == "f32":
            C, heads = rng.choice(((64, 1), (64, 2), (128, 2), (320, 5)))
            F, top, dtype = rng.randint(4, 16), 20, "f32"
        H, W = _map(rng, 8, top)
        if kind == TEMPORAL:
            slice_len = -(-H * W // rng.choice((1, 2, 3, 4, 4, 8)))
        else:
            slice_len = min(F, rng.choice((1, 1, 2, 3, 4)))
        ctx = rng.choice(((77, 768), (77, 1024), (1, 1024), (16, 768))) if kind == SPATIAL else (0, 0)
        return _block(kind, C, F, H, W, heads, slice_len, B=B, dtype=dtype, pe=kind == TEMPORAL and rng.random() < 0.5, ctx=ctx,
                      packed=op != "rehash_step" and rng.random() < 0.5, rehash=op == "rehash_step")
    if op == "check":
        H, W = _map(rng, 8, 72)
        return _check(rng.choice((64, 320, 640)), F, H, W, B=B, dtype=rng.choice(("bf16", "bf16", "f32")))
    C = rng.choice((320, 640, 1280))
    H, W = _map(rng, 8, 72 * 320 // C)
    if op == "resblock":
        return _resblock(C, F, H, W, rng.choice((1, 1, 2, 4)), B=B, C_out=rng.choice((C, C, 320, 640)), temb=rng.choice((0, 1280)))
    return _resample(op, C, F, H, W, rng.choice((1, 1, 2, 4)), B=B)


def draw(rng):
    fixed = listed()
    top = max(work(c)["flops"] for c in fixed)
    while True:
        case = _draw_one(rng)
        most = max((work(c)["flops"] for c in fixed if _class(c) == _class(case)), default=top)
        if case["op"] == "resample":
            most *= 4  # doubling a feature contracts on four times the positions, halving it on a quarter
        if case["op"] == "rehash_check" or work(case)["flops"] <= most:
            return case


def _normal(gen, shape, dtype, std=1.0, mean=0.0):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(std).add_(mean).to(dtype)


def _feature(case, gen, channels=None):
    return _normal(gen, (case["B"], channels or case["C"], case["F"], case["H"], case["W"]), DTYPE[case["dtype"]])


def _block_weights(case, gen):
    C, D, Cc, dt = case["C"], case["heads"] * case["dim_head"], case["ctx_dim"], DTYPE[case["dtype"]]
    spatial = case["kind"] == SPATIAL
    mats = {"w_in": (C, D), "wq": (D, D), "wk": (D, D), "wv": (D, D), "wo": (D, D), "w1": (D, 8 * D), "w2": (4 * D, D), "w_out": (D, C)}
    vecs = {"b_in": D, "bo": D, "b1": 8 * D, "b2": D, "b_out": C, "gn_b": C, "ln1_b": D, "ln3_b": D}
    gains = {"gn_g": C, "ln1_g": D, "ln3_g": D}
    if spatial:
        mats.update(wq2=(D, D), wk2=(Cc, D), wv2=(Cc, D), wo2=(D, D))
        vecs.update(bo2=D, ln2_b=D)
        gains.update(ln2_g=D)
    t = {n: _normal(gen, s, dt, s[0] ** -0.5 if n in ("wq", "wk", "wq2", "wk2") else 0.02) for n, s in mats.items()}
    t.update({n: _normal(gen, (s,), dt, 0.1) for n, s in vecs.items()})
    t.update({n: _normal(gen, (s,), dt, 0.1, 1.0) for n, s in gains.items()})
    return si.BlockWeights(si.SI_BLOCK_SPATIAL if spatial else si.SI_BLOCK_TEMPORAL, case["heads"], case["dim_head"], 32, t,
                           add_sin_pe=case["pe"])


def _resblock_weights(case, gen):
    C, Co, T, dt = case["C"], case["C_out"], case["temb"], torch.bfloat16
    t = {"w_conv1": _normal(gen, (Co, C, 3, 3), dt, 0.02), "w_conv2": _normal(gen, (Co, Co, 3, 3), dt, 0.02)}
    vecs = {"b_conv1": Co, "b_conv2": Co, "gn1_b": C, "gn2_b": Co}
    if T:
        t["w_temb"] = _normal(gen, (T, Co), dt, 0.02)
        vecs["b_temb"] = Co
    if Co != C:
        t["w_skip"] = _normal(gen, (Co, C), dt, 0.02)
        vecs["b_skip"] = Co
    t.update({n: _normal(gen, (s,), dt, 0.1) for n, s in vecs.items()})
    t.update({n: _normal(gen, (s,), dt, 0.1, 1.0) for n, s in (("gn1_g", C), ("gn2_g", Co))})
    return si.ResBlockWeights(32, t, temb_dim=T, c_out=Co)


def _bytes(n):
    assert n > 0, "the library rejected the arguments"
    return torch.empty(n, dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    s = {"case": case, "x": _feature(case, gen)}
    x, op = s["x"], case["op"]
    if op in ("block", "rehash_step"):
        s["ctx"] = _normal(gen, (case["B"], case["ctx_tokens"], case["ctx_dim"]), x.dtype) if case["kind"] == SPATIAL else None
        s["w"] = _block_weights(case, gen)
        s["axis"] = si.SI_AXIS_F if case["kind"] == SPATIAL else si.SI_AXIS_HW
        s["ws"] = _bytes(si.si_workspace_bytes(x, s["w"], s["ctx"], s["axis"], case["slice_len"]))
        s["out"] = torch.empty_like(x)
        if op == "rehash_step":
            # the anchor: an earlier step's feature, which the block was computed on; x has moved a little since
            s["cache"] = si.RehashCache(x)
            before = _normal(gen, x.shape, torch.float32, 0.1).add_(x).to(x.dtype)
            si.si_block_forward_rehash(before, s["w"], s["ctx"], s["out"], s["axis"], case["slice_len"], s["ws"], s["cache"], 0.95)
        elif case["packed"]:
            si.si_block_forward(x, s["w"], s["ctx"], s["out"], s["axis"], case["slice_len"], s["ws"])
    elif op == "resblock":
        s["w"] = _resblock_weights(case, gen)
        s["temb"] = _normal(gen, (case["B"], case["temb"]), x.dtype) if case["temb"] else None
        s["ws"] = _bytes(si.si_resblock_workspace_bytes(x, s["w"], case["slice_len"]))
        s["out"] = torch.empty((case["B"], case["C_out"], *x.shape[2:]), dtype=x.dtype, device="cuda")
    elif op == "resample":
        C, (H, W) = case["C"], _resampled(case)
        s["kind"] = si.SI_RESAMPLE_DOWN if case["kind"] == "down" else si.SI_RESAMPLE_UP
        s["w"], s["b"] = _normal(gen, (C, C, 3, 3), x.dtype, 0.02), _normal(gen, (C,), x.dtype, 0.1)
        s["ws"] = _bytes(si.si_resample_workspace_bytes(x, s["kind"], case["slice_len"]))
        s["out"] = torch.empty((case["B"], C, case["F"], H, W), dtype=x.dtype, device="cuda")
    else:
        s["before"] = _normal(gen, x.shape, torch.float32, 0.3).add_(x).to(x.dtype)
        s["scratch"] = _bytes(si.si_rehash_scratch_bytes(x.numel()))
        s["cos"] = torch.empty(1, dtype=torch.float64, device="cuda")
        s["decision"] = torch.empty(1, dtype=torch.int32, device="cuda")
    return s


def run(s):
    case, x = s["case"], s["x"]
    op = case["op"]
    if op == "block":
        si.si_block_forward_ex(x, s["w"], s["ctx"], s["out"], s["axis"], case["slice_len"], s["ws"],
                               si.SI_FWD_WEIGHTS_PACKED if case["packed"] else 0)
        return s["out"]
    if op == "rehash_step":
        reused, cos = si.si_block_forward_rehash(x, s["w"], s["ctx"], s["out"], s["axis"], case["slice_len"], s["ws"], s["cache"], 0.95)
        return {"out": s["out"], "reused": reused, "cos": cos}
    if op == "resblock":
        si.si_resblock_forward(x, s["w"], s["temb"], s["out"], case["slice_len"], s["ws"])
        return s["out"]
    if op == "resample":
        si.si_resample_forward(x, s["kind"], s["w"], s["b"], s["out"], case["slice_len"], s["ws"])
        return s["out"]
    si.si_rehash_check(x, s["before"], 0.95, s["cos"], s["decision"], s["scratch"])
    return {"cos": s["cos"], "decision": s["decision"]}


def _resampled(case):
    return (-(-case["H"] // 2), -(-case["W"] // 2)) if case["kind"] == "down" else (2 * case["H"], 2 * case["W"])


def work(case):
    """Features in and out once, parameters once; contractions as 2mnk, attention as 4 Nq Nk d per head."""
    size = 4 if case["dtype"] == "f32" else 2
    B, C, F, P, op = case["B"], case["C"], case["F"], case["H"] * case["W"], case["op"]
    T = B * F * P
    if op == "rehash_check":
        return {"bytes": 2 * T * C * size, "flops": 6 * T * C}
    if op == "rehash_step":
        return {"bytes": 4 * T * C * size, "flops": 6 * T * C}  # x and the anchor are compared, the cached output is copied
    if op == "block":
        D, M, Cc = case["heads"] * case["dim_head"], case["ctx_tokens"], case["ctx_dim"]
        params = 2 * C * D + 16 * D * D
        flops = 2 * T * params
        if case["kind"] == SPATIAL:
            params += 2 * D * D + 2 * Cc * D
            flops += 4 * T * D * D + 4 * B * M * Cc * D + 4 * T * (P + M) * D
        else:
            flops += 4 * T * F * D
        return {"bytes": (2 * T * C + params + B * M * Cc) * size, "flops": flops}
    if op == "resblock":
        Co, E = case["C_out"], case["temb"]
        params = 9 * (C + Co) * Co + E * Co + (C * Co if Co != C else 0)
        flops = 18 * T * (C + Co) * Co + (2 * T * C * Co if Co != C else 0) + 2 * B * E * Co
        return {"bytes": (T * (C + Co) + params) * size, "flops": flops}
    H, W = _resampled(case)
    To = B * F * H * W
    return {"bytes": ((T + To) * C + 9 * C * C) * size, "flops": 18 * To * C * C}


def tolerance(case):
    """About four times what the calls differ by from the same operators in 64 bits, the largest seen over the
    listed cases and a score of drawn ones."""
    if case["op"] in ("rehash_check", "rehash_step"):
        # 64-bit sums in another order (6e-16); the decision and the handed-back output stay what they are
        return {"rel": 1e-14, "max": 1e-14}
    if case["dtype"] == "f32":
        return {"rel": 3e-7, "max": 2.5e-6}  # 7.5e-8, 5.8e-7
    if case["op"] == "resample":
        return {"rel": 7e-3, "max": 1.6e-2}  # exact operands, one rounding of the result to bf16: 1.7e-3, 3.9e-3
    return {"rel": 8e-3, "max": 4e-2}  # the roundings of the contractions' operands as well: 2.0e-3, 9.5e-3
