"""Attention holds its probabilities and sums in fp32 wherever the bf16 matrix-core kernel (heads of 64, H*W a multiple
of 8) does not run: inputs on which the values cancel, so that a probability rounded to fewer bits changes the result
by its own size, against the float64 oracle."""
import numpy as np
import pytest

import oracle
import si_workloads as wl
from helpers import tiny_spec

pytestmark = pytest.mark.gpu

SCORE_CH = 8  # channels that scores are formed from; the values come from the others


def _antisymmetric_tokens(rng, n, width):
    """n tokens, the second half minus the first (an odd one out is zero): values cancel at equal probabilities."""
    h = n // 2
    t = np.zeros((n, width))
    t[:h, :SCORE_CH] = 0.2 * rng.standard_normal((h, SCORE_CH))
    t[:h, SCORE_CH:] = rng.standard_normal((h, width - SCORE_CH))
    t[0, :SCORE_CH] *= 5
    t[h:2 * h] = -t[:h]
    return t


def _weights(spec, rng, cross):
    """Attention's output alone reaches the result: x fills the lower half of the channels, the out-projection the upper
    half of D, proj_out reads that half only, everything else adds nothing."""
    D, C = spec.heads * spec.dim_head, spec.C
    w = {k: np.zeros_like(v) if not k.endswith("_g") else v for k, v in wl.make_weights(spec).items()}
    w["w_in"][:C // 2, :D // 2] = np.eye(C // 2, D // 2)
    q, k, v, o = ("wq2", "wk2", "wv2", "wo2") if cross else ("wq", "wk", "wv", "wo")
    for h in range(spec.heads):
        for c in range(SCORE_CH):
            w[q][c, h * spec.dim_head + c] = 2.0 ** -8  # scores of 1e-3: probabilities within 1e-3 of each other
            w[k][c, h * spec.dim_head + c] = 1.0
    w[v][SCORE_CH:, :] = rng.standard_normal(w[v][SCORE_CH:, :].shape) / np.sqrt(D)
    w[o][:, D // 2:] = 1024 * rng.standard_normal((D, D - D // 2)) / np.sqrt(D)
    w["w_out"][D // 2:] = 64 * rng.standard_normal((D - D // 2, C)) / np.sqrt(D)
    return {n: wl.round_to_storage(a, "bf16") for n, a in w.items()}


# probabilities in bf16 are off by 2^-9 where they differ by 1e-3: errors of 0.3 .. 2 of the branch.  In fp32 what is
# left are the roundings of LN's output, q, k, v and the attention's output to bf16, 1.1e-3 each on average: 3e-3 .. 6e-3
BRANCH_REL = 2e-2


@pytest.mark.parametrize("cross", [False, True])
@pytest.mark.parametrize("heads,d,hw", [(4, 40, (8, 8)), (8, 40, (16, 24)), (2, 80, (9, 7)), (2, 80, (40, 40)), (5, 64, (9, 11)), (1, 128, (8, 12)), (4, 16, (8, 8))])
def test_spatial(heads, d, hw, cross):
    from gpu_helpers import errors, run_block
    C = heads * d
    n = hw[0] * hw[1]
    spec = tiny_spec(wl.SPATIAL, B=1, C=C, F=2, H=hw[0], W=hw[1], heads=heads, dim_head=d, groups=1, M=90, Cc=C, dtype="bf16")
    rng = np.random.default_rng(n + d)
    x = np.zeros((1, C, 2, n))
    for f in range(2):
        x[0, :C // 2, f] = _antisymmetric_tokens(rng, n, C // 2).T
    x = wl.round_to_storage(x.reshape(1, C, 2, *hw), "bf16")
    ctx = wl.round_to_storage(_antisymmetric_tokens(rng, 90, C)[None], "bf16")
    w = _weights(spec, rng, cross)
    ref = oracle.block_forward_ref(x, w, spec, ctx)
    e = errors(run_block(spec, x, w, ctx, 1), ref, x)
    print(e)
    assert e["rel_l2_branch"] <= BRANCH_REL


# temporal sequences: q, k and v themselves are read off the device (one-frame sequences return their values), so that
# the comparison holds attention alone
VALUE_GAIN = 4096.0  # keeps the output in the normal range of the fp16 operand of proj_out


def _temporal_inputs(F, heads, d, hw):
    """Frames 2 i and 2 i + 1 agree in the channels that scores come from and are opposite in those that values come
    from; a weak share of the latter makes their scores differ by about 1e-5."""
    D = C = heads * d
    spec = tiny_spec(wl.TEMPORAL, B=1, C=C, F=F, H=hw[0], W=hw[1], heads=heads, dim_head=d, groups=C // 8, dtype="bf16")
    rng = np.random.default_rng(F + d)
    P, half, quarter = hw[0] * hw[1], D // 2, D // 4
    x = np.zeros((1, C, F, P))
    x[0, :SCORE_CH] = np.repeat(rng.standard_normal((SCORE_CH, (F + 1) // 2, P)), 2, axis=1)[:, :F]
    x[0, SCORE_CH:quarter] = np.repeat(rng.standard_normal((quarter - SCORE_CH, (F + 1) // 2, P)), 2, axis=1)[:, :F]
    x[0, SCORE_CH:quarter, 1::2] *= -1
    if F % 2:
        x[0, SCORE_CH:quarter, F - 1] = 0  # the odd frame out has no values
    w = {k: np.zeros_like(v) if not k.endswith("_g") else v for k, v in wl.make_weights(spec).items()}
    for c in range(quarter):  # every channel and its negative: LayerNorm's mean is zero, its output opposite where x is
        w["w_in"][c, c] = 1
        w["w_in"][c, quarter + c] = -1
    for h in range(heads):
        for c in range(SCORE_CH // 2):
            w["wq"][c, h * d + c] = 0.25
            w["wk"][c, h * d + c] = 1
            w["wq"][c, h * d + 4 + c] = 2.0 ** -8
            w["wk"][SCORE_CH + c, h * d + 4 + c] = 2.0 ** -6
    w["wv"][SCORE_CH:quarter] = rng.standard_normal((quarter - SCORE_CH, D)) / np.sqrt(quarter)
    w["wo"][:half, half:] = VALUE_GAIN * np.eye(half)
    w["w_out"][half:, half:] = np.eye(half)
    return spec, wl.round_to_storage(x.reshape(1, C, F, *hw), "bf16"), {n: wl.round_to_storage(a, "bf16") for n, a in w.items()}


def _attention_output(spec, x, w):
    """The first half of the heads' channels of the attention output, [B, F, P, D / 2]."""
    from gpu_helpers import run_block
    half = spec.C // 2
    out = run_block(spec, x, w, None, x.shape[3] * x.shape[4])[:, half:]
    return (out / VALUE_GAIN).reshape(x.shape[0], half, x.shape[2], -1).transpose(0, 2, 3, 1)


# the output's rounding to bf16 is 1.7e-3; expf and the sums add 6e-8 to each of the terms that differ by 1e-5.  Probabilities
# of 16 significand bits move in steps of 4e-6: 2.5e-2 and more
TEMPORAL_REL = 5e-3


@pytest.mark.parametrize("F", [5, 14, 16, 31, 32])
@pytest.mark.parametrize("heads,d", [(2, 40), (2, 64), (2, 80), (1, 128)])
def test_temporal(heads, d, F):
    spec, x, w = _temporal_inputs(F, heads, d, (3, 5))
    D, half = heads * d, heads * d // 2
    # every frame as a batch entry of one frame: attention hands back its value projection
    single = wl.scaled(spec, B=F, F=1)
    frames = np.ascontiguousarray(x.transpose(2, 1, 0, 3, 4))
    q, k, v = (_attention_output(single, frames, dict(w, wv=w[n]))[:, 0].transpose(1, 0, 2) for n in ("wq", "wk", "wv"))
    got = _attention_output(spec, x, w)[0].transpose(1, 0, 2)
    nh = half // d  # whole heads among the channels that are read; a single head of 128 shows the first half of its own
    for h in range(max(nh, 1)):
        cs = slice(h * d, min(h * d + d, half))
        ref = oracle.attention_ref(q[:, :, cs], k[:, :, cs], v[:, :, cs], 1) if nh else None
        if ref is None:  # channels past the first eight hold no scores
            s = np.einsum("pic,pjc->pij", q[..., :8], k[..., :8]) / np.sqrt(d)
            p = np.exp(s - s.max(-1, keepdims=True))
            ref = np.einsum("pij,pjc->pic", p / p.sum(-1, keepdims=True), v[:, :, cs])
        e = np.linalg.norm(got[:, :, cs] - ref) / np.linalg.norm(ref)
        print(F, heads, d, h, "rel", e, "size", np.sqrt(np.mean(ref ** 2)) / np.sqrt(np.mean(v[:, :, cs] ** 2)))
        assert e <= TEMPORAL_REL
