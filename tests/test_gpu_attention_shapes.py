"""Attention at every head dimension class and at ragged lengths, through the block forward, vs the CPU oracle: spatial
self- and cross-attention, temporal attention of up to 32 frames."""
import numpy as np
import pytest

import oracle
import si_workloads as wl
from helpers import tiny_spec

pytestmark = pytest.mark.gpu

BF16_REL_L2, BRANCH_REL = 5e-3, 6e-3  # whole output; error of the branch (out - x) over its norm


def _check(spec, ctx, slice_len, wq_scale=1.0):
    from gpu_helpers import errors, run_block
    x = wl.make_x(spec)
    w = wl.make_weights(spec, randomize_affine=True, matrix_std=0.05)
    for k in ("wq", "wk", "wq2", "wk2"):
        if k in w:
            w[k] = wl.round_to_storage(w[k] * np.float32(wq_scale), "bf16")
    ref = oracle.block_forward_ref(x, w, spec, ctx)
    out = run_block(spec, x, w, ctx, slice_len)
    assert np.all(np.isfinite(out)), "output has NaN/Inf or unwritten elements"
    e = errors(out, ref, x)
    print(spec.heads, spec.dim_head, spec.H, spec.W, e)
    assert e["rel_l2"] <= BF16_REL_L2
    # largest element: half a bf16 ulp of the largest output, and six standard deviations of the branch's own
    # error (operand roundings: 4.4e-3 .. 5.7e-3 of the branch at these widths, the same as with fp32 attention)
    half_ulp = 2.0 ** (np.floor(np.log2(e["max_ref"])) - 8)
    assert e["max_abs"] <= half_ulp + 6 * BRANCH_REL * float(np.std(ref - x)), (half_ulp, float(np.std(ref - x)))


# head dimensions: one to sixteen 8-channel pieces, odd and even counts; D = 32 n runs on the ring GEMMs (attention output
# in fragment order), other widths on the row-major GEMM
@pytest.mark.parametrize("heads,d", [(8, 8), (4, 16), (3, 24), (4, 32), (4, 40), (2, 40), (4, 48), (2, 56), (4, 72), (2, 80), (2, 96), (2, 112), (1, 128)])
@pytest.mark.parametrize("hw,M", [((8, 8), 1), ((5, 13), 33), ((12, 16), 64)])
def test_spatial(heads, d, hw, M):
    spec = tiny_spec(wl.SPATIAL, B=2, C=64, F=3, H=hw[0], W=hw[1], heads=heads, dim_head=d, groups=8, M=M, Cc=16, dtype="bf16")
    _check(spec, wl.make_context(spec), 2)


# lengths around the 16-key tiles, 64-key chunks and 128-query tiles; up to 32 positions run on the short kernel
@pytest.mark.parametrize("P", [1, 31, 33, 63, 65, 97, 127, 129, 191, 225])
@pytest.mark.parametrize("heads,d", [(4, 40), (2, 80)])
def test_spatial_ragged_lengths(P, heads, d):
    spec = tiny_spec(wl.SPATIAL, B=1, C=64, F=2, H=1, W=P, heads=heads, dim_head=d, groups=8, M=P % 50 + 1, Cc=16, dtype="bf16")
    _check(spec, wl.make_context(spec), 1, wq_scale=3.0)  # sharpened scores: the running maximum moves between chunks


@pytest.mark.parametrize("heads,d", [(8, 8), (4, 32), (2, 40), (4, 40), (2, 56), (2, 64), (2, 80), (2, 96), (1, 112), (2, 128)])
@pytest.mark.parametrize("F", [1, 7, 32])
def test_temporal(heads, d, F):
    """5 x 7 positions in windows of 10: sequences that fill no workgroup, a ragged last window."""
    spec = tiny_spec(wl.TEMPORAL, B=2, C=96, F=F, H=5, W=7, heads=heads, dim_head=d, groups=8, pe=True, dtype="bf16")
    _check(spec, None, 10, wq_scale=2.0)


@pytest.mark.parametrize("heads,d,hw,M", [(1, 40, (64, 64), 77), (2, 80, (48, 50), 200)])
def test_spatial_long(heads, d, hw, M):
    """Thousands of keys, tens of 64-key chunks, with scores sharp enough that the running maximum keeps moving."""
    spec = tiny_spec(wl.SPATIAL, B=1, C=64, F=1, H=hw[0], W=hw[1], heads=heads, dim_head=d, groups=8, M=M, Cc=16, dtype="bf16")
    _check(spec, wl.make_context(spec), 1, wq_scale=3.0)


@pytest.mark.parametrize("heads,d", [(2, 40), (2, 64), (1, 128)])
@pytest.mark.parametrize("F", [33, 64, 65, 130])
def test_temporal_long(heads, d, F):
    """Sequences past the short kernel: one 64-key chunk, several, a last one of one and of two keys."""
    spec = tiny_spec(wl.TEMPORAL, B=1, C=96, F=F, H=3, W=5, heads=heads, dim_head=d, groups=8, pe=True, dtype="bf16")
    _check(spec, None, 4, wq_scale=2.0)
