"""Staged blocks at every register width of the small windows' LayerNorm (one to eight times 256 channels, rows that end inside
their last 256), with windows at aligned positions (whole tiles of the slice-in, 16-byte slice-out) and at ragged ones."""
import numpy as np
import pytest

import oracle
import si_workloads as wl
from helpers import tiny_spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [96, 288, 544, 800, 1056, 1312, 1568, 2048])
def test_widths_and_alignments(D):
    from gpu_helpers import errors, run_block
    spec = tiny_spec(wl.TEMPORAL, B=1, C=D, F=4, H=9, W=16, heads=D // 32, dim_head=32, groups=32, dtype="bf16", pe=True)
    x, w = wl.make_x(spec), wl.make_weights(spec, randomize_affine=True)
    a, b = run_block(spec, x, w, None, 64), run_block(spec, x, w, None, 60)
    assert np.array_equal(a, b)
    ref = oracle.block_forward_ref(x, w, spec, None)
    e = errors(a, ref, x)
    # A value is off by its own last rounding, half a bf16 step at the largest value's exponent, and by the branch's error before
    # it.  A bf16 rounding is off by at most 2^-8 of the value, about 2^-9 rms over a binade; a contraction keeps the relative rms
    # of its operands' independent errors; four roundings in series (LayerNorm, attention, GEGLU, residual copy) add in
    # quadrature to 2^-8 rms of the branch.  Of up to 1.2e6 such values none lies beyond 6 deviations (2e-9 each).
    bound = 2.0 ** (np.floor(np.log2(np.abs(ref).max())) - 8) + 6 * 2.0 ** -8 * np.sqrt(np.mean((ref - x) ** 2))
    print(e, "bound", bound)
    assert e["max_abs"] <= bound and e["rel_l2"] <= 5e-3


@pytest.mark.parametrize("C,D,heads", [(640, 640, 10), (1280, 1280, 20)])
def test_windows_of_many_rows_agree(C, D, heads):
    """Windows of 16384 and of 8192 rows give the bits of windows of 1024."""
    from gpu_helpers import run_block
    spec = tiny_spec(wl.TEMPORAL, B=1, C=C, F=16, H=32, W=32, heads=heads, dim_head=D // heads, groups=32, dtype="bf16")
    x, w = wl.make_x(spec), wl.make_weights(spec, randomize_affine=True)
    a = run_block(spec, x, w, None, 64)
    assert np.array_equal(run_block(spec, x, w, None, 512), a) and np.array_equal(run_block(spec, x, w, None, 1024), a)
