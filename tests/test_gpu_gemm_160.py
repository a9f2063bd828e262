"""Staged GEMMs in tiles of 160 and 320 columns: long windows run on them, short ones on the ring kernel, and both sum in the
same order, so a call's bits do not depend on its windows -- at ragged token counts (tiles that end inside the last row
block), contractions of 5 .. 40 stages, every epilogue (residual with and without its fp16 copy, q / k / v with transposed
values, GEGLU, slice-out)."""
import numpy as np
import pytest

import oracle
import si_workloads as wl
from helpers import tiny_spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,kw,long,short,against_oracle", [
    (wl.TEMPORAL, dict(B=1, C=640, F=14, H=45, W=10, heads=8, dim_head=80, pe=True), 450, 60, True),    # 6300 tokens
    (wl.SPATIAL, dict(B=1, C=640, F=7, H=33, W=32, heads=10, dim_head=64, M=77, Cc=64), 7, 1, False),  # 7392 tokens
    (wl.SPATIAL, dict(B=1, C=320, F=12, H=39, W=40, heads=8, dim_head=40, M=5, Cc=64), 12, 6, False),  # 18720 tokens, K = 320
    (wl.TEMPORAL, dict(B=1, C=1280, F=16, H=9, W=15, heads=20, dim_head=64), 135, 16, False),           # 2160 tokens
])
def test_long_and_short_windows_agree(kind, kw, long, short, against_oracle):
    from gpu_helpers import errors, run_block
    spec = tiny_spec(kind, groups=32, dtype="bf16", **kw)
    x, w, c = wl.make_x(spec), wl.make_weights(spec, randomize_affine=True), wl.make_context(spec)
    a, b = run_block(spec, x, w, c, long), run_block(spec, x, w, c, short)
    assert np.all(np.isfinite(a)) and np.array_equal(a, b)
    if against_oracle:
        e = errors(a, oracle.block_forward_ref(x, w, spec, c), x)
        print(e)
        assert e["max_abs"] <= 2e-2 and e["rel_l2"] <= 5e-3


@pytest.mark.parametrize("C", [64, 128])
def test_fewer_stages_than_slots(C):
    """proj_in over 64 and 128 channels: one and two stages for three slots.  Windows of 8064 tokens, two in flight, run in tiles of
    160 columns, those of 1024 on the ring kernel (from 8192 tokens the LayerNorm sums in another order)."""
    from gpu_helpers import run_block
    spec = tiny_spec(wl.TEMPORAL, B=1, C=C, F=16, H=64, W=64, heads=5, dim_head=64, groups=32, dtype="bf16")
    x, w = wl.make_x(spec), wl.make_weights(spec, randomize_affine=True)
    a, b = run_block(spec, x, w, None, 504), run_block(spec, x, w, None, 64)
    assert np.all(np.isfinite(a)) and np.array_equal(a, b)
