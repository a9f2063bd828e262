"""fp32 temporal blocks: the one-kernel form and the staged kernels give the same bits, so that a call's result does not
depend on which of them its window length selects."""
import numpy as np
import pytest

import oracle
import si_workloads as wl
from helpers import tiny_spec

pytestmark = pytest.mark.gpu

BRANCH_REL = 1e-5  # six contractions of up to 1280 fp32 terms one after the other, 2e-6 each


# wider than 128 channels, frames that fill less than three quarters of the 16 or 32 token columns: windows of up to 4096
# tokens run in one kernel, the unsliced call (B F P above 4096 tokens) on the staged ones
@pytest.mark.parametrize("heads,d,F", [(3, 64, 9), (3, 64, 17), (5, 64, 10), (5, 32, 11), (4, 40, 23)])
def test_window_length_does_not_change_the_bits(heads, d, F):
    from gpu_helpers import errors, run_block
    D = heads * d
    spec = tiny_spec(wl.TEMPORAL, B=2, C=D, F=F, H=15, W=17, heads=heads, dim_head=d, groups=8, pe=F % 2 == 1, dtype="f32")
    x, w = wl.make_x(spec), wl.make_weights(spec, randomize_affine=True, matrix_std=0.05)
    assert 2 * F * 255 > 4096 >= 2 * F * 60
    full = run_block(spec, x, w, None, 255)
    for sl in (60, 7):
        assert np.array_equal(run_block(spec, x, w, None, sl), full)
    e = errors(full, oracle.block_forward_ref(x, w, spec), x)
    print(e)
    assert e["rel_l2_branch"] <= BRANCH_REL
