"""The fp32 temporal block in one kernel, at the edges of its tiles, vs the CPU oracle in fp64."""
import numpy as np
import pytest

import oracle
import si_workloads as wl
from helpers import tiny_spec

pytestmark = pytest.mark.gpu

# a dot product of n <= 1280 fp32 terms is off by about sqrt(n) * 2^-24 = 2e-6 of its size; six follow one another
BRANCH_REL = 1e-5


# frames: one, none that divide the 16 or 32 token columns, both full; widths: C != D, D of 16 .. 320, one wavefront's
# column tile only, contraction lengths that end inside a 64-wide chunk; 24 channels stay on the staged kernels
@pytest.mark.parametrize("F", [1, 5, 8, 16, 17, 32])
@pytest.mark.parametrize("C,heads,d", [(16, 2, 8), (64, 1, 64), (48, 2, 40), (96, 4, 8), (128, 2, 64), (24, 1, 16), (320, 5, 64)])
def test_temporal_f32(C, heads, d, F):
    from gpu_helpers import errors, run_block
    spec = tiny_spec(wl.TEMPORAL, B=2, C=C, F=F, H=3, W=7, heads=heads, dim_head=d, groups=8, pe=F % 2 == 1, dtype="f32")
    x, w = wl.make_x(spec), wl.make_weights(spec, randomize_affine=True, matrix_std=0.05)
    ref = oracle.block_forward_ref(x, w, spec)
    outs = [run_block(spec, x, w, None, sl) for sl in (4, 21)]
    assert np.array_equal(outs[0], outs[1])
    e = errors(outs[0], ref, x)
    print(e)
    assert np.all(np.isfinite(outs[0])) and e["rel_l2_branch"] <= BRANCH_REL
