"""The 3x3 convolution kernel that keeps a patch of source tokens in LDS, where it can go wrong: tiles that straddle
images and end inside the last one, odd maps (no 32-token blocks), the widest maps it takes (ten to twelve 64-token
blocks per patch), one channel chunk and several, one column tile and two, doubled maps -- against the float64 oracle."""
import numpy as np
import pytest

import oracle
import si_workloads as wl
from test_gpu_resample import _check as check_resample, _inputs, _run
from test_gpu_resblock import _check as check_resblock

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,c_out", [
    ((1, 32, 1, 145, 255), 160),   # widest map, ragged last tile, a single channel chunk, then several
    ((4, 32, 1, 96, 99), 160),     # four images, tiles straddle them
])
def test_same_map(shape, c_out):
    from gpu_helpers import run_resblock
    B, C, F, H, W = shape
    spec = wl.scaled(wl.RES_CONFIGS["res1"], B=B, C=C, F=F, H=H, W=W, C_out=c_out)
    x, temb = wl.make_x(spec), wl.make_temb(spec)
    w = wl.make_res_weights(spec, randomize_affine=True)
    check_resblock(f"halo {shape} -> {c_out}", run_resblock(spec, x, w, temb, F),
                   oracle.resblock_forward_ref(x, w, spec, temb), x)


@pytest.mark.parametrize("shape", [
    (1, 160, 1, 73, 130),
    (4, 160, 1, 49, 49),
    (1, 160, 1, 41, 200),          # ten 64-token blocks per patch
    (1, 160, 1, 34, 240),          # twelve
    (1, 320, 1, 46, 90),           # two column tiles
])
def test_doubled_map(shape):
    x, w, b = _inputs(*shape, seed=sum(shape))
    check_resample(f"halo up {shape}", _run(x, w, b, "up", 1), oracle.upsample_ref(x, w, b))


def test_sliced_equals_unsliced_on_device():
    """The kernel is chosen by one frame's size, so every slicing gives the same bits."""
    from gpu_helpers import run_resblock
    spec = wl.scaled(wl.RES_CONFIGS["res1"], B=1, C=160, F=9, H=108, W=171)
    x, w, temb = wl.make_x(spec), wl.make_res_weights(spec), wl.make_temb(spec)
    full = run_resblock(spec, x, w, temb, 9)
    for sl in (1, 2):
        assert np.array_equal(run_resblock(spec, x, w, temb, sl), full)
