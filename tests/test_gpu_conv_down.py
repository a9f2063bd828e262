"""The stride-2 convolution that reads the feature in place (320-channel column tiles), where it can go wrong: maps of an odd
number of positions (the last group of four, of the last image above all), one output, ragged and whole 256-output tiles,
one and two column tiles, patches of one to three units per thread, the widest maps it takes and the first that it leaves
to the ring kernel -- against the float64 oracle."""
import numpy as np
import pytest

import oracle
from test_gpu_resample import _check, _inputs, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (1, 320, 1, 2, 2),          # four positions, one output
    (2, 320, 3, 5, 7),          # 35 positions: groups of four straddle every image's end
    (1, 320, 1, 1, 6),          # a single row
    (2, 320, 2, 9, 11),
    (1, 320, 1, 33, 37),        # 323 outputs: a second, ragged tile
    (1, 320, 2, 40, 128),       # whole tiles, rows of 64 outputs
    (1, 640, 1, 17, 30),        # two column tiles
    (1, 320, 1, 12, 176),       # three units per thread
    (1, 320, 1, 12, 230),       # wider than a patch
])
def test_against_oracle(shape):
    x, w, b = _inputs(*shape, seed=sum(shape), bias=shape[1] == 320)
    got = _run(x, w, b, "down", 1)
    _check(f"down {shape}", got, oracle.downsample_ref(x, w, b))
    if shape[2] > 1:
        assert np.array_equal(got, _run(x, w, b, "down", shape[2]))


@pytest.mark.parametrize("shape", [
    (1, 320, 9, 2, 2), (2, 320, 9, 5, 7), (1, 320, 9, 1, 6), (1, 320, 9, 33, 37), (1, 640, 9, 17, 30), (1, 320, 9, 12, 176),
    (1, 1280, 9, 9, 11),        # four column tiles
    (1, 960, 8, 24, 20),        # three; 128 x 64 tiles on the ring kernel
    (2, 320, 16, 40, 40),       # 128 x 160 tiles there: 12800 outputs
    (4, 640, 30, 32, 34),       # 256 x 160: 32640 outputs in half-empty tiles
])
def test_many_windows_and_one_agree(shape):
    """One window per frame runs on conv_down_kernel, an unsliced call of these sizes on the ring kernel, in the same order."""
    import torch
    import paper_2411_01171_amd as si
    x, w, b = _inputs(*shape, seed=sum(shape))
    xd = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    need = [si.si_resample_workspace_bytes(xd, si.SI_RESAMPLE_DOWN, n) for n in (1, shape[2])]
    assert need[0] == 18 * shape[1] ** 2 < need[1]
    got = _run(x, w, b, "down", 1)
    assert np.array_equal(got, _run(x, w, b, "down", shape[2]))
    last = slice(shape[2] - 1, shape[2])
    _check(f"down {shape}", got[:, :, last], oracle.downsample_ref(x[:, :, last], w, b))
