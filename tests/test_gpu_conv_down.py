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
