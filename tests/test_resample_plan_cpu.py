"""Which kernel a DownSample takes, read off the workspace (conv_down_kernel has no operand buffer): many windows run on it, in
one launch; small unsliced calls and calls of few windows, where most of its 256-output tiles would be empty, do not; nor do
more tiles than one launch may have."""
import ctypes as C

import pytest


def _bytes(shape, slice_len):
    from paper_2411_01171_amd import binding as B
    x = B._Tensor5(0x1000, B.SI_BF16, *shape)
    return B.lib().si_resample_workspace_bytes(C.byref(x), B.SI_RESAMPLE_DOWN, slice_len)


def _weights(channels):
    return 9 * channels * channels * 2  # the re-laid-out kernel, a multiple of 256 bytes for multiples of 320 channels


@pytest.mark.parametrize("shape,slice_len,in_one_launch", [
    ((2, 1280, 25, 8, 8), 25, False),     # 16 of 256 outputs per tile
    ((2, 1280, 25, 8, 8), 1, True),
    ((2, 1280, 6, 18, 32), 4, False),
    ((1, 320, 1, 64, 64), 1, False),      # four tiles on 256 CUs
    ((2, 640, 25, 9, 11), 25, False),
    ((2, 320, 25, 72, 128), 1, True),
    ((2, 320, 25, 72, 128), 25, True),    # 450 full tiles
    ((2, 256, 25, 72, 128), 1, False),    # no 320-channel tiles
    ((1, 320, 12, 12, 230), 1, False),    # wider than a patch
])
def test_kernel_by_size(shape, slice_len, in_one_launch):
    assert (_bytes(shape, slice_len) == _weights(shape[1])) == in_one_launch


def test_launch_limit():
    """129 x 65535 workgroups of 512 threads would be more than the 2^32 threads that a launch may have."""
    assert _bytes((129, 320, 65535, 2, 2), 1) > _weights(320)
