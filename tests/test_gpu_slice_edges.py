"""Slice-out of windows that are no whole 16-byte pieces: odd maps (one token per lane), even ones (pairs)."""
import numpy as np
import pytest

import si_workloads as wl
from helpers import tiny_spec

pytestmark = pytest.mark.gpu


def test_resblock_large_row_tiles():
    """Unsliced in tiles of 256 tokens x 160 channels, frame by frame in narrower ones, on a map of 35 x 37 positions."""
    from gpu_helpers import run_resblock
    spec = wl.scaled(wl.RES_CONFIGS["res1"], B=2, C=160, F=60, H=35, W=37, temb_dim=0)
    x, w = wl.make_x(spec), wl.make_res_weights(spec, randomize_affine=True)
    assert np.array_equal(run_resblock(spec, x, w, None, 60), run_resblock(spec, x, w, None, 7))


def test_odd_map_slice_out_is_not_serial():
    """A window of an odd map moves its residual one value at a time, but all of a block's values together: the projection that
    ends in it had taken 50 us where one of an even map takes 10."""
    import torch
    import paper_2411_01171_amd as si
    from paper_2411_01171_amd.devio import device_weights, to_dev
    took = []
    for H, W in ((31, 33), (32, 32)):
        spec = tiny_spec(wl.TEMPORAL, B=2, C=640, F=16, H=H, W=W, heads=8, dim_head=80, groups=32, dtype="bf16")
        x, bw = to_dev(wl.make_x(spec), "bf16"), device_weights(spec, wl.make_weights(spec))
        out = torch.empty_like(x)
        ws = torch.empty(si.si_workspace_bytes(x, bw, None, si.SI_AXIS_HW, 64), dtype=torch.uint8, device="cuda")
        for _ in range(2):
            si.si_block_forward(x, bw, None, out, si.SI_AXIS_HW, 64, ws)
        torch.cuda.synchronize()
        si.si_stage_timing_enable(True)
        try:
            si.si_stage_timing_read()
            for _ in range(5):
                si.si_block_forward(x, bw, None, out, si.SI_AXIS_HW, 64, ws)
            torch.cuda.synchronize()
            ms, n = si.si_stage_timing_read()["proj_out"]
        finally:
            si.si_stage_timing_enable(False)
        took.append(ms / n)
    print(took)
    assert took[0] < 2.5 * took[1]
