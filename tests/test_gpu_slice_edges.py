"""Slice-in and slice-out where windows are no whole 64 x 64 tiles and no whole 16-byte pieces: odd maps and windows (one token per
lane), even ones (pairs), windows shorter than a tile, images of fewer than four positions, channels that end inside a tile --
windows against the unsliced run bit for bit, and the unsliced run against the float64 oracle."""
import numpy as np
import pytest

import oracle
import si_workloads as wl
from helpers import tiny_spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,heads,H,W,windows", [
    (96, 3, 1, 1, (1,)),              # one position
    (96, 3, 1, 2, (1,)),
    (160, 5, 1, 3, (1, 2)),
    (32, 1, 2, 2, (1, 3)),
    (96, 3, 5, 13, (1, 3, 16, 64)),   # 65 positions: a tile and one more; odd channel rows
    (160, 5, 7, 9, (4, 17, 32, 62)),  # a tile less one
    (96, 3, 10, 13, (6, 33, 65)),     # even map, even and odd windows
    (640, 10, 9, 15, (16, 45, 64)),
])
def test_block_windows(C, heads, H, W, windows):
    from gpu_helpers import errors, run_block
    spec = tiny_spec(wl.TEMPORAL, B=2, C=C, F=3, H=H, W=W, heads=heads, dim_head=C // heads, groups=32, dtype="bf16")
    x, w = wl.make_x(spec), wl.make_weights(spec, randomize_affine=True)
    whole = run_block(spec, x, w, None, H * W)
    e = errors(whole, oracle.block_forward_ref(x, w, spec, None), x)
    print(e)
    assert e["max_abs"] <= 2e-2 and e["rel_l2"] <= 5e-3
    for n in windows:
        assert np.array_equal(run_block(spec, x, w, None, n), whole), n


@pytest.mark.parametrize("kw,windows", [
    (dict(C=96, F=5, H=1, W=3), (1, 2)),
    (dict(C=160, F=4, H=5, W=13), (1, 3)),
    (dict(C=160, C_out=96, F=3, H=9, W=9, temb_dim=0), (1,)),
])
def test_resblock_windows(kw, windows):
    from gpu_helpers import errors, run_resblock
    spec = wl.scaled(wl.RES_CONFIGS["res1"], **kw)
    x, w, temb = wl.make_x(spec), wl.make_res_weights(spec, randomize_affine=True), wl.make_temb(spec)
    whole = run_resblock(spec, x, w, temb, spec.F)
    ref = oracle.resblock_forward_ref(x, w, spec, temb)
    e = errors(whole, ref, x if x.shape == ref.shape else np.zeros_like(ref))
    print(e)
    assert e["max_abs"] <= 2e-2 and e["rel_l2"] <= 5e-3
    for n in windows:
        assert np.array_equal(run_resblock(spec, x, w, temb, n), whole), n


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
    assert took[0] < 3.5 * took[1]  # 21 and 10 us; 49 before
