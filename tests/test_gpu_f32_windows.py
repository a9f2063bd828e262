"""fp32 temporal blocks: the one-kernel form and the staged kernels give the same bits, so that a call's result does not
depend on which of them its window length selects."""
import numpy as np
import pytest

import oracle
import si_workloads as wl
from helpers import tiny_spec

pytestmark = pytest.mark.gpu

BRANCH_REL = 1e-5  # six contractions of up to 1280 fp32 terms one after the other, 2e-6 each


def _run(spec, x, w, slice_len):
    """The output and the names of the stages that ran."""
    import paper_2411_01171_amd as si
    from gpu_helpers import run_block
    si.si_stage_timing_read()
    si.si_stage_timing_enable(True)
    try:
        out = run_block(spec, x, w, None, slice_len)
    finally:
        si.si_stage_timing_enable(False)
    return out, {name for name, (_, launches) in si.si_stage_timing_read().items() if launches}


# windows of 60 positions run in one kernel, the unsliced call (18000 .. 36000 token columns) on the staged kernels
@pytest.mark.parametrize("heads,d,F", [(3, 64, 9), (3, 64, 17), (5, 64, 10), (5, 64, 16), (5, 32, 11), (4, 40, 23)])
def test_window_length_does_not_change_the_bits(heads, d, F):
    from gpu_helpers import errors
    D = heads * d
    spec = tiny_spec(wl.TEMPORAL, B=2, C=D, F=F, H=33, W=17, heads=heads, dim_head=d, groups=8, pe=F % 2 == 1, dtype="f32")
    x, w = wl.make_x(spec), wl.make_weights(spec, randomize_affine=True, matrix_std=0.05)
    full, stages = _run(spec, x, w, 561)
    assert "temporal_block_f32" not in stages and "ff2" in stages
    for sl in (60, 7):
        part, stages = _run(spec, x, w, sl)
        assert "temporal_block_f32" in stages and "ff2" not in stages
        assert np.array_equal(part, full)
    e = errors(full, oracle.block_forward_ref(x, w, spec), x)
    print(e)
    assert e["rel_l2_branch"] <= BRANCH_REL


def test_more_sequences_than_one_launch_holds():
    """9 frames leave room for one sequence per workgroup: 2^23 + 4096 positions are 2^32 threads and more, five launches.  The map is a
    1024-position one repeated, whose GroupNorm statistics it shares up to their fp32 rounding."""
    import torch
    import paper_2411_01171_amd as si
    from gpu_helpers import AXIS, device_weights, to_dev
    spec = tiny_spec(wl.TEMPORAL, B=1, C=16, F=9, H=1, W=1024, heads=2, dim_head=8, groups=8, dtype="f32")
    small, w = wl.make_x(spec), wl.make_weights(spec, randomize_affine=True, matrix_std=0.05)
    wd = device_weights(spec, w)

    def run(x):
        n = si.si_workspace_bytes(x, wd, None, AXIS[spec.slice_axis], 1024)
        assert n > 0
        out = torch.full_like(x, float("nan"))
        si.si_block_forward(x, wd, None, out, AXIS[spec.slice_axis], 1024, torch.empty(n, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        return out

    xs = to_dev(small, "f32")
    reps = (1 << 23) // 1024 + 4
    ref, got = run(xs), run(xs.repeat(1, 1, 1, 1, reps).view(1, 16, 9, reps, 1024).contiguous())
    diff = (got - ref).abs().amax(dim=(0, 1, 2, 4))  # per repetition
    # a mean or variance off by one fp32 rounding moves a normalised value by 1e-7 of its size, six contractions widen that
    assert bool(torch.isfinite(diff).all()) and float(diff.max()) <= 1e-5 * float(ref.abs().max())
