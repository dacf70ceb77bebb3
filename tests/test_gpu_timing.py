"""What the kernel timing books where: the launches of a solve per kind follow
from its parameters, and the features kind holds the features alone."""
import pytest

from paper_1804_03787_amd import synth
from tests.test_gpu_parity import _need_gpu

pytestmark = pytest.mark.gpu

W, H = 96, 72


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("blocks,iters,histeq", [((), 2, False), ((16,), 3, False), ((32, 16), 2, True), ((16,), 0, False)])
def test_launches_per_kind(blocks, iters, histeq, batched):
    msgpm = _need_gpu()
    pr = synth.planar_pair(W, H, seed=1, scale=0.1)
    g = msgpm.Pair(W, H, C=3, r=1, grad_weight=0.0, blocks=blocks, iters=iters, hyps=16, seed=2, histeq=histeq)
    msgpm.timing_enable(True)
    try:
        msgpm.timing_read()
        if batched:
            msgpm.Batch([g]).solve([pr.frame1], [pr.frame2])
        else:
            g.solve(pr.frame1, pr.frame2)
        n = {k: v[1] for k, v in msgpm.timing_read().items()}
    finally:
        msgpm.timing_enable(False)
    levels, passes = len(blocks), (1 + len(blocks)) * (iters > 0)
    # histogram equalisation: one timed group of launches, or three steps of a batch
    assert n["features"] == 1 + histeq * (3 if batched else 1)
    assert n["pm_list"] == levels + passes      # pixel lists, patch moments
    assert n["pm_init"] == 2 * iters
    assert n["pm_restricted"] == 2 * iters * levels
    assert n["pm_restricted_ident"] == (0 if batched else 2 * iters * levels)
    assert n["ransac"] == n["symmetry"] == 2 * levels and n["assign"] == 4 * levels
