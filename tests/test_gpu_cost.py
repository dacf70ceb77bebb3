"""The cost refresh in its three modes (every pixel under the identity, the
unassigned pixels from the lists, the assigned pixels under their plane) against
the oracle, at frame sizes around the tiles and list runs of its workgroups;
pixels a mode does not select keep their cost."""
import numpy as np
import pytest

import oracle
from tests import parity
from tests.test_gpu_parity import _check_step, _gpu_params, _need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [dict(C=5, r=4), dict(C=5, r=3, fp16=True), dict(C=3, r=1, grad_weight=0.0)],
                         ids=["r4", "r3_fp16", "r1"])
@pytest.mark.parametrize("W,H", [(15, 7), (16, 8), (17, 9), (128, 2), (3, 130), (61, 45)])
@pytest.mark.parametrize("assigned", [0.0, 0.5, 1.0])
def test_cost_refresh(W, H, p, assigned):
    msgpm = _need_gpu()
    p = dict(p, blocks=(8,), iters=1, hyps=16, seed=4)
    rng = np.random.default_rng(W * H)
    f1, f2 = (rng.random((H, W, 3)).astype(np.float32) for _ in range(2))
    o = oracle.Oracle(f1, f2, **p)
    g = msgpm.Pair(W, H, **_gpu_params(p))
    g.set_features(f1, f2)
    n = len(o.pH)
    motion = np.eye(3) + rng.normal(size=(n, 3, 3)) * [[0.1, 0.1, 3], [0.1, 0.1, 3], [1e-4, 1e-4, 0]]
    motion[::7, 2] = [0, 0, -1]  # planes without a motion
    o.pH[:] = motion.reshape(n, 9)
    y, x = np.mgrid[0:H, 0:W]
    for d in range(2):
        o.set_nnf(d, oracle.pack((rng.integers(0, W, (H, W)) - x).ravel(), (rng.integers(0, H, (H, W)) - y).ravel()))
        label = rng.integers(0, n, W * H)
        o.win[d][:] = np.where(rng.random(W * H) < assigned, label, -1)
        o.hlabel[d][:] = np.where(rng.random(W * H) < 0.6, label, -1)
        o.cost[d][:] = -1.0  # no cost of a patch
    parity.push_state(o, g)
    report = {}
    for mode in (1, 0):
        o.run_step("eval_cost", (mode,))
        g.eval_cost(mode)
        got = parity.pull_state(g)
        _check_step("eval_cost", (mode,), o, got, None, p, report)
        if mode == 1:
            for d in range(2):
                assert np.array_equal(got["cost"][d] == -1, o.win[d] >= 0)
    for d in range(2):
        o.cost[d][:] = -1.0
    parity.push_state(o, g)
    g.finalize()
    for d in range(2):
        o.finalize(d)
    got = parity.pull_state(g)
    _check_step("eval_cost", (2,), o, got, None, p, report)
    for d in range(2):
        assert np.array_equal(got["cost"][d] == -1, o.win[d] < 0)
