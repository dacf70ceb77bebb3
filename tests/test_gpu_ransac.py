"""RANSAC plane fits against the oracle, bit for bit, over the forms of the
scoring loop (windows whole or not, of a width that is a multiple of the points
per lane or not, thresholds of 1 and others) and over matches whose 4-point
systems have equally large pivots, rows of zeros and exact zeros."""
import numpy as np
import pytest
import torch

import oracle
from tests import parity
from tests.test_gpu_parity import _need_gpu

pytestmark = pytest.mark.gpu


def _field(kind, W, H, rng):
    """Packed offsets of one direction."""
    y, x = np.mgrid[0:H, 0:W]
    if kind == "lattice":      # a translation: source and target coordinates equal up to a shift
        tx, ty = x + 3, y - 2
    elif kind == "mirror":     # few distinct targets, many of them collinear or coincident
        tx, ty = (W - 1 - x) // 4 * 4, y // 3 * 3
    elif kind == "wild":
        tx, ty = rng.integers(0, W, (H, W)), rng.integers(0, H, (H, W))
    else:                      # a plane with outliers
        w = 1 + 2e-4 * x - 1e-4 * y
        tx = np.floor((1.02 * x - 0.03 * y + 4) / w + 0.5).astype(int)
        ty = np.floor((0.03 * x + 0.98 * y - 3) / w + 0.5).astype(int)
        out = rng.random((H, W)) < 0.3
        tx, ty = np.where(out, rng.integers(0, W, (H, W)), tx), np.where(out, rng.integers(0, H, (H, W)), ty)
    return oracle.pack((np.clip(tx, 0, W - 1) - x).ravel(), (np.clip(ty, 0, H - 1) - y).ravel()).astype(np.int32)


@pytest.mark.parametrize("kind", ["plane", "lattice", "mirror", "wild"])
@pytest.mark.parametrize("W,H,blocks,tau,hyps", [
    (150, 110, (64, 16), 1.0, 256),     # 8 and 4 points of one row per lane
    (150, 110, (64, 16), 1.5, 300),     # another threshold; hypotheses in two batches
    (90, 71, (30, 13, 8), 1.0, 100),    # widths that are no multiple; windows of 64 points
    (20, 131, (128, 24), 1.0, 64),      # windows as wide as the frame: 20 and 20 columns
])
def test_ransac_equals_oracle(kind, W, H, blocks, tau, hyps):
    msgpm = _need_gpu()
    rng = np.random.default_rng(W + len(kind))
    f = rng.random((H, W, 3)).astype(np.float32)
    p = dict(C=3, r=1, grad_weight=0.0, blocks=blocks, iters=1, hyps=hyps, seed=9, tau=tau, m_min_abs=4, mu=0.01)
    o = oracle.Oracle(f, f, **p)
    g = msgpm.Pair(W, H, **p)
    g.set_features(f, f)
    nnf = [_field(kind, W, H, rng) for _ in range(2)]
    g.init_state(*nnf)
    for d in range(2):
        o.set_nnf(d, nnf[d])
        o.win[d][:] = np.where(rng.random(W * H) < 0.4, 0, -1)
        g.win(d).copy_(torch.from_numpy(o.win[d]).to(g.device))
    for level in range(len(blocks)):
        for stage in (1, 2):
            for d in range(2):
                o.ransac(d, level, stage)
            g.ransac(level, stage)
    got = g.planes()
    assert not parity.compare_planes(o, got)
    assert (got["hyp"] >= 0).any()
