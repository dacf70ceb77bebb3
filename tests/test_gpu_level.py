"""Frames of little contrast on a large level, where the FP32 rounding of the
bilinear samples is as large as the differences between patches: the passes of
the whole pipeline must still accept what the single half-sweeps, which evaluate
every candidate, accept, bit for bit."""
import functools

import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_parity import _need_gpu
from tests.test_gpu_search import _state, _step_by_step

pytestmark = pytest.mark.gpu

W, H, BLOCK = 192, 144, 24


def _scene(level, ulps, contrast):
    """Flat blocks, their values `ulps` steps of the level's FP32 spacing (or of
    `contrast`), in frame 2 distorted by a homography and off by a step here and
    there, so that pixels with a region plane stay unassigned; the homography's
    offsets as initial NNF."""
    rng = np.random.default_rng(3)
    step = float(contrast / ulps if contrast else np.spacing(np.float32(abs(level))))
    y, x = np.mgrid[0:H, 0:W]
    A = np.array([[1.04, 0.02, -3.3], [-0.015, 1.04, -2.1], [1e-5, -2e-5, 1]])
    value = rng.integers(0, ulps, (H // BLOCK + 4, W // BLOCK + 4, 3))
    off = rng.integers(-1, 2, value.shape) * (rng.random(value.shape[:2])[..., None] < 0.5)

    def project(M):
        w = M[2, 0] * x + M[2, 1] * y + M[2, 2]
        return (M[0, 0] * x + M[0, 1] * y + M[0, 2]) / w, (M[1, 0] * x + M[1, 1] * y + M[1, 2]) / w

    def at(px, py):
        by, bx = (py // BLOCK).astype(int) + 1, (px // BLOCK).astype(int) + 1
        return value[np.clip(by, 0, value.shape[0] - 1), np.clip(bx, 0, value.shape[1] - 1)]

    frames = [at(x, y), at(*project(np.linalg.inv(A))) + off[y // BLOCK, x // BLOCK]]
    init = []
    for M in (A, np.linalg.inv(A)):
        qx, qy = project(M)
        tx, ty = (np.clip(np.floor(q + 0.5), 0, n - 1).astype(int) for q, n in ((qx, W), (qy, H)))
        init.append(torch.from_numpy(oracle.pack((tx - x).ravel(), (ty - y).ravel()).astype(np.int32)))
    return [(level + step * f).astype(np.float32) for f in frames], init, step


@pytest.mark.parametrize("level,ulps,contrast", [(1.0, 4, 0), (1000.0, 2, 0), (1000.0, 4, 0), (-1000.0, 4, 0),
                                                 (200.0, 4, 0), (1000.0, 4, 0.01), (0.5, 4, 0.4)])
@pytest.mark.parametrize("kw", [dict(C=5, r=4), dict(C=3, r=2), dict(C=3, r=1)], ids=["r4", "r2", "r1"])
def test_little_contrast_on_a_large_level(level, ulps, contrast, kw):
    msgpm = _need_gpu()
    frames, init, step = _scene(level, ulps, contrast)
    kw = dict(kw, blocks=(32, 16), iters=4, hyps=128, seed=7, grad_weight=0.0, eps=0.5 * step, R0=64)
    a, b = msgpm.Pair(W, H, **kw), msgpm.Pair(W, H, **kw)
    a.init_state = functools.partial(a.init_state, *init)
    ref = _state(a, *_step_by_step(msgpm, a, *frames))
    got = _state(b, *b.solve(*frames, *init))
    assert min(b.counters()["pm_restricted"]) > 100000  # distorted patches were searched
    for name in ref:
        assert np.array_equal(ref[name], got[name]), name
