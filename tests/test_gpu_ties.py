"""Frames with many bit-equal patch costs (stripes, flat blocks, bars, repeated
tiles, in a few exact levels): every form of the whole pipeline must take the
candidates that a one-at-a-time loop takes, the first offered among equals, so
that single, graph, batched and served solves equal the sequence of phase calls
bit for bit."""
import numpy as np
import pytest
import torch

from tests.test_gpu_parity import _need_gpu
from tests.test_gpu_search import _state, _step_by_step

pytestmark = pytest.mark.gpu

W, H = 333, 210  # workgroups of 64 pixels, ragged
BASE = dict(C=5, r=4, blocks=(16,), iters=4, hyps=64, seed=11)


def _frames(kind):
    rng = np.random.default_rng(6)
    y, x = np.mgrid[0:H, 0:W]

    def frame(sx, sy):
        if kind == "stripes":
            v = (x + sx) // 6 % 3 * 0.5
        elif kind == "blocks":
            v = levels[(y + sy) // 12, (x + sx) // 12]
        elif kind == "tiles":
            v = levels[(y + sy) % 9, (x + sx) % 9]
        else:  # bars above and below a texture in levels of 1/8
            v = np.where((y < H // 4) | (y >= H - H // 4), 0.0, noise[y, x + sx])
        return np.repeat(v[..., None], 3, axis=2).astype(np.float32)

    levels = rng.integers(0, 4, (H // 12 + 2, W // 12 + 2)) / 4
    noise = rng.integers(0, 8, (H, W + 8)) / 8
    return frame(0, 0), frame(3, 2)


@pytest.mark.parametrize("kw", [dict(BASE, R0=16), dict(BASE), dict(BASE, r=2, C=3, grad_weight=0.0, fp16=True, R0=8)],
                         ids=["r4_R16", "r4", "r2_fp16_R8"])
@pytest.mark.parametrize("kind", ["stripes", "blocks", "bars", "tiles"])
def test_equal_costs_go_to_the_first_candidate(kind, kw):
    msgpm = _need_gpu()
    f1, f2 = _frames(kind)
    g = msgpm.Pair(W, H, **kw)
    ref = _state(g, *_step_by_step(msgpm, g, f1, f2))

    def same(form, pair, res):
        got = _state(pair, *res)
        for name in ref:
            assert np.array_equal(ref[name], got[name]), (form, name)

    for form in ("single", "repeated"):
        same(form, g, g.solve(f1, f2))
    a, b = (torch.as_tensor(f).cuda() for f in (f1, f2))
    same("graph", g, g.solve(a, b, graph=True))
    gs = [msgpm.Pair(W, H, **kw) for _ in range(2)]
    for pair, res in zip(gs, msgpm.Batch(gs).solve([f1, f1], [f2, f2])):
        same("batch", pair, res)
    srv = msgpm.Server(hbm_budget=1 << 34, max_active=2)
    tickets = [srv.submit(pair, f1, f2) for pair in gs]
    srv.step()
    for t in tickets:
        srv.wait(t, 60_000_000)
        pair, *res = srv.result(t)
        same("served", pair, res)
    srv.close()
