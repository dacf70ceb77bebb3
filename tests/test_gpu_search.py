"""The pipeline's PatchMatch passes (candidates dropped by memory and by moment
bounds) against the same half-sweeps called one by one, which evaluate every
candidate: whole solves and the sequence of phase calls they stand for must
leave the same offsets, costs, assignments, planes and outputs, bit for bit."""
import numpy as np
import pytest
import torch

from paper_1804_03787_amd import synth
from tests.test_gpu_parity import _need_gpu

pytestmark = pytest.mark.gpu


def _step_by_step(msgpm, g, f1, f2):
    """msgpm_solve's sequence through the phase entry points."""
    p = g.p

    def sweeps(slot, restricted):
        if p.pm_iters == 0:
            g.eval_cost(restricted)
        for it in range(p.pm_iters):
            for colour in range(2):
                g.pm_halfsweep(colour, it, slot, restricted | (msgpm.PM_FRESH if it == 0 else 0))

    g.set_features(f1, f2)
    g.init_state()
    sweeps(0, 0)
    for level in range(p.n_levels):
        for stage in (1, 2):
            g.ransac(level, stage)
            g.assign(level, stage, True)
            g.symmetry(level, stage)
            g.assign(level, stage, False)
        g.fb_unassign()
        if p.flags & msgpm.FLAG_CUE_UNIQUE:
            g.unique()
        g.nnf_update(level)
        sweeps(level + 1, 1)
    if p.fill_sweeps:
        g.fill()
    return g.finalize()


def _state(g, flows, occs):
    torch.cuda.synchronize()
    s = {"planes": g.planes().view(np.uint8)}
    for d in range(2):
        s[f"flow{d}"] = flows[d].cpu().numpy().view(np.uint32)
        s[f"occ{d}"] = occs[d].cpu().numpy()
        for name in ("nnf", "cost", "win", "loss", "hlabel"):
            a = getattr(g, name)(d).cpu().numpy()
            s[f"{name}{d}"] = a.view(np.uint64 if a.dtype == np.float64 else np.uint32)
    return s


def _frames(W, H, seed, kind):
    pr = synth.planar_pair(W, H, seed=seed, scale=max(W, H) / 1024, n_quads=8)
    f1, f2 = pr.frame1.copy(), pr.frame2.copy()
    if kind == "u8":          # 8-bit values: equal costs are common
        f1, f2 = (np.round(np.clip(f, 0, 1) * 31).astype(np.float32) / 31 for f in (f1, f2))
    elif kind == "0..255":
        f1, f2 = f1 * np.float32(255), f2 * np.float32(255)
    elif kind == "offset":    # little contrast on a large level
        f1, f2 = (np.float32(1000) + np.float32(0.25) * f for f in (f1, f2))
    elif kind == "flat":      # one colour, but for a few pixels far outside the range
        f1, f2 = (np.full_like(f, 0.5) for f in (f1, f2))
        f1[H // 3, W // 4], f2[H // 2, W // 2], f2[1, 1] = 9.0, 9.0, -1e20
    elif kind == "tiny":
        f1, f2 = f1 * np.float32(1e-12), f2 * np.float32(1e-12)
    elif kind == "spots":     # outliers, infinities and NaN in both frames
        rng = np.random.default_rng(seed)
        for f in (f1, f2):
            for v in (1e8, -1e8, 1e18, np.inf, -np.inf, np.nan):
                for _ in range(3):
                    f[rng.integers(H), rng.integers(W), rng.integers(3)] = v
    return f1, f2


BASE = dict(C=5, r=4, blocks=(16,), iters=3, hyps=64, seed=3)


@pytest.mark.parametrize("W,H,kw,kind", [
    (9, 7, dict(BASE, blocks=(8,)), "plain"),              # smaller than a tile and a patch
    (16, 8, dict(BASE, r=1, C=3, grad_weight=0.0, blocks=(8,)), "plain"),  # one tile
    (17, 9, dict(BASE, r=2, blocks=(8,)), "plain"),        # one pixel more, odd
    (129, 97, dict(BASE, iters=1), "plain"),               # first half-sweeps that are the last
    (130, 63, dict(BASE, iters=2, fp16=True), "u8"),
    (161, 99, dict(BASE, r=3, blocks=(32, 16)), "u8"),
    (128, 96, dict(BASE, R0=1), "u8"),                     # one radius; every draw within the tried positions
    (128, 96, dict(BASE, R0=32767), "plain"),              # fifteen radii
    (320, 210, dict(BASE, iters=5, blocks=(32, 16), cue_overlap=True, cue_unique=True, fill_sweeps=8), "plain"),
    (513, 380, dict(BASE, iters=4, blocks=(64, 16)), "plain"),          # tiles of 64 pixels, ragged
    (513, 380, dict(BASE, iters=4, r=3, C=3, grad_weight=0.0, fp16=True, blocks=(64, 16)), "u8"),
    (96, 72, dict(BASE), "0..255"),
    (96, 72, dict(BASE, grad_weight=0.0), "offset"),
    (96, 72, dict(BASE), "flat"),
    (96, 72, dict(BASE), "tiny"),
    (96, 72, dict(BASE), "spots"),
    (96, 72, dict(BASE, r=2, C=3, grad_weight=0.0, fp16=True), "spots"),
])
def test_passes_equal_single_half_sweeps(W, H, kw, kind):
    msgpm = _need_gpu()
    f1, f2 = _frames(W, H, 5, kind)
    a, b = msgpm.Pair(W, H, **kw), msgpm.Pair(W, H, **kw)
    b.ws.fill_(0x5a)  # whatever an earlier use left there
    ref = _state(a, *_step_by_step(msgpm, a, f1, f2))
    got = _state(b, *b.solve(f1, f2))
    for name in ref:
        assert np.array_equal(ref[name], got[name]), name
