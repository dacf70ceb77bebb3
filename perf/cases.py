"""Performance cases: the frame-pair solves and the phases of them that users of this library run.

`listed()` holds the cases, `draw(rng)` makes further ones of the same ranges, `prepare` makes a case's inputs and the
objects a program keeps, `run` is one pass through the public Python entry points, `work` says what a pass cannot do
without, and `exact` gives the outputs in FP64 where they are a plain function of the inputs.

Inputs are piecewise-planar scenes made on the GPU: blurred-noise textures on a background and on convex quads, each
moving by a similarity with a slight perspective, a global gain between the frames, optionally quantised to 8 bits as
decoded video frames are.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1804_03787_amd import msgpm

DEV = "cuda"
BATCH_SIZES = ((320, 240), (640, 360), (1024, 436), (1280, 544), (317, 241), (641, 359))
SERVE_SIZES = ((1024, 436), (640, 360), (1024, 436), (641, 359))
MASK32 = 0xFFFFFFFF


def _case(kind, W, H, **kw):
    """kind: solve (one pair; graph: as one HIP graph launch), batch / serve (n pairs of uneven sizes together,
    through the batched graph or the server), sweep (one half-sweep of the search over every pixel), restricted (one half-sweep
    over the unassigned pixels, patches distorted by planes), planes (the two plane stages of one level, its
    forward-backward check and its NNF update), finalize (final costs, flow and masks)."""
    c = dict(kind=kind, W=W, H=H, n=1, C=5, r=4, blocks="64,32,16", iters=8, hyps=256, fp16=False, graph=False,
             cues=False, fill=0, histeq=False, strict=False, u8=False)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call, one frame pair of the smoke test's size: launches and host work count
        dict(_case("solve", 128, 96, r=3, blocks="16", iters=4, hyps=64), name="tiny solve"),
        # the paper's preset: 7x7 RGB patches, windows of 81 and 41, an odd-sized 8-bit pair, plain launches
        dict(_case("solve", 639, 357, r=3, C=3, blocks="81,41", u8=True), name="paper preset"),
        # the default workload, one graph launch per pair, in both storage forms
        dict(_case("solve", 1024, 436, graph=True), name="1024x436"),
        dict(_case("solve", 1024, 436, graph=True, fp16=True), name="1024x436 fp16"),
        # every option of the method on an 8-bit pair whose exposure changes
        dict(_case("solve", 641, 479, cues=True, fill=64, histeq=True, strict=True, u8=True), name="options"),
        # the largest frames served, with a fourth window level
        dict(_case("solve", 2048, 872, graph=True, fp16=True, blocks="128,64,32,16"), name="2048x872 fp16"),
        # pairs of uneven sizes solved together
        dict(_case("batch", 0, 0, n=6, graph=True, fp16=True), name="batch"),
        # a burst of requests to the server
        dict(_case("serve", 0, 0, n=4, fp16=True), name="serve"),
        # single phases, as a program that steps through the method calls them
        dict(_case("sweep", 1024, 436), name="sweep"),
        dict(_case("restricted", 767, 431, r=3, fp16=True), name="restricted sweep"),
        dict(_case("planes", 1024, 436), name="plane level"),
        dict(_case("finalize", 1280, 544), name="finalize"),
    ]


def draw(rng):
    kind = rng.choice(["solve"] * 5 + ["batch", "serve", "sweep", "restricted", "planes", "finalize"])
    W = int(round(math.exp(rng.uniform(math.log(64), math.log(1280)))))
    H = max(48, int(round(W * rng.uniform(0.4, 0.9))))
    H = min(H, 696320 // W)
    c = _case(kind, W, H, C=rng.choice([3, 5, 5]), r=rng.choice([1, 2, 3, 4, 4]),
              blocks=rng.choice(["64,32,16", "64,32,16", "32,16", "81,41", "16"]), iters=rng.randint(3, 8),
              hyps=rng.choice([64, 128, 256, 256, 300]), fp16=rng.random() < 0.5, u8=rng.random() < 0.5)
    if kind == "solve":
        c.update(graph=rng.random() < 0.5, cues=rng.random() < 0.25, fill=rng.choice([0, 0, 0, 16]),
                 histeq=rng.random() < 0.25, strict=rng.random() < 0.25)
    elif kind in ("batch", "serve"):
        c.update(W=0, H=0, n=rng.randint(2, 4), graph=kind == "batch", iters=rng.randint(3, 5))
    return c


# ---- inputs ------------------------------------------------------------------------------------------------------

def _blur(t):
    """Gaussian blur, sigma 2, of an (h, w, 3) canvas, cropped by 8 on every side."""
    k = [math.exp(-d * d / 8.0) for d in range(-8, 9)]
    h, w, _ = t.shape
    t = sum(k[i] * t[i:h - 16 + i] for i in range(17))
    return sum(k[i] * t[:, i:w - 16 + i] for i in range(17))


def _similarity(cx, cy, scale, deg, tx, ty, p0=0.0, p1=0.0):
    a = math.radians(deg)
    to = np.array([[1, 0, cx + tx], [0, 1, cy + ty], [0, 0, 1.0]])
    back = np.array([[1, 0, -cx], [0, 1, -cy], [0, 0, 1.0]])
    return to @ np.array([[scale * math.cos(a), -scale * math.sin(a), 0],
                          [scale * math.sin(a), scale * math.cos(a), 0], [p0, p1, 1.0]]) @ back


def _map(Hm, x, y):
    w = Hm[2, 0] * x + Hm[2, 1] * y + Hm[2, 2]
    return (Hm[0, 0] * x + Hm[0, 1] * y + Hm[0, 2]) / w, (Hm[1, 0] * x + Hm[1, 1] * y + Hm[1, 2]) / w


def _scene(W, H, seed, u8=False):
    """(frame1, frame2, layers, flow0, flow1): HWC float32 frames, the layers' homographies and the layers' motion at
    every pixel, frame 1 to 2 and back (FP64)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    rng = np.random.default_rng(seed)
    s = max(0.12, W / 1024)
    pad = int(160 * s) + 16
    tex = _blur(torch.randn((H + 2 * pad + 16, W + 2 * pad + 16, 3), device=DEV, generator=g))
    lo, hi = tex.amin((0, 1)), tex.amax((0, 1))
    tex = (tex - lo) / (hi - lo)
    th, tw, _ = tex.shape

    cam = _similarity(W / 2, H / 2, rng.uniform(0.96, 1.04), rng.uniform(-4, 4), *(rng.uniform(-30, 30, 2) * s),
                      *rng.uniform(-2e-5, 2e-5, 2))
    layers = [(cam, None, (0, 0))]
    for _ in range(20):
        cx, cy, rad = rng.uniform(0, W), rng.uniform(0, H), rng.uniform(30, 140) * s
        ang = [(k + rng.uniform(0.2, 0.8)) * math.pi / 2 for k in range(4)]
        poly = [(cx + rad * math.cos(a), cy + rad * math.sin(a)) for a in ang]
        rel = _similarity(cx, cy, rng.uniform(0.97, 1.03), rng.uniform(-3, 3), *(rng.uniform(-16, 16, 2) * s))
        layers.append((cam @ rel, poly, (int(rng.integers(th)), int(rng.integers(tw)))))

    ys, xs = torch.meshgrid(torch.arange(H, device=DEV, dtype=torch.float64),
                            torch.arange(W, device=DEV, dtype=torch.float64), indexing="ij")

    def inside(poly, x, y):
        ok = torch.ones_like(x, dtype=torch.bool)
        if poly is not None:
            for (ax, ay), (bx, by) in zip(poly, poly[1:] + poly[:1]):
                ok &= (bx - ax) * (y - ay) - (by - ay) * (x - ax) >= 0
        return ok

    def sample(x, y, shift):
        u = (x + pad + shift[1]) % (tw - 1)
        v = (y + pad + shift[0]) % (th - 1)
        u0, v0 = u.floor(), v.floor()
        fu, fv = (u - u0)[..., None], (v - v0)[..., None]
        i, j = v0.long().clamp(0, th - 2), u0.long().clamp(0, tw - 2)
        return ((1 - fv) * ((1 - fu) * tex[i, j] + fu * tex[i, j + 1]) +
                fv * ((1 - fu) * tex[i + 1, j] + fu * tex[i + 1, j + 1]))

    f1 = torch.zeros((H, W, 3), dtype=torch.float64, device=DEV)
    f2 = torch.zeros_like(f1)
    flow0, flow1 = (torch.zeros((H, W, 2), dtype=torch.float64, device=DEV) for _ in range(2))
    for Hm, poly, shift in layers:
        m = inside(poly, xs, ys)[..., None]
        f1 = torch.where(m, sample(xs, ys, shift), f1)
        qx, qy = _map(Hm, xs, ys)
        flow0 = torch.where(m, torch.stack((qx - xs, qy - ys), -1), flow0)
        px, py = _map(np.linalg.inv(Hm), xs, ys)
        m = inside(poly, px, py)[..., None]
        f2 = torch.where(m, sample(px, py, shift), f2)
        flow1 = torch.where(m, torch.stack((px - xs, py - ys), -1), flow1)
    f2 = f2 * rng.uniform(0.85, 1.15)
    if u8:
        f1, f2 = ((f.clamp(0, 1) * 255).round() / 255 for f in (f1, f2))
    return f1.float().contiguous(), f2.float().contiguous(), [l[0] for l in layers], flow0, flow1


def _pack(dx, dy):
    return ((dx & 0xFFFF) | (dy << 16)).to(torch.int32).reshape(-1).contiguous()


def _nnf(flow, seed, wild):
    """A nearest-neighbour field in the middle of the search: the motion rounded to the grid, one pixel off at a third
    of the pixels, anywhere in the frame at the share `wild` of them."""
    H, W, _ = flow.shape
    g = torch.Generator(device=DEV)
    g.manual_seed(seed + 77)
    rnd = lambda n: torch.randint(0, n, (H, W), device=DEV, generator=g)  # noqa: E731
    x, y = torch.arange(W, device=DEV)[None], torch.arange(H, device=DEV)[:, None]
    near = rnd(3) == 0
    tx = x + (flow[..., 0] + 0.5).floor().long() + torch.where(near, rnd(3) - 1, 0)
    ty = y + (flow[..., 1] + 0.5).floor().long() + torch.where(near, rnd(3) - 1, 0)
    far = rnd(1000) < int(1000 * wild)
    tx = torch.where(far, rnd(W), tx).clamp(0, W - 1)
    ty = torch.where(far, rnd(H), ty).clamp(0, H - 1)
    return _pack(tx - x, ty - y)


def _params(c, seed):
    return dict(C=c["C"], r=c["r"], blocks=tuple(int(b) for b in c["blocks"].split(",")), iters=c["iters"],
                hyps=c["hyps"], grad_weight=1.0 if c["C"] == 5 else 0.0, seed=seed % 1000003, fp16=c["fp16"],
                cue_overlap=c["cues"], cue_unique=c["cues"], fill_sweeps=c["fill"], histeq=c["histeq"],
                merge_strict=c["strict"])


def _out(W, H):
    return ([torch.empty((H, W, 2), dtype=torch.float32, device=DEV) for _ in range(2)],
            [torch.empty((H, W), dtype=torch.uint8, device=DEV) for _ in range(2)])


def _label_layers(layers, W, H):
    """Per direction a homography list and per pixel an index into it or -1: planes in vertical bands, every fifth
    pixel without one."""
    Hs = layers[:8]
    xs = torch.arange(W, device=DEV)[None].expand(H, W)
    ys = torch.arange(H, device=DEV)[:, None].expand(H, W)
    label = torch.where((xs * 7 + ys * 3) % 5 == 0, -1, (xs * len(Hs)) // W).reshape(-1)
    return [Hs, [np.linalg.inv(h) for h in Hs]], label.to(torch.int32)


def prepare(case, seed):
    c = case
    if c["kind"] in ("batch", "serve"):
        sizes = (BATCH_SIZES if c["kind"] == "batch" else SERVE_SIZES)[:c["n"]]
        scenes = [_scene(W, H, seed + 131 * i, c["u8"]) for i, (W, H) in enumerate(sizes)]
        pairs = [msgpm.Pair(W, H, device=DEV, **_params(c, seed + i)) for i, (W, H) in enumerate(sizes)]
        st = dict(c=c, pairs=pairs, f1=[s[0] for s in scenes], f2=[s[1] for s in scenes])
        if c["kind"] == "batch":
            st["batch"] = msgpm.Batch(pairs)
        else:
            st["server"] = msgpm.Server(sum(int(p.L.total_bytes) for p in pairs), c["n"], device=DEV)
        return st
    W, H = c["W"], c["H"]
    f1, f2, layers, flow0, flow1 = _scene(W, H, seed, c["u8"])
    pair = msgpm.Pair(W, H, device=DEV, **_params(c, seed))
    st = dict(c=c, pair=pair, f1=f1, f2=f2, layers=layers)
    if c["kind"] == "solve":
        st["out"] = _out(W, H)
        return st
    pair.set_features(f1, f2)
    st["init"] = [_nnf(flow0, seed, 0.4), _nnf(flow1, seed + 1, 0.4)]
    if c["kind"] == "planes":
        st["init"] = [_nnf(flow0, seed, 0.2), _nnf(flow1, seed + 1, 0.2)]
    pair.init_state(*st["init"])
    if c["kind"] in ("restricted", "finalize"):
        Hs, label = _label_layers(layers, W, H)
        arr, half = pair.planes(), pair.n_planes // 2
        for d in range(2):
            for k, Hm in enumerate(Hs[d]):
                arr[d * half + k]["H"] = (Hm / Hm[2, 2]).reshape(-1)
        pair.set_planes(arr)
        for d in range(2):
            index = torch.where(label >= 0, label + d * half, label)
            (pair.hlabel if c["kind"] == "restricted" else pair.win)(d).copy_(index)
    return st


def run(state):
    c = state["c"]
    if c["kind"] == "batch":
        return state["batch"].solve(state["f1"], state["f2"], graph=c["graph"])
    if c["kind"] == "serve":
        server = state["server"]
        tickets = [server.submit(p, a, b) for p, a, b in zip(state["pairs"], state["f1"], state["f2"])]
        server.step()
        for t in tickets:
            server.wait(t)
        return [server.result(t)[1:] for t in tickets]
    pair = state["pair"]
    if c["kind"] == "solve":
        return pair.solve(state["f1"], state["f2"], out=state["out"], graph=c["graph"])
    if c["kind"] == "sweep":
        pair.init_state(*state["init"])
        pair.eval_cost(0)
        pair.pm_halfsweep(0, 3, 0, False)
    elif c["kind"] == "restricted":
        for d in range(2):
            pair.nnf(d).copy_(state["init"][d])
        pair.pm_halfsweep(1, 2, 1, 1 | msgpm.PM_FRESH)
    elif c["kind"] == "finalize":
        flows, occs = pair.finalize()
        return [flows, occs, [pair.cost(d) for d in range(2)]]
    else:
        pair.init_state(*state["init"])
        for stage in (1, 2):
            pair.ransac(0, stage)
            pair.assign(0, stage, True)
            pair.symmetry(0, stage)
            pair.assign(0, stage, False)
        pair.fb_unassign()
        pair.nnf_update(0)
        rec = pair.planes_bytes().view(torch.float64).view(pair.n_planes, 18)
        return dict(H=rec[:, :9], info=rec[:, 9:].view(torch.int32), nnf=[pair.nnf(d) for d in range(2)],
                    win=[pair.win(d) for d in range(2)], loss=[pair.loss(d) for d in range(2)],
                    hlabel=[pair.hlabel(d) for d in range(2)])
    return [[pair.nnf(d) for d in range(2)], [pair.cost(d) for d in range(2)]]


# ---- work --------------------------------------------------------------------------------------------------------

def work(case):
    """Bytes: frames (or stored features and fields) in, results out, each once.  Flops: per pixel of a search pass one
    full patch cost and, per candidate, one record's difference; per window the hypotheses' tests of its points."""
    c = case
    taps = (2 * c["r"] + 1) ** 2
    patch, touch = taps * (3 * c["C"] + 2), 3 * c["C"]
    blocks = [int(b) for b in c["blocks"].split(",")]
    feat = (c["C"] + 1) * 2 if c["fp16"] else 4 * c["C"]

    def candidates(W, H):
        return 4 + max(W, H).bit_length()

    def planes(W, H, b):
        m = lambda n: 1 if n <= b else -(-(n - b) // (b // 2)) + 1  # noqa: E731
        return m(W) * m(H) * min(b, W) * min(b, H) * 2 * c["hyps"] * 19

    def solve(W, H):
        n = 2 * W * H
        return (n * (3 * 4 + 8 + 1), n * (patch + c["iters"] * candidates(W, H) * touch) + sum(planes(W, H, b) for b in blocks))

    if c["kind"] in ("batch", "serve"):
        sizes = (BATCH_SIZES if c["kind"] == "batch" else SERVE_SIZES)[:c["n"]]
        each = [solve(W, H) for W, H in sizes]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    W, H = c["W"], c["H"]
    n = 2 * W * H
    if c["kind"] == "solve":
        b, f = solve(W, H)
        return {"bytes": b, "flops": f}
    if c["kind"] in ("sweep", "restricted"):
        swept = n if c["kind"] == "sweep" else n // 2
        return {"bytes": n * (feat + 4 + 8), "flops": swept * patch + (n // 2) * candidates(W, H) * touch}
    if c["kind"] == "finalize":
        return {"bytes": n * (feat + 8 + 4 + 8 + 1), "flops": n * taps * (12 * c["C"] + 2) * 0.8}
    return {"bytes": n * (feat + 4 + 4 + 4 + 8 + 4), "flops": planes(W, H, blocks[0])}


# ---- the same in FP64 --------------------------------------------------------------------------------------------

def _features(f, c):
    """(H, W, C) FP64: the frame and its luma gradients, rounded to FP16 where the case stores them so."""
    v = f.double()
    if c["C"] == 5:
        Y = 0.299 * v[..., 0] + 0.587 * v[..., 1] + 0.114 * v[..., 2]
        X = torch.cat((Y[:, :1], Y, Y[:, -1:]), 1)
        Z = torch.cat((Y[:1], Y, Y[-1:]), 0)
        v = torch.cat((v, (0.5 * (X[:, 2:] - X[:, :-2]))[..., None], (0.5 * (Z[2:] - Z[:-2]))[..., None]), -1)
    return v.float().half().double() if c["fp16"] else v


def _patch_cost(c, F1, F2, x, y, tx, ty, Hm=None):
    """SSD of the patches of (x, y) in F1 and of (tx, ty) in F2, the latter distorted by the per-pixel homographies Hm
    (n, 3, 3) and sampled bilinearly."""
    H, W, C = F1.shape
    r = c["r"]
    A, B = F1.reshape(-1, C), F2.reshape(-1, C)
    weight = torch.tensor([1.0, 1, 1] + [1.0] * (C - 3), dtype=torch.float64, device=F1.device)
    out = torch.zeros(x.shape, dtype=torch.float64, device=F1.device)

    def project(px, py):
        w = Hm[:, 2, 0] * px + Hm[:, 2, 1] * py + Hm[:, 2, 2]
        return ((Hm[:, 0, 0] * px + Hm[:, 0, 1] * py + Hm[:, 0, 2]) / w,
                (Hm[:, 1, 0] * px + Hm[:, 1, 1] * py + Hm[:, 1, 2]) / w)

    if Hm is not None:
        q0 = project(x.double(), y.double())
    for dy in range(-r, r + 1):
        for dx in range(-r, r + 1):
            a = A[(y + dy).clamp(0, H - 1) * W + (x + dx).clamp(0, W - 1)]
            if Hm is None:
                b = B[(ty + dy).clamp(0, H - 1) * W + (tx + dx).clamp(0, W - 1)]
            else:
                q = project((x + dx).double(), (y + dy).double())
                Dx, Dy = q[0] - q0[0], q[1] - q0[1]
                ux, uy = tx + Dx.floor().long(), ty + Dy.floor().long()
                fx = torch.where((ux >= 0) & (ux < W - 1), Dx - Dx.floor(), 0.0)[:, None]
                fy = torch.where((uy >= 0) & (uy < H - 1), Dy - Dy.floor(), 0.0)[:, None]
                bx, by = ux.clamp(0, W - 1), uy.clamp(0, H - 1)
                cx, cy = (bx + 1).clamp(max=W - 1), (by + 1).clamp(max=H - 1)
                b = ((1 - fy) * ((1 - fx) * B[by * W + bx] + fx * B[by * W + cx]) +
                     fy * ((1 - fx) * B[cy * W + bx] + fx * B[cy * W + cx]))
            out += ((a - b) ** 2 * weight).sum(-1)
    return out


def _mulhilo(a, m):
    """128-bit product of int64 tensors holding 64-bit words with the 64-bit constant m: (high, low)."""
    m0, m1 = m & MASK32, m >> 32
    a0, a1 = a & MASK32, (a >> 32) & MASK32
    top = lambda v: (v >> 32) & MASK32  # noqa: E731

    def mul(u, k):  # 32 x 32 -> 64 bits, as (high, low) 32-bit halves
        p, q = u * (k & 0xFFFF), u * (k >> 16)
        lo = p + ((q & 0xFFFF) << 16)
        return (q >> 16) + (lo >> 32), lo & MASK32

    h00, l00 = mul(a0, m0)
    h01, l01 = mul(a0, m1)
    h10, l10 = mul(a1, m0)
    h11, l11 = mul(a1, m1)
    mid = h00 + l01 + l10
    hi = h01 + h10 + l11 + top(mid)
    return ((h11 + (hi >> 32)) << 32) | (hi & MASK32), ((mid & MASK32) << 32) | l00


def _i64(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _draws(p, k, it, word3, seed, R):
    """The random-search offsets of pixels p at radius number k: Philox4x64-10 (Salmon et al., SC'11)."""
    c = [p.clone(), torch.full_like(p, k), torch.full_like(p, it), torch.full_like(p, word3)]
    k0, k1 = seed, 0
    for rnd in range(10):
        if rnd:
            k0, k1 = k0 + 0x9E3779B97F4A7C15, k1 + 0xBB67AE8584CAA73B
        h0, l0 = _mulhilo(c[0], 0xD2E7470EE14C6C93)
        h1, l1 = _mulhilo(c[2], 0xCA5A826395121157)
        c = [h1 ^ c[1] ^ _i64(k0), l1, h0 ^ c[3] ^ _i64(k1), l0]
    n = 2 * R + 1
    return [((((w >> 32) & MASK32) * n) >> 32) - R for w in c[:2]]


def _offsets(v):
    v = v.long()
    return (((v & 0xFFFF) ^ 0x8000) - 0x8000), v >> 16


def _exact_sweep(c, F, init, seed, colour, it, slot, label=None, Hs=None):
    """Costs after one half-sweep from the fields `init`, every swept pixel's cost computed first."""
    H, W, _ = F[0].shape
    ys, xs = torch.meshgrid(torch.arange(H, device=DEV), torch.arange(W, device=DEV), indexing="ij")
    xs, ys = xs.reshape(-1), ys.reshape(-1)
    R0 = max(W, H)
    costs = []
    for d in range(2):
        ox, oy = _offsets(init[d])
        F1, F2 = F[d], F[1 - d]
        every = _patch_cost(c, F1, F2, xs, ys, xs + ox, ys + oy) if label is None else torch.zeros_like(xs, dtype=torch.float64)
        groups = [None] if label is None else [-1] + list(range(len(Hs[d])))
        for grp in groups:
            sel = (xs + ys) % 2 == colour
            if grp is not None:
                sel &= label == grp
            p = sel.nonzero().reshape(-1)
            if not len(p):
                continue
            x, y = xs[p], ys[p]
            Hm = None
            if grp is not None and grp >= 0:
                Hm = torch.from_numpy(Hs[d][grp] / Hs[d][grp][2, 2]).to(DEV).expand(len(p), 3, 3)
            bx, by = x + ox[p], y + oy[p]
            best = _patch_cost(c, F1, F2, x, y, bx, by, Hm)

            def offer(tx, ty, ok):
                nonlocal bx, by, best
                v = _patch_cost(c, F1, F2, x, y, tx, ty, Hm)
                better = ok & (v < best)
                bx, by, best = torch.where(better, tx, bx), torch.where(better, ty, by), torch.where(better, v, best)

            for sx, sy in ((-1, 0), (1, 0), (0, -1), (0, 1)):
                nx, ny = x + sx, y + sy
                ok = (nx >= 0) & (nx < W) & (ny >= 0) & (ny < H)
                q = ny.clamp(0, H - 1) * W + nx.clamp(0, W - 1)
                offer((x + ox[q]).clamp(0, W - 1), (y + oy[q]).clamp(0, H - 1), ok)
            if Hm is not None:
                qx, qy = _map(Hs[d][grp], x.double(), y.double())
                offer((qx + 0.5).floor().long().clamp(0, W - 1), (qy + 0.5).floor().long().clamp(0, H - 1), best >= 0)
            cx, cy = bx, by
            k = 0
            while R0 >> k:
                dx, dy = _draws(p, k, it, (2 << 24) | (d << 16) | (slot << 8), seed % 1000003, R0 >> k)
                offer((cx + dx).clamp(0, W - 1), (cy + dy).clamp(0, H - 1), best >= 0)
                k += 1
            every[p] = best
        costs.append(every)
    return costs


def exact(case, seed):
    c = case
    if c["kind"] not in ("sweep", "restricted", "finalize") or c["histeq"]:
        return None
    W, H = c["W"], c["H"]
    f1, f2, layers, flow0, flow1 = _scene(W, H, seed, c["u8"])
    F = [_features(f1, c), _features(f2, c)]
    init = [_nnf(flow0, seed, 0.4), _nnf(flow1, seed + 1, 0.4)]
    if c["kind"] == "sweep":
        return [[None, None], _exact_sweep(c, F, init, seed, 0, 3, 0)]
    Hs, label = _label_layers(layers, W, H)
    if c["kind"] == "restricted":
        return [[None, None], _exact_sweep(c, F, init, seed, 1, 2, 1, label, Hs)]
    ys, xs = torch.meshgrid(torch.arange(H, device=DEV), torch.arange(W, device=DEV), indexing="ij")
    xs, ys = xs.reshape(-1), ys.reshape(-1)
    flows, costs = [], []
    for d in range(2):
        dx, dy = _offsets(init[d])
        flow = torch.stack((dx, dy), -1).double()
        cost = torch.zeros(W * H, dtype=torch.float64, device=DEV)
        for k, Hk in enumerate(Hs[d]):
            p = (label == k).nonzero().reshape(-1)
            if not len(p):
                continue
            x, y = xs[p], ys[p]
            qx, qy = _map(Hk, x.double(), y.double())
            flow[p] = torch.stack((qx - x, qy - y), -1)
            Hm = torch.from_numpy(Hk / Hk[2, 2]).to(DEV).expand(len(p), 3, 3)
            cost[p] = _patch_cost(c, F[d], F[1 - d], x, y, x + dx[p], y + dy[p], Hm)
        flows.append(flow.reshape(H, W, 2))
        costs.append(cost)
    return [flows, [None, None], costs]
