"""Timed workloads of the interpolation library, through its public entry
points, with their inputs, their floors and a plain 64-bit statement of
their results.

    listed()             the workloads
    draw(rng)            one more of the same ranges
    prepare(case, seed)  inputs on the GPU, the context and the captured
                         graph that a program keeps
    run(state)           one pass
    work(case)           bytes and operations a pass cannot do without
    exact(case, seed)    the results in 64 bits (plain torch)

Inputs are layered scenes like the ones the paper measures on: polygon
layers with affine motions, an edge-cost map with a response at the layer
boundaries over a noise floor, and matches on a grid thinned at occlusions
and in low-saliency regions, a few of them outliers.
"""
from __future__ import annotations

import math
import random

import torch

import paper_1501_02565_amd as epic

NW, LA = epic.NW, epic.LA
SQRT2 = 1.4142135623730951
# image sizes of a mixed batch (height, width)
MIX_SIZES = [(192, 256), (480, 640), (436, 1024), (375, 1242)]


# --------------------------------------------------------------------------
# the workloads
# --------------------------------------------------------------------------

def listed():
    return [
        # one small pair: latency and launches are all there is
        dict(name="interp_128x96", kind="interp", H=96, W=128, N=300, K=32, a=1.0, mode=LA),
        # odd sizes, a partly filled tile on both edges, the piecewise-constant model
        dict(name="interp_637x479_nw", kind="interp", H=479, W=637, N=3001, K=50, a=0.8, mode=NW),
        # one pair of the size and match count a matcher gives on a film frame
        dict(name="interp_1024x436", kind="interp", H=436, W=1024, N=8000, K=100, a=1.0, mode=LA),
        # the largest single request of a server
        dict(name="interp_2048x1080", kind="interp", H=1080, W=2048, N=40000, K=100, a=1.0, mode=LA),
        # everything in double: the reference setting of the library
        dict(name="fp64_1024x436", kind="fp64", H=436, W=1024, N=8000, K=100, a=1.0, mode=LA),
        # the consistency check of the matches before the interpolation, on a road-camera frame
        dict(name="checked_1242x375", kind="checked", H=375, W=1242, N=10000, K=100, a=0.8, mode=LA),
        # from the image itself: gradient cost and interpolation in one call
        dict(name="image_1280x720", kind="image", H=720, W=1280, N=12000, K=100, a=1.0, mode=LA, channels=3),
        # offline throughput: many pairs of mixed sizes captured once and replayed
        dict(name="batch_64_graph", kind="batch", pairs=64, mix=4000, graph=True, K=100, a=1.0, mode=LA),
        # what a server admits at once: a few pairs of mixed sizes, new every time
        dict(name="batch_6_eager", kind="batch", pairs=6, mix=17, graph=False, K=50, a=1.0, mode=LA),
        # cost maps of a batch of frames in one call
        dict(name="costs_64", kind="costs", images=64, mix=4000, channels=3),
        # the exact per-pixel variant, for comparison with the approximated one
        dict(name="exact_1024x436", kind="exact", H=436, W=1024, N=8000, K=100, a=1.0, mode=LA),
        # the refinement that follows the interpolation
        dict(name="refine_1024x436", kind="refine", H=436, W=1024, channels=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes and match counts spread over their logarithm."""
    kind = rng.choice(["interp", "interp", "interp", "fp64", "checked", "image", "batch", "batch", "costs", "exact",
                       "refine"])
    model = dict(K=rng.choice([32, 50, 64, 100, rng.randint(16, 128)]), a=round(rng.uniform(0.5, 2.0), 3),
                 mode=rng.choice([NW, LA, LA]))
    if kind == "batch":
        n = _log(rng, 2, 48)
        return dict(kind=kind, pairs=n, mix=rng.randint(1, 1 << 20), graph=bool(n > 8 or rng.random() < 0.3), **model)
    if kind == "costs":
        return dict(kind=kind, images=_log(rng, 1, 60), mix=rng.randint(1, 1 << 20), channels=rng.choice([1, 3, 3, 4]))
    hi = {"interp": (1080, 2048), "image": (1080, 2048), "fp64": (480, 1242), "checked": (720, 1280),
          "exact": (300, 640), "refine": (720, 1280)}[kind]
    H, W = _log(rng, 96, hi[0]), _log(rng, 128, hi[1])
    if kind == "refine":
        return dict(kind=kind, H=H, W=W, channels=rng.choice([1, 3, 3]))
    N = _log(rng, 300, min(40000 if hi[0] > 1000 else 12000, max(310, H * W // 45)))
    case = dict(kind=kind, H=H, W=W, N=N, **model)
    if kind == "exact":
        case["N"] = min(N, 4000)
    if kind == "image":
        case["channels"] = rng.choice([1, 3, 3])
    return case


def _pairs(case):
    """(H, W, N) of every pair of a batch: fixed by the case alone."""
    r = random.Random(case["mix"])
    out = []
    for _ in range(case.get("pairs") or case["images"]):
        H, W = r.choice(MIX_SIZES)
        out.append((H, W, r.randint(500, min(15000, H * W // 9))))
    return out


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _blur(x, sigma):
    """Separable Gaussian, borders reflected."""
    r = int(4 * sigma + 0.5)
    w = [math.exp(-0.5 * (k / sigma) ** 2) for k in range(-r, r + 1)]
    s = sum(w)
    for dim in (0, 1):
        n = x.shape[dim]
        i = torch.arange(-r, n + r, device=x.device) % (2 * n)
        i = torch.where(i >= n, 2 * n - 1 - i, i)
        p = x.index_select(dim, i)
        acc = torch.zeros_like(x)
        for k in range(2 * r + 1):
            acc.add_(p.narrow(dim, k, n), alpha=w[k] / s)
        x = acc
    return x


def _boundary(layer):
    b = torch.zeros_like(layer, dtype=torch.bool)
    v = layer[:, 1:] != layer[:, :-1]
    h = layer[1:] != layer[:-1]
    b[:, 1:] |= v
    b[:, :-1] |= v
    b[1:] |= h
    b[:-1] |= h
    return b


class _Scene:
    """Layers, motion and cost map of one image; matches() and image() on request."""

    def __init__(self, H, W, seed, t_range=32.0):
        self.H, self.W = H, W
        self.rng = random.Random(seed)
        self.gen = torch.Generator(device="cuda").manual_seed(seed & 0x7fffffff)
        rng = self.rng
        self.ys, self.xs = torch.meshgrid(torch.arange(H, device="cuda", dtype=torch.float32),
                                          torch.arange(W, device="cuda", dtype=torch.float32), indexing="ij")
        layer = torch.zeros((H, W), dtype=torch.int64, device="cuda")
        motion = []
        n = rng.randint(3, 6)
        for li in range(n):
            cx, cy = (W - 1) / 2, (H - 1) / 2
            if li:
                cx, cy = rng.uniform(0.15, 0.85) * W, rng.uniform(0.15, 0.85) * H
                m = rng.randint(5, 8)
                ang = sorted(rng.uniform(0, 2 * math.pi) for _ in range(m))
                poly = []
                for t in ang:
                    rad = rng.uniform(0.1, 0.3) * min(H, W)
                    poly.append((cx + rad * math.cos(t), cy + rad * math.sin(t)))
                inside = torch.zeros((H, W), dtype=torch.bool, device="cuda")
                for i in range(m):
                    (ax, ay), (bx, by) = poly[i], poly[(i + 1) % m]
                    if ay == by:
                        continue
                    cross = (self.ys < ay) != (self.ys < by)
                    inside ^= cross & (self.xs < (bx - ax) / (by - ay) * (self.ys - ay) + ax)
                layer[inside] = li
            motion.append([rng.uniform(-0.05, 0.05) for _ in range(4)] +
                          [rng.uniform(-t_range, t_range) for _ in range(2)] + [cx, cy])
        self.layer, self.n, self.t_range = layer, n, t_range
        p = torch.tensor(motion, device="cuda")[layer]
        dx, dy = self.xs - p[..., 6], self.ys - p[..., 7]
        self.flow = torch.stack([p[..., 0] * dx + p[..., 1] * dy + p[..., 4],
                                 p[..., 2] * dx + p[..., 3] * dy + p[..., 5]], -1)
        self.edge = _boundary(layer)

    def cost(self):
        c = _blur(self.edge.float(), 1.0)
        return (c + 0.05 * torch.rand(c.shape, device="cuda", generator=self.gen) + 1e-3).contiguous()

    def matches(self, N, outliers=0.05):
        """Exactly N rows x, y, x', y' on a grid, thinned, in raster order."""
        H, W = self.H, self.W
        s = max(1, int(math.sqrt(0.75 * H * W / N)))
        sal = _blur(torch.randn((H, W), device="cuda", generator=self.gen), 8.0)
        while True:
            ok = torch.zeros((H, W), dtype=torch.bool, device="cuda")
            ok[s // 2::s, s // 2::s] = True
            if s > 1:
                ok &= ~self.edge
            pix = ok.flatten().nonzero().squeeze(1)
            if s == 1 or 0.88 * pix.numel() >= N:
                break
            s -= 1
        keep = max(N, int(0.88 * pix.numel()))
        pix = pix[sal.flatten()[pix].argsort(descending=True, stable=True)[:keep]]
        pix = pix[torch.randperm(pix.numel(), device="cuda", generator=self.gen)[:N]]
        bad = pix[:int(outliers * N)]
        u = self.flow.reshape(-1, 2).clone()
        u[bad] = (2 * torch.rand((bad.numel(), 2), device="cuda", generator=self.gen) - 1) * self.t_range
        pix = pix.sort().values
        x, y = (pix % W).float(), torch.div(pix, W, rounding_mode="floor").float()
        return torch.stack([x, y, x + u[pix, 0], y + u[pix, 1]], 1).contiguous()

    def image(self, channels, shift=False):
        """A textured frame (with `shift`, one carried along by a fraction of
        the motion, for the refinement's second frame)."""
        base = torch.tensor([[self.rng.uniform(0.15, 0.85) for _ in range(channels)] for _ in range(self.n)],
                            device="cuda")[self.layer]
        for c in range(channels):
            base[..., c] += 0.25 * _blur(torch.randn((self.H, self.W), device="cuda", generator=self.gen), 2.0)
        img = (base + 0.01 * torch.rand(base.shape, device="cuda", generator=self.gen)).clamp(0, 1)
        img = img if channels > 1 else img[..., 0]
        if not shift:
            return img.contiguous()
        moved = torch.roll(img, (1, 2), (0, 1))
        moved = moved + 0.01 * torch.rand(img.shape, device="cuda", generator=self.gen)
        u = torch.stack([2 + _blur(torch.randn((self.H, self.W), device="cuda", generator=self.gen), 6.0) * 4,
                         1 + _blur(torch.randn((self.H, self.W), device="cuda", generator=self.gen), 6.0) * 4], -1)
        return img.contiguous(), moved.contiguous(), u.contiguous()


def _inputs(case, seed):
    kind = case["kind"]
    if kind in ("batch", "costs"):
        out = []
        for i, (H, W, N) in enumerate(_pairs(case)):
            s = _Scene(H, W, seed * 1009 + i)
            out.append(s.image(case["channels"]) if kind == "costs" else (s.cost(), s.matches(N)))
        return out
    s = _Scene(case["H"], case["W"], seed, 100.0 if case.get("N", 0) == 8000 else 32.0)
    if kind == "refine":
        return s.image(case["channels"], shift=True)
    first = s.image(case["channels"]) if kind == "image" else s.cost()
    return first, s.matches(case["N"])


def prepare(case, seed):
    kind = case["kind"]
    inp = _inputs(case, seed)
    if kind == "costs":
        plan = epic.ImageCostPlan(inp)
        return dict(kind=kind, plan=plan)
    if kind == "batch":
        ws = sum(epic.workspace_bytes(c.shape[0], c.shape[1], m.shape[0], case["K"]) for c, m in inp)
        ctx = epic.Context(workspace=ws)
        problems = [(c, m, case["K"], case["a"], case["mode"]) for c, m in inp]
        outs = [torch.empty(c.shape + (2,), device="cuda") for c, _ in inp]
        graph = ctx.capture(problems, outs) if case["graph"] else None
        return dict(kind=kind, ctx=ctx, problems=problems, outs=outs, graph=graph)
    H, W = case["H"], case["W"]
    out = torch.empty((H, W, 2), device="cuda")
    if kind == "refine":
        ctx = epic.Context(workspace=epic.refine_bytes(H, W, case["channels"]) + (64 << 20))
        return dict(kind=kind, ctx=ctx, inp=inp, out=out)
    N, K = case["N"], case["K"]
    ws = epic.workspace_bytes(H, W, N, K, precision=1 if kind == "fp64" else 0)
    if kind == "image":
        ws += 4 * H * W + 4096
    if kind == "exact":
        ws = max(ws, 1024 * epic.workspace_bytes(H, W, 1, 1)) + 8 * K * (H * W + N) + (64 << 20)
    ctx = epic.Context(workspace=ws, precision=1 if kind == "fp64" else 0, prune_px=5.0 if kind == "checked" else 0.0)
    return dict(kind=kind, ctx=ctx, inp=inp, out=out, K=K, a=case["a"], mode=case["mode"])


def run(s):
    kind = s["kind"]
    if kind == "costs":
        return s["plan"].run()
    if kind == "batch":
        if s["graph"] is not None:
            return s["graph"].launch()
        return s["ctx"].interp_batch(s["problems"], s["outs"])
    if kind == "refine":
        return s["ctx"].refine(*s["inp"], out=s["out"])
    first, matches = s["inp"]
    call = {"image": s["ctx"].interp_image, "exact": s["ctx"].interp_exact}.get(kind, s["ctx"].interp)
    return call(first, matches, s["K"], s["a"], s["mode"], out=s["out"])


def work(case):
    """Bytes: every input read and every output written once.  Operations:
    per pixel and transform one relaxation from each of 8 neighbours (an add
    and a minimum) and the 4 forward pairs of the match graph, per match (per
    pixel in the exact variant) a fit of K neighbours (15 sums of about 2
    operations); the refinement's 5 x 30 sweeps of about 26 operations."""
    kind = case["kind"]
    if kind == "costs":
        px = sum(H * W for H, W, _ in _pairs(case))
        return {"bytes": 4.0 * px * (case["channels"] + 1), "flops": 7.0 * px * case["channels"]}
    if kind == "refine":
        px, ch = case["H"] * case["W"], case["channels"]
        return {"bytes": px * (8.0 * ch + 16), "flops": px * (150 * 26.0 + 60 * ch + 5 * 80)}
    pairs = _pairs(case) if kind == "batch" else [(case["H"], case["W"], case["N"])]
    read = 4.0 * case["channels"] if kind == "image" else 4.0
    times = 2 if kind == "checked" else 1
    b = f = 0.0
    for H, W, N in pairs:
        b += H * W * (read + 8) + 16.0 * N
        fits = H * W if kind == "exact" else N
        f += times * (H * W * 30.0 + fits * min(case["K"], N) * 30.0)
        if kind == "exact":
            f += H * W * min(case["K"], N) * 16.0
    return {"bytes": b, "flops": f}


# --------------------------------------------------------------------------
# the results in 64 bits (plain torch)
# --------------------------------------------------------------------------

_NB = [(1, 0), (-1, 0), (0, 1), (0, -1), (1, 1), (-1, 1), (1, -1), (-1, -1)]      # dx, dy


def _steps(cost):
    """Step cost to each neighbour, in a frame of infinities one pixel wide."""
    H, W = cost.shape
    c = torch.full((H + 2, W + 2), math.inf, dtype=torch.float64, device=cost.device)
    c[1:-1, 1:-1] = cost.double()
    mid = c[1:-1, 1:-1]
    return [(1.0 if dx == 0 or dy == 0 else SQRT2) * (0.5 * (mid + c[1 + dy:H + 1 + dy, 1 + dx:W + 1 + dx]))
            for dx, dy in _NB]


def _relax(seeds, steps):
    """Distances from the pixels where `seeds` is 0 (any leading batch)."""
    H, W = seeds.shape[-2:]
    D = torch.full(seeds.shape[:-2] + (H + 2, W + 2), math.inf, dtype=torch.float64, device=seeds.device)
    D[..., 1:-1, 1:-1] = seeds
    while True:
        before = D.clone()
        for _ in range(16):
            for (dx, dy), w in zip(_NB, steps):
                D[..., 1:-1, 1:-1] = torch.minimum(D[..., 1:-1, 1:-1], D[..., 1 + dy:H + 1 + dy, 1 + dx:W + 1 + dx] + w)
        if torch.equal(before, D):
            return D


def _seed_pixels(matches, H, W):
    x, y = torch.floor(matches[:, 0].double() + 0.5).long(), torch.floor(matches[:, 1].double() + 0.5).long()
    ok = (x >= 0) & (y >= 0) & (x < W) & (y < H)
    return torch.where(ok, y * W + x, -1)


def _owners(matches, H, W):
    """Lowest match of each seeded pixel: (H * W,) with a large number elsewhere."""
    N = matches.shape[0]
    pix = _seed_pixels(matches, H, W)
    own = torch.full((H * W,), 1 << 40, dtype=torch.int64, device=matches.device)
    ok = pix >= 0
    own.scatter_reduce_(0, pix[ok], torch.arange(N, device=matches.device)[ok], "amin")
    return own


def _voronoi(cost, matches):
    H, W = cost.shape
    steps = _steps(cost)
    own = _owners(matches, H, W).view(H, W)
    D = _relax(torch.where(own < 1 << 40, 0.0, math.inf).double(), steps)
    L = torch.full((H + 2, W + 2), 1 << 40, dtype=torch.int64, device=cost.device)
    L[1:-1, 1:-1] = own
    mid = D[1:-1, 1:-1]
    tight = [(D[1 + dy:H + 1 + dy, 1 + dx:W + 1 + dx] + w) == mid for (dx, dy), w in zip(_NB, steps)]
    tight = [t & torch.isfinite(mid) for t in tight]
    while True:
        before = L.clone()
        for _ in range(16):
            for (dx, dy), t in zip(_NB, tight):
                q = torch.where(t, L[1 + dy:H + 1 + dy, 1 + dx:W + 1 + dx], 1 << 40)
                L[1:-1, 1:-1] = torch.minimum(L[1:-1, 1:-1], q)
        if torch.equal(before, L):
            return D, L[1:-1, 1:-1].contiguous(), steps


def _neighbour_lists(D, L, steps, N):
    """The match graph as padded lists (N, degree): neighbour, weight."""
    H, W = L.shape
    keys, ws = [], []
    for k in (0, 2, 4, 5):                         # forward neighbours
        dx, dy = _NB[k]
        y0, y1, x0, x1 = 0, H - dy, max(0, -dx), W - max(0, dx)
        lp, lq = L[y0:y1, x0:x1], L[y0 + dy:y1 + dy, x0 + dx:x1 + dx]
        w = (D[1 + y0:1 + y1, 1 + x0:1 + x1] + steps[k][y0:y1, x0:x1]) + \
            D[1 + y0 + dy:1 + y1 + dy, 1 + x0 + dx:1 + x1 + dx]
        m = lp != lq
        lp, lq, w = lp[m], lq[m], w[m]
        for a, b in ((lp, lq), (lq, lp)):
            keys.append(a * N + b)
            ws.append(w)
    u, inv = torch.unique(torch.cat(keys), return_inverse=True)
    wt = torch.full((u.numel(),), math.inf, dtype=torch.float64, device=L.device)
    wt.scatter_reduce_(0, inv, torch.cat(ws), "amin")
    src, dst = torch.div(u, N, rounding_mode="floor"), u % N
    deg = torch.bincount(src, minlength=N)
    pos = torch.arange(u.numel(), device=L.device) - (deg.cumsum(0) - deg)[src]
    dmax = max(1, int(deg.max()))
    nb = torch.zeros((N, dmax), dtype=torch.int64, device=L.device)
    w = torch.full((N, dmax), math.inf, dtype=torch.float64, device=L.device)
    nb[src, pos], w[src, pos] = dst, wt
    return nb, w


def _nearest(nb, w, K, sources):
    """K nearest matches of each source: (distance, index), infinite padding."""
    N = nb.shape[0]
    out_d, out_i = [], []
    step = max(1, min(len(sources), (1 << 27) // N))
    for c in range(0, len(sources), step):
        s = sources[c:c + step]
        d = torch.full((N, len(s)), math.inf, dtype=torch.float64, device=nb.device)
        d[s, torch.arange(len(s), device=nb.device)] = 0.0
        kk = min(K, N)
        while True:
            for last in (False, False, False, False, True):
                old = d
                d = d.clone()
                for j in range(nb.shape[1]):
                    d = torch.minimum(d, old[nb[:, j]] + w[:, j:j + 1])
            top = torch.topk(d, kk, dim=0, largest=False)
            kth = top.values[-1]
            if not bool(((d < old) & (d <= kth)).any()):
                break
        out_d.append(top.values.T)
        out_i.append(top.indices.T)
    return torch.cat(out_d), torch.cat(out_i)


def _fit(d, rows, ax, ay, au, av, a, mode, wpow=2):
    """Models about the anchors: B (n, 4) and c (n, 2)."""
    ok = torch.isfinite(d)
    k = torch.where(ok, torch.exp(-a * torch.where(ok, d, 0.0)), 0.0)
    dx, dy = rows[..., 0] - ax[:, None], rows[..., 1] - ay[:, None]
    du, dv = rows[..., 2] - rows[..., 0] - au[:, None], rows[..., 3] - rows[..., 1] - av[:, None]
    S = lambda t: t.sum(1)
    B = torch.zeros((d.shape[0], 4), dtype=torch.float64, device=d.device)
    c = torch.stack([au + S(k * du) / S(k), av + S(k * dv) / S(k)], 1)
    if mode == NW:
        return B, c
    w = k * k if wpow == 2 else k
    sw = S(w)
    mx, my = S(w * dx) / sw, S(w * dy) / sw
    ex, ey = dx - mx[:, None], dy - my[:, None]
    sxx, sxy, syy = S(w * ex * ex), S(w * ex * ey), S(w * ey * ey)
    sxu, syu, sxv, syv = S(w * ex * du), S(w * ey * du), S(w * ex * dv), S(w * ey * dv)
    su, sv = S(w * du), S(w * dv)
    cxx, cxy, cyy = sxx / sw, sxy / sw, syy / sw
    disc = torch.sqrt((cxx - cyy) ** 2 + 4 * cxy * cxy)
    l1, l2 = 0.5 * (cxx + cyy + disc), 0.5 * (cxx + cyy - disc)
    good = (ok.sum(1) >= 3) & (l1 > 0) & (l2 > 1e-9 * l1)
    det = torch.where(good, sxx * syy - sxy * sxy, 1.0)
    b = torch.stack([syy * sxu - sxy * syu, sxx * syu - sxy * sxu, syy * sxv - sxy * syv, sxx * syv - sxy * sxv], 1)
    b = b / det[:, None]
    cl = torch.stack([au + su / sw - (b[:, 0] * mx + b[:, 1] * my), av + sv / sw - (b[:, 2] * mx + b[:, 3] * my)], 1)
    return torch.where(good[:, None], b, B), torch.where(good[:, None], cl, c)


def _interp(cost, matches, K, a, mode, check=0.0):
    H, W = cost.shape
    N = matches.shape[0]
    m = matches.double()
    a = float(torch.tensor(a, dtype=torch.float32))
    D, L, steps = _voronoi(cost, matches)
    nb, w = _neighbour_lists(D, L, steps, N)
    used = torch.unique(L)
    d, idx = _nearest(nb, w, K, used)
    au, av = m[used, 2] - m[used, 0], m[used, 3] - m[used, 1]
    B, c = _fit(d, m[idx], m[used, 0], m[used, 1], au, av, a, NW if check else mode)
    if check:
        keep = used[torch.hypot(au - c[:, 0], av - c[:, 1]) <= check]
        return _interp(cost, matches[keep].contiguous(), K, a, mode)
    at = torch.zeros(N, dtype=torch.int64, device=L.device)
    at[used] = torch.arange(len(used), device=L.device)
    j = at[L]
    ys, xs = torch.meshgrid(torch.arange(H, device=L.device), torch.arange(W, device=L.device), indexing="ij")
    dx, dy = xs - m[L, 0], ys - m[L, 1]
    return torch.stack([B[j, 0] * dx + B[j, 1] * dy + c[j, 0], B[j, 2] * dx + B[j, 3] * dy + c[j, 1]], -1)


def _per_pixel(cost, matches, K, a, mode):
    """The exact variant: every pixel's own K nearest matches."""
    H, W = cost.shape
    m = matches.double()
    a = float(torch.tensor(a, dtype=torch.float32))
    steps = _steps(cost)
    own = _owners(matches, H, W)
    pix = (own < 1 << 40).nonzero().squeeze(1)
    src = own[pix]
    n = len(src)
    D = torch.empty((n, H * W), dtype=torch.float64, device=cost.device)
    for c in range(0, n, 64):
        s = torch.full((min(64, n - c), H * W), math.inf, dtype=torch.float64, device=cost.device)
        s[torch.arange(s.shape[0], device=cost.device), pix[c:c + 64]] = 0.0
        D[c:c + 64] = _relax(s.view(-1, H, W), steps)[:, 1:-1, 1:-1].reshape(-1, H * W)
    top = torch.topk(D, min(K, n), dim=0, largest=False)
    idx, d = src[top.indices.T], top.values.T
    p = torch.arange(H * W, device=cost.device)
    px, py = (p % W).double(), torch.div(p, W, rounding_mode="floor").double()
    near = m[idx[:, 0]]
    _, c = _fit(d, m[idx], px, py, near[:, 2] - near[:, 0], near[:, 3] - near[:, 1], a, mode)
    return c.view(H, W, 2)


def _gradient_cost(img, eps):
    g = img.double()
    g = g if g.dim() == 3 else g[..., None]
    H, W = g.shape[:2]
    xl, xr = [torch.arange(W, device=g.device).add(s).clamp(0, W - 1) for s in (-1, 1)]
    yu, yd = [torch.arange(H, device=g.device).add(s).clamp(0, H - 1) for s in (-1, 1)]
    return torch.sqrt(((0.5 * (g[:, xr] - g[:, xl])) ** 2 + (0.5 * (g[yd] - g[yu])) ** 2).sum(-1)) + eps


def _refine(I1, I2, u0):
    """One-level energy minimisation: 5 linearisations of 30 red-black sweeps."""
    lam, delta, gamma, kappa, eps, zeta, omega = [float(torch.tensor(v, dtype=torch.float32))
                                                  for v in (0.1, 0.1, 0.7, 5.0, 1e-3, 0.1, 1.6)]
    I1, I2, u0 = I1.double(), I2.double(), u0.double()
    if I1.dim() == 2:
        I1, I2 = I1[..., None], I2[..., None]
    H, W, _ = I1.shape
    dev = I1.device
    ys, xs = torch.meshgrid(torch.arange(H, device=dev), torch.arange(W, device=dev), indexing="ij")
    fx, fy = (xs + u0[..., 0]).clamp(0, W - 1), (ys + u0[..., 1]).clamp(0, H - 1)
    x0, y0 = fx.floor().long().clamp(max=max(W - 2, 0)), fy.floor().long().clamp(max=max(H - 2, 0))
    x1, y1 = (x0 + 1).clamp(max=W - 1), (y0 + 1).clamp(max=H - 1)
    fx, fy = (fx - x0)[..., None], (fy - y0)[..., None]
    Iw = (1 - fy) * ((1 - fx) * I2[y0, x0] + fx * I2[y0, x1]) + fy * ((1 - fx) * I2[y1, x0] + fx * I2[y1, x1])
    xl, xr = [torch.arange(W, device=dev).add(s).clamp(0, W - 1) for s in (-1, 1)]
    yu, yd = [torch.arange(H, device=dev).add(s).clamp(0, H - 1) for s in (-1, 1)]
    Ix, Iy = 0.5 * (Iw[:, xr] - Iw[:, xl]), 0.5 * (Iw[yd] - Iw[yu])
    gx, gy = 0.5 * (I1[:, xr] - I1[:, xl]), 0.5 * (I1[yd] - I1[yu])
    Iz = Iw - I1
    Ixx, Iyy = Iw[:, xr] - 2 * Iw + Iw[:, xl], Iw[yd] - 2 * Iw + Iw[yu]
    Ixy = 0.25 * (Iw[yd][:, xr] - Iw[yd][:, xl] - Iw[yu][:, xr] + Iw[yu][:, xl])
    Ixz, Iyz = Ix - gx, Iy - gy
    z2 = zeta * zeta
    th, thx, thy = 1 / (Ix ** 2 + Iy ** 2 + z2), 1 / (Ixx ** 2 + Ixy ** 2 + z2), 1 / (Ixy ** 2 + Iyy ** 2 + z2)
    S = lambda t: t.sum(-1)
    JC = [S(th * p) for p in (Ix * Ix, Ix * Iy, Iy * Iy, Ix * Iz, Iy * Iz, Iz * Iz)]
    JG = [S(thx * p + thy * q) for p, q in ((Ixx * Ixx, Ixy * Ixy), (Ixx * Ixy, Ixy * Iyy), (Ixy * Ixy, Iyy * Iyy),
                                            (Ixx * Ixz, Ixy * Iyz), (Ixy * Ixz, Iyy * Iyz), (Ixz * Ixz, Iyz * Iyz))]
    alpha = torch.exp(-kappa * torch.sqrt(S(gx * gx + gy * gy)))
    psi = lambda s2: 0.5 / torch.sqrt(s2.clamp(min=0) + eps * eps)
    quad = lambda J, u, v: J[0] * u * u + 2 * J[1] * u * v + J[2] * v * v + 2 * J[3] * u + 2 * J[4] * v + J[5]
    du, dv = torch.zeros((2, H, W), dtype=torch.float64, device=dev)
    red = (xs + ys) % 2 == 0
    U0, V0 = u0[..., 0], u0[..., 1]

    def gather(e, s, f):            # sum over the 4 edges of weight * f at the other end
        out = torch.zeros_like(f)
        out[:, 1:] += e * f[:, :-1]
        out[:, :-1] += e * f[:, 1:]
        out[1:] += s * f[:-1]
        out[:-1] += s * f[1:]
        return out
    for _ in range(5):
        wc, wg = delta * psi(quad(JC, du, dv)), gamma * psi(quad(JG, du, dv))
        a11, a12, a22, b1, b2 = [wc * p + wg * q for p, q in zip(JC[:5], JG[:5])]
        U, V = U0 + du, V0 + dv
        e = lam * 0.5 * (alpha[:, 1:] + alpha[:, :-1]) * psi((U[:, 1:] - U[:, :-1]) ** 2 + (V[:, 1:] - V[:, :-1]) ** 2)
        s = lam * 0.5 * (alpha[1:] + alpha[:-1]) * psi((U[1:] - U[:-1]) ** 2 + (V[1:] - V[:-1]) ** 2)
        g = gather(e, s, torch.ones_like(du))
        r1, r2 = gather(e, s, U0) - g * U0 - b1, gather(e, s, V0) - g * V0 - b2
        d1, d2 = a11 + g, a22 + g
        w1, w2 = torch.where(d1 > 0, omega / d1, 0.0), torch.where(d2 > 0, omega / d2, 0.0)
        for _ in range(30):
            for colour in (red, ~red):
                nu = (r1 - a12 * dv + gather(e, s, du)) * w1 + (1 - omega) * du
                nu = torch.where(d1 > 0, nu, du)
                nv = (r2 - a12 * nu + gather(e, s, dv)) * w2 + (1 - omega) * dv
                nv = torch.where(d2 > 0, nv, dv)
                du, dv = torch.where(colour, nu, du), torch.where(colour, nv, dv)
    return torch.stack([U0 + du, V0 + dv], -1)


def exact(case, seed):
    kind = case["kind"]
    inp = _inputs(case, seed)
    eps = float(torch.tensor(epic.GRAD_EPS, dtype=torch.float32))
    if kind == "costs":
        return [_gradient_cost(im, eps) for im in inp]
    if kind == "refine":
        return _refine(*inp)
    K, a, mode = case["K"], case["a"], case["mode"]
    if kind == "batch":
        # the pairs of the batch up to a budget of all-pairs graph searches
        out, spent = [], 0
        for c, m in inp:
            spent += m.shape[0] ** 2
            out.append(_interp(c, m, K, a, mode) if spent <= 6e8 else None)
        return out
    first, matches = inp
    if kind == "exact":
        # every match's distances to every pixel: small cases only
        return _per_pixel(first, matches, K, a, mode) if case["N"] * case["H"] * case["W"] <= 3e8 else None
    if kind == "image":
        # the interpolation's input is the 32-bit cost map
        return _interp(_gradient_cost(first, eps).float(), matches, K, a, mode)
    return _interp(first, matches, K, a, mode, 5.0 if kind == "checked" else 0.0)
