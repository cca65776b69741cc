"""Performance cases: the calls a program makes on the library, at sizes from
a single small batch of boxes to the largest workloads of the benchmark.

listed() names the cases, draw() gives others of the same ranges, prepare()
makes a case's inputs on the GPU from a seed, run() is one pass through the
public entry points, work() what a pass cannot do without, and exact() its
results in 64 bits by plain torch (its own formulas: no code of the library).

A case's fields: kind (which entry point), n (pairs, or rows of a matrix),
m (columns of a matrix), kmax (vertex slots), dim (5 or 7 box parameters),
z3 (3D), scenes / nmin / nmax (ragged self-pair scenes), api:
  "calls"    the explicit forward and backward functions
  "autograd" the autograd function and torch.autograd.grad
  "forward"  the forward alone, nothing saved
  "kept"     the autograd function with the segment table and the work list
             that a training loop keeps from step to step
"""
import math
import random

import torch

import paper_2011_11134_amd as dg

F32, F64 = torch.float32, torch.float64


def listed():
    return [
        # a small batch of box pairs per training step (the 1,024-pair case):
        # launches and the host's path count, not the chip
        {"name": "pairs_rect_1k", "kind": "pairs", "n": 1024, "kmax": 4, "z3": False, "api": "calls"},
        # every anchor of a batch against its target: the 1,048,576-pair case
        {"name": "pairs_rect_1m", "kind": "pairs", "n": 1 << 20, "kmax": 4, "z3": False,
         "api": "calls"},
        # 3D boxes as a loss in a training step, a large batch of odd size
        {"name": "pairs_3d_2m", "kind": "pairs", "n": 2000003, "kmax": 4, "z3": True,
         "api": "autograd"},
        # convex polygons of 3..8 vertices, the 262,144-pair case
        {"name": "pairs_poly_262k", "kind": "poly", "n": 1 << 18, "kmax": 8, "api": "calls"},
        # boxes by their parameters: the 1,048,576-pair case, and a batch of
        # 3D boxes of ordinary size in a training step
        {"name": "boxes_2d_1m", "kind": "boxes", "n": 1 << 20, "dim": 5, "api": "calls"},
        {"name": "boxes_3d_20k", "kind": "boxes", "n": 20011, "dim": 7, "api": "autograd"},
        # the intersection polygons themselves and their backward
        {"name": "intersect_1m", "kind": "intersect", "n": 1 << 20, "api": "calls"},
        # simple, generally non-convex polygons, the 262,144-pair case
        {"name": "simple_262k", "kind": "simple", "n": 1 << 18, "kmax": 8, "api": "calls"},
        # all detections against all boxes, IoU only: the 4096 x 4096 case
        {"name": "matrix_4096", "kind": "matrix", "n": 4096, "m": 4096, "api": "forward"},
        # predictions against the boxes of a frame with gradients to both sets
        {"name": "matrix_train_1733x301", "kind": "matrix", "n": 1733, "m": 301,
         "api": "autograd"},
        # the 64-scene case: per-scene 3D self pairs of 50..2000 boxes, training
        {"name": "scenes_64", "kind": "scenes", "scenes": 64, "nmin": 50, "nmax": 2000,
         "api": "kept"},
        # a small evaluation batch: the scenes' sizes are new with every call
        {"name": "scenes_8_eval", "kind": "scenes", "scenes": 8, "nmin": 20, "nmax": 200,
         "api": "forward"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["pairs", "poly", "boxes", "intersect", "simple", "matrix", "scenes"])
    if kind == "pairs":
        return {"kind": kind, "n": _log_int(rng, 700, 1500000), "kmax": 4,
                "z3": rng.random() < 0.5, "api": rng.choice(["calls", "autograd", "forward"])}
    if kind == "poly":
        return {"kind": kind, "n": _log_int(rng, 700, 400000), "kmax": rng.choice([4, 6, 8, 8]),
                "api": rng.choice(["calls", "autograd"])}
    if kind == "boxes":
        return {"kind": kind, "n": _log_int(rng, 700, 1500000), "dim": rng.choice([5, 7]),
                "api": rng.choice(["calls", "autograd", "forward"])}
    if kind == "intersect":
        return {"kind": kind, "n": _log_int(rng, 700, 1200000), "api": rng.choice(["calls", "autograd"])}
    if kind == "simple":
        return {"kind": kind, "n": _log_int(rng, 700, 400000), "kmax": rng.choice([6, 8, 8]),
                "api": rng.choice(["calls", "autograd"])}
    if kind == "matrix":
        return {"kind": kind, "n": _log_int(rng, 100, 4096), "m": _log_int(rng, 60, 4096),
                "api": rng.choice(["forward", "autograd"])}
    api = rng.choice(["kept", "forward"])
    return {"kind": kind, "scenes": _log_int(rng, 4, 60), "nmin": rng.randint(10, 50),
            "nmax": _log_int(rng, 120, 1900), "api": api}


# ------------------------------------------------------------------ inputs

class _Rng:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed) + 1000)

    def uniform(self, lo, hi, *shape):
        return torch.rand(*shape, generator=self.g, device="cuda", dtype=F64) * (hi - lo) + lo

    def normal(self, sigma, *shape):
        return torch.randn(*shape, generator=self.g, device="cuda", dtype=F64) * sigma

    def grad(self, *shape):
        return torch.rand(*shape, generator=self.g, device="cuda", dtype=F32) * 2 - 1

    def counts(self, lo, hi, n):
        return torch.randint(lo, hi + 1, (n,), generator=self.g, device="cuda")


def _quads(cx, cy, w, l, yaw):
    lx = torch.tensor([0.5, 0.5, -0.5, -0.5], dtype=F64, device="cuda")
    wy = torch.tensor([-0.5, 0.5, 0.5, -0.5], dtype=F64, device="cuda")
    u, v = l[:, None] * lx, w[:, None] * wy
    c, s = torch.cos(yaw)[:, None], torch.sin(yaw)[:, None]
    return torch.stack([cx[:, None] + c * u - s * v, cy[:, None] + s * u + c * v], -1).float()


def _box_pairs(r, n):
    """Box pairs as a regression head and its targets give them: the second
    box a little moved, resized and turned."""
    p = [r.uniform(-2, 2, n), r.uniform(-2, 2, n), r.uniform(1, 3, n), r.uniform(1, 3, n),
         r.uniform(-math.pi, math.pi, n)]
    q = [p[0] + r.normal(0.3, n), p[1] + r.normal(0.3, n),
         (p[2] + r.normal(0.1, n)).clamp_min(0.1), (p[3] + r.normal(0.1, n)).clamp_min(0.1),
         p[4] + r.normal(0.2, n)]
    return p, q


def _heights(r, n):
    return r.uniform(-2, 1, n), r.uniform(1.4, 1.8, n)


def _bev(r, n):
    """Car boxes in a bird's-eye view of 70 m x 80 m."""
    return _quads(r.uniform(0, 70, n), r.uniform(-40, 40, n), r.uniform(1.5, 2.2, n),
                  r.uniform(3.5, 5.0, n), r.uniform(-math.pi, math.pi, n))


def _convex(r, n, kmax):
    """Convex polygons of 3..kmax vertices on ellipses; redrawn where rounding
    left a vertex that does not turn left."""
    nv = r.counts(3, kmax, n)
    xy = torch.zeros(n, kmax, 2, dtype=F32, device="cuda")
    todo = torch.arange(n, device="cuda")
    slot = torch.arange(kmax, device="cuda")
    while todo.numel():
        t, k = todo.numel(), nv[todo]
        live = slot < k[:, None]
        ang = torch.where(live, r.uniform(0, 2 * math.pi, t, kmax), math.inf).sort(1).values
        ang = torch.where(live, ang, 0.0)
        x = r.uniform(-1, 1, t)[:, None] + r.uniform(0.5, 2, t)[:, None] * torch.cos(ang)
        y = r.uniform(-1, 1, t)[:, None] + r.uniform(0.5, 2, t)[:, None] * torch.sin(ang)
        c = torch.where(live[..., None], torch.stack([x, y], -1), 0.0).float()
        d = c.double()
        nx = torch.where(slot + 1 < k[:, None], slot + 1, 0)
        b = d.gather(1, nx[..., None].expand(-1, -1, 2))
        e = b - d
        f = e.gather(1, nx[..., None].expand(-1, -1, 2))
        ok = ((e[..., 0] * f[..., 1] - e[..., 1] * f[..., 0] > 0) | ~live).all(1)
        xy[todo[ok]] = c[ok]
        todo = todo[~ok]
    return xy, nv.to(torch.uint8)


def _simple(r, n, kmax, cx, cy):
    """Simple polygons of 3..kmax vertices, star-shaped about their centres."""
    nv = r.counts(3, kmax, n)
    gaps = torch.zeros(n, kmax, dtype=F64, device="cuda")
    todo = torch.arange(n, device="cuda")
    slot = torch.arange(kmax, device="cuda")
    while todo.numel():
        t = todo.numel()
        live = slot < nv[todo][:, None]
        g = torch.where(live, r.uniform(0.2, 1.0, t, kmax), 0.0)
        g = g / g.sum(1, keepdim=True) * (2 * math.pi)
        ok = (((g >= 0.15) & (g <= 0.9 * math.pi)) | ~live).all(1)
        gaps[todo[ok]] = g[ok]
        todo = todo[~ok]
    ang = r.uniform(0, 2 * math.pi, n, 1) + gaps.cumsum(1) - gaps
    rad = r.uniform(0.4, 1.6, n, kmax)
    live = slot < nv[:, None]
    x = torch.where(live, cx[:, None] + rad * torch.cos(ang), 0.0)
    y = torch.where(live, cy[:, None] + rad * torch.sin(ang), 0.0)
    return torch.stack([x, y], -1).float(), nv.to(torch.uint8)


def _scene_sizes(case):
    """The scenes' box counts: the case's own, the same for every seed."""
    r = random.Random("%d %d %d" % (case["scenes"], case["nmin"], case["nmax"]))
    return [r.randint(case["nmin"], case["nmax"]) for _ in range(case["scenes"])]


def _offsets(case):
    off = [0]
    for c in _scene_sizes(case):
        off.append(off[-1] + c)
    return off


def _inputs(case, seed):
    r, kind = _Rng(seed), case["kind"]
    s = {}
    if kind in ("pairs", "boxes", "intersect"):
        n = case["n"]
        p, q = _box_pairs(r, n)
        if kind == "boxes":
            if case["dim"] == 7:
                (z, h), (_, h2) = _heights(r, n), _heights(r, n)
                p, q = p + [z, h], q + [z + r.normal(0.3, n), h2]
            s["a"], s["b"] = torch.stack(p, 1).float(), torch.stack(q, 1).float()
            s["g"] = r.grad(n)
            return s
        s["a"], s["b"] = _quads(*p), _quads(*q)
        if kind == "intersect":
            s["g"] = r.grad(n, 8, 2)
            return s
        if case["z3"]:
            (z, h), (_, h2) = _heights(r, n), _heights(r, n)
            z2 = z + r.normal(0.3, n)
            s["az"] = ((z - h / 2).float(), (z + h / 2).float())
            s["bz"] = ((z2 - h2 / 2).float(), (z2 + h2 / 2).float())
        s["g"] = r.grad(n)
    elif kind == "poly":
        s["a"], s["an"] = _convex(r, case["n"], case["kmax"])
        s["b"], s["bn"] = _convex(r, case["n"], case["kmax"])
        s["g"] = r.grad(case["n"])
    elif kind == "simple":
        n = case["n"]
        cx, cy = r.uniform(-1, 1, n), r.uniform(-1, 1, n)
        s["a"], s["an"] = _simple(r, n, case["kmax"], cx, cy)
        s["b"], s["bn"] = _simple(r, n, case["kmax"], cx + r.normal(0.5, n), cy + r.normal(0.5, n))
        s["g"] = r.grad(n)
    elif kind == "matrix":
        s["a"], s["b"] = _bev(r, case["n"]), _bev(r, case["m"])
        if case["api"] == "autograd":
            s["g"] = r.grad(case["n"], case["m"])
    else:
        off = _offsets(case)
        s["a"] = _bev(r, off[-1])
        z, h = _heights(r, off[-1])
        s["az"] = ((z - h / 2).float(), (z + h / 2).float())
        s["off"] = off
        if case["api"] == "kept":
            s["g"] = r.grad(sum((y - x) ** 2 for x, y in zip(off, off[1:])))
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["kind"], s["api"] = case["kind"], case["api"]
    if case["api"] in ("autograd", "kept"):
        s["a"].requires_grad_(True)
        if "b" in s:
            s["b"].requires_grad_(True)
        for z in ("az", "bz"):
            if z in s:
                s[z] = tuple(t.requires_grad_(True) for t in s[z])
    if case["kind"] == "scenes":
        # the batch's offsets, as a data loader gives them
        s["off"] = torch.tensor(s["off"], dtype=torch.int64)
        if case["api"] == "kept":
            n = s["a"].shape[0]
            seg = dg.segments(n, n, s["off"], self_pairs=True)
            s["work"] = (seg, dg.SavedPairs(max(1 << 16, seg[4] // 16), 8, seg[5], s["a"].device))
    return s


# --------------------------------------------------------------------- run

def run(s):
    kind, api = s["kind"], s["api"]
    a, b, g = s["a"], s.get("b"), s.get("g")
    if kind in ("pairs", "poly"):
        an, bn = s.get("an"), s.get("bn")
        az, bz = s.get("az"), s.get("bz")
        if api == "autograd":
            if az is not None:
                iou = dg.IoU3DPairs.apply(a, az[0], az[1], b, bz[0], bz[1])
                return (iou,) + torch.autograd.grad(iou, (a, *az, b, *bz), g)
            iou = dg.IoUPairs.apply(a, b, an, bn)
            return (iou,) + torch.autograd.grad(iou, (a, b), g)
        if api == "forward":
            return dg.iou_pairs(a, b, an, bn, az, bz, save=False)[0]
        iou, nx, xf = dg.iou_pairs(a, b, an, bn, az, bz)
        ga, gb, gaz, gbz = dg.iou_pairs_backward(a, b, g, nx, xf, an, bn, az, bz)
        return (iou, nx, xf, ga, gb) + (() if gaz is None else (gaz, gbz))
    if kind == "boxes":
        if api == "autograd":
            iou = dg.IoUBoxes.apply(a, b)
            return (iou,) + torch.autograd.grad(iou, (a, b), g)
        if api == "forward":
            return dg.iou_boxes(a, b, save=False)[0]
        iou, nx, xf = dg.iou_boxes(a, b)
        return (iou, nx) + dg.iou_boxes_backward(a, b, g, nx, xf)
    if kind == "intersect":
        if api == "autograd":
            xy, nx, xf = dg.Intersect.apply(a, b)
            return (xy, nx, xf) + torch.autograd.grad(xy, (a, b), g)
        xy, nx, xf = dg.intersect(a, b)
        return (xy, nx, xf) + dg.intersect_backward(a, b, g, nx, xf)
    if kind == "simple":
        an, bn = s["an"], s["bn"]
        if api == "autograd":
            iou = dg.IoUSimplePairs.apply(a, b, an, bn)
            return (iou,) + torch.autograd.grad(iou, (a, b), g)
        iou, xm, sm, ins = dg.iou_simple_pairs(a, b, an, bn)
        return (iou, xm, sm, ins) + dg.iou_simple_backward(a, b, g, xm, sm, ins, an, bn)
    if kind == "matrix":
        if api == "forward":
            return dg.iou_matrix(a, b)[0]
        iou = dg.IoUMatrix.apply(a, b)
        return (iou,) + torch.autograd.grad(iou, (a, b), g)
    if api == "forward":
        return dg.iou_matrix(a, a_z=s["az"], a_off=s["off"], self_pairs=True)[0]
    iou = dg.IoU3DScenes.apply(a, s["az"][0], s["az"][1], s["off"], None, s["work"])
    return (iou,) + torch.autograd.grad(iou, (a, *s["az"]), g)


# -------------------------------------------------------------------- work

def work(case):
    """Bytes: every input read once, every output (saved state and gradients
    among them) written once.  Operations: a pair of quadrilaterals takes
    about 320 forward and 420 backward, growing with the product of the
    vertex counts; a matrix's pairs four comparisons each (six in 3D), and
    the full count for the pairs that can meet (about 1 in 100 here)."""
    kind, api = case["kind"], case["api"]
    back = api != "forward"
    if kind in ("matrix", "scenes"):
        if kind == "matrix":
            pairs, boxes, row = case["n"] * case["m"], case["n"] + case["m"], 32
        else:
            c = _scene_sizes(case)
            pairs, boxes, row = sum(v * v for v in c), sum(c), 40
        byts = 4 * pairs + row * boxes
        flops = (4 if kind == "matrix" else 6) * pairs + 320 * pairs // 100
        if back:  # upstream gradients of the pairs that meet, gradients of the boxes
            byts += 4 * (pairs // 100) + 2 * row * boxes
            flops += 420 * pairs // 100
        return {"bytes": byts, "flops": flops}
    n = case["n"]
    if kind == "boxes":
        inp, out, state, f = 8 * case["dim"], 4, 9, 1
    elif kind == "intersect":
        inp, out, state, f = 64, 64, 9, 1
    else:
        k = case["kmax"]
        inp = 16 * k + (16 if case.get("z3") else 0) + (2 if "z3" not in case else 0)
        out, state = 4, 1 + 2 * k if kind != "simple" else 17
        f = ((3 + k) / 2 / 4) ** 2 if kind != "pairs" else 1
    byts = n * (inp + out + (state if back else 0))
    if back:  # the inputs, the state and the upstream gradient read, gradients written
        byts += n * (out + inp)
    return {"bytes": byts, "flops": int(n * f * (740 if back else 320))}


# ------------------------------------------------------------------- exact
# The area of an intersection in 64 bits by Green's theorem: half the sum,
# over the edges of both polygons, of the cross product of an edge's ends times
# the fraction of the edge inside the other polygon, which is its start's
# inclusion plus or minus (1 - t) for each crossing at t.  Gradients by autograd.

def _next(p, n):
    k = p.shape[1]
    i = torch.arange(k, device=p.device)
    i = torch.where(i + 1 < n[:, None], i + 1, 0)
    return p.gather(1, i[..., None].expand(-1, -1, 2)), torch.arange(k, device=p.device) < n[:, None]


def _cross(u, v):
    return u[..., 0] * v[..., 1] - u[..., 1] * v[..., 0]


def _edge_state(p, n, q, m):
    """For every edge i of p and j of q: whether they cross, where along each
    (t on p's edge, s on q's), and whether p's vertex i is left of q's edge."""
    p1, pl = _next(p, n)
    q1, ql = _next(q, m)
    e, f = p1 - p, q1 - q
    w = p[:, :, None] - q[:, None]
    w1 = p1[:, :, None] - q[:, None]
    o0, o1 = _cross(f[:, None], w), _cross(f[:, None], w1)
    r0 = _cross(e[:, :, None], -w)
    r1 = _cross(e[:, :, None], q1[:, None] - p[:, :, None])
    hit = ((o0 > 0) != (o1 > 0)) & ((r0 > 0) != (r1 > 0)) & pl[:, :, None] & ql[:, None]
    t = torch.where(hit, o0, 0) / torch.where(hit, o0 - o1, 1)
    s = torch.where(hit, r0, 0) / torch.where(hit, r0 - r1, 1)
    return hit, t, s, o0 > 0, r0 > 0, p1, q1, pl, ql


def _inside(p, q, q1, ql):
    """Crossing-number inclusion of every vertex of p in q."""
    up0, up1 = q[:, None, :, 1] > p[:, :, None, 1], q1[:, None, :, 1] > p[:, :, None, 1]
    left = _cross((q1 - q)[:, None], p[:, :, None] - q[:, None]) > 0
    return ((up0 != up1) & (left == up1) & ql[:, None]).sum(2) % 2


def _areas(p, n, q, m):
    """Areas of the intersection, of p and of q."""
    c = p[:, :1].detach()
    p, q = p - c, q - c
    hit, t, s, pleft, qleft, p1, q1, pl, ql = _edge_state(p, n, q, m)
    zero = torch.zeros((), dtype=F64, device=p.device)
    fp = _inside(p, q, q1, ql) + torch.where(hit, torch.where(pleft, t - 1, 1 - t), zero).sum(2)
    fq = _inside(q, p, p1, pl) + torch.where(hit, torch.where(qleft, s - 1, 1 - s), zero).sum(1)
    cp = torch.where(pl, _cross(p, p1), zero)
    cq = torch.where(ql, _cross(q, q1), zero)
    return 0.5 * ((cp * fp).sum(1) + (cq * fq).sum(1)), 0.5 * cp.sum(1), 0.5 * cq.sum(1)


def _iou64(p, n, q, m, pz=None, qz=None):
    i, a, b = _areas(p, n, q, m)
    if pz is not None:
        i = i * (torch.minimum(pz[1], qz[1]) - torch.maximum(pz[0], qz[0])).clamp_min(0)
        a, b = a * (pz[1] - pz[0]), b * (qz[1] - qz[0])
    return i / (a + b - i)


def _full(x):
    return torch.full((x.shape[0],), x.shape[1], device=x.device)


def _pairs64(fn, tensors, g, chunk=1 << 17):
    """fn over chunks of the pairs: (values, gradients of sum(g * values))."""
    outs, grads = [], []
    for k in range(0, g.shape[0], chunk):
        x = [t[k:k + chunk].double().requires_grad_(True) for t in tensors]
        v = fn(k, *x)
        outs.append(v.detach())
        grads.append(torch.autograd.grad(v, x, g[k:k + chunk].double()))
    return torch.cat(outs), [torch.cat(c) for c in zip(*grads)]


def _corners64(b):
    cx, cy, w, l, yaw = b[:, :5].unbind(1)
    lx = torch.tensor([0.5, 0.5, -0.5, -0.5], dtype=F64, device=b.device)
    wy = torch.tensor([-0.5, 0.5, 0.5, -0.5], dtype=F64, device=b.device)
    u, v = l[:, None] * lx, w[:, None] * wy
    c, s = torch.cos(yaw)[:, None], torch.sin(yaw)[:, None]
    return torch.stack([cx[:, None] + c * u - s * v, cy[:, None] + s * u + c * v], -1)


def _vertices64(p, q):
    """Ordered intersection vertices of quadrilaterals, [n, 8, 2], from the
    smallest of (vertex of p, vertex of q, crossing)."""
    n = _full(p)
    hit, t, _, _, _, p1, q1, pl, ql = _edge_state(p, n, q, n)
    x = p[:, :, None] + t[..., None] * (p1 - p)[:, :, None]
    pts = torch.cat([p, q, x.flatten(1, 2)], 1)
    live = torch.cat([_inside(p, q, q1, ql) > 0, _inside(q, p, p1, pl) > 0, hit.flatten(1)], 1)
    cnt = live.sum(1)
    with torch.no_grad():
        mid = torch.where(live[..., None], pts, 0).sum(1) / cnt.clamp_min(1)[:, None]
        d = pts - mid[:, None]
        ang = torch.where(live, torch.atan2(d[..., 1], d[..., 0]), math.inf)
        order = ang.argsort(1)[:, :8]  # counter-clockwise, the live ones first
        slot = torch.arange(8, device=p.device)
        first = torch.where(slot < cnt[:, None], order, 99).argmin(1)
        turn = (slot + first[:, None]) % cnt.clamp_min(1)[:, None]
        pick = order.gather(1, torch.where(slot < cnt[:, None], turn, slot))
    v = pts.gather(1, pick[..., None].expand(-1, -1, 2))
    return torch.where((slot < cnt[:, None])[..., None], v, 0)


def _meeting(lo, hi, blo, bhi):
    """Index pairs of boxes [lo, hi] and [blo, bhi] that overlap."""
    return ((lo[:, None] < bhi[None]) & (blo[None] < hi[:, None])).all(-1).nonzero(as_tuple=True)


def _bounds(xy, z=None):
    lo, hi = xy.amin(1), xy.amax(1)
    if z is not None:
        lo, hi = torch.cat([lo, z[0][:, None]], 1), torch.cat([hi, z[1][:, None]], 1)
    return lo, hi


def exact(case, seed):
    s, kind, api = _inputs(case, seed), case["kind"], case["api"]
    a, b, g = s["a"], s.get("b"), s.get("g")
    if kind == "boxes":
        z = case["dim"] == 7

        def boxes(k, x, y):
            zx = (x[:, 5] - x[:, 6] / 2, x[:, 5] + x[:, 6] / 2) if z else None
            zy = (y[:, 5] - y[:, 6] / 2, y[:, 5] + y[:, 6] / 2) if z else None
            p, q = _corners64(x), _corners64(y)
            return _iou64(p, _full(p), q, _full(q), zx, zy)
        iou, (ga, gb) = _pairs64(boxes, (a, b), g)
        return iou if api == "forward" else (iou, ga, gb) if api == "autograd" else (iou, None, ga, gb)
    if kind == "intersect":
        xy, (ga, gb) = _pairs64(lambda k, p, q: _vertices64(p, q), (a, b), g)
        return xy, None, None, ga, gb
    if kind in ("pairs", "poly", "simple"):
        an, bn = (s["an"].long(), s["bn"].long()) if "an" in s else (_full(a), _full(b))
        if "az" in s:
            def pairs3(k, p, pl, ph, q, ql, qh):
                return _iou64(p, _full(p), q, _full(q), (pl, ph), (ql, qh))
            iou, gr = _pairs64(pairs3, (a, *s["az"], b, *s["bz"]), g)
            if api == "calls":
                gr = [gr[0], gr[3], torch.stack(gr[1:3], 1), torch.stack(gr[4:6], 1)]
        else:
            def pairs2(k, p, q):
                return _iou64(p, an[k:k + p.shape[0]], q, bn[k:k + q.shape[0]])
            iou, gr = _pairs64(pairs2, (a, b), g)
        if api == "forward":
            return iou
        state = () if api == "autograd" else (None,) * (3 if kind == "simple" else 2)
        return (iou,) + state + tuple(gr)
    if kind == "matrix":
        i, j = _meeting(*_bounds(a), *_bounds(b))
        x, y = a.double().requires_grad_(True), b.double().requires_grad_(True)
        p, q = x[i], y[j]
        v = _iou64(p, _full(p), q, _full(q))
        out = torch.zeros(case["n"], case["m"], dtype=F64, device="cuda")
        out[i, j] = v.detach()
        if api == "forward":
            return out
        return (out,) + torch.autograd.grad(v, (x, y), g[i, j].double())
    off = s["off"]
    out = torch.zeros(sum((y - x) ** 2 for x, y in zip(off, off[1:])), dtype=F64, device="cuda")
    lo, hi = _bounds(a, s["az"])
    rows, cols, at, twin, o = [], [], [], [], 0
    for x, y in zip(off, off[1:]):
        i, j = _meeting(lo[x:y], hi[x:y], lo[x:y], hi[x:y])
        i, j = i[i < j], j[i < j]
        n = y - x
        out[o:o + n * n].view(n, n).diagonal().fill_(1)
        rows.append(i + x)
        cols.append(j + x)
        at.append(o + i * n + j)
        twin.append(o + j * n + i)
        o += n * n
    rows, cols, at, twin = (torch.cat(v) for v in (rows, cols, at, twin))
    x = [t.double().requires_grad_(True) for t in (a, *s["az"])]
    p, q = x[0][rows], x[0][cols]
    v = _iou64(p, _full(p), q, _full(q), (x[1][rows], x[2][rows]), (x[1][cols], x[2][cols]))
    out[at] = v.detach()
    out[twin] = v.detach()
    if api == "forward":
        return out
    return (out,) + torch.autograd.grad(v, x, (g[at] + g[twin]).double())
