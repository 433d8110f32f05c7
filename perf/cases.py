"""The work a program has this library do, as measurable cases.

A case is one pass through the public entry points on inputs that are already where such a program
holds them: device tensors for the direct calls and the autograd function, host arrays for the
serving loop.  Meshes are n x n grids of cloth that ripple and sag over the frames of a trajectory;
observed clouds lie on a perturbed copy of the surface with 5 mm of noise, in random order, as a
depth camera's points against a simulation that does not match it yet.

Kinds of cases (`kind`):
  step    one optimisation step of a calibration: the autograd function from the mesh to the
          per-frame losses and back to the vertex gradient
  calls   the same step as the four direct calls, with every intermediate kept by the caller
  search  the Chamfer forward alone, on two clouds (evaluation of a registration, no gradient)
  sample  surface sampling alone, from a subset of the faces and given random words
  grad    the two backward calls on saved neighbours, with the gradient to the observed cloud
  serve   a batch of uneven requests through the serving loop, host to host
"""
import math
import random

import numpy as np
import torch

import paper_2204_03139_amd as dc
from paper_2204_03139_amd.serving import Server

MOST_PAIRS = 100 * 65536 * 65536       # the largest listed search, in point pairs
MOST_PAIRS_FP32 = 24 * 32768 * 20011   # the largest listed fp32 search
MOST_POINTS = 100 * 65536              # the most points of one cloud over all frames


def listed():
    return [
        # one frame of a coarse cloth: the call where latency and launches count
        dict(name="step-1x2048", kind="step", T=1, n=25, na=2048, nb=2048, prec=0, red=0),
        # the paper's own scale: a 7 x 7 cloth over 25 frames, 3,500 observed points, its loss (Eq. 2)
        dict(name="step-25x3500-eq2", kind="step", T=25, n=7, na=3500, nb=3500, prec=0, red=1),
        # an ordinary trajectory, both losses' directions, each search precision
        dict(name="calls-40x8192-fp32", kind="calls", T=40, n=50, na=8192, nb=8192, prec=0, red=0),
        dict(name="step-40x8192-bf16", kind="step", T=40, n=50, na=8192, nb=8192, prec=1, red=0),
        # the largest trajectory, Eq. 1 and the one-directional Eq. 2
        dict(name="calls-100x65536-bf16", kind="calls", T=100, n=100, na=65536, nb=65536, prec=1,
             red=0),
        dict(name="step-100x65536-eq2", kind="step", T=100, n=100, na=65536, nb=65536, prec=1,
             red=1),
        # uneven clouds in full precision: fewer observed than simulated points, neither a round number
        dict(name="calls-24x32768x20011", kind="calls", T=24, n=80, na=32768, nb=20011, prec=0,
             red=0),
        # one dense scan against another, no trajectory to fill the chip with
        dict(name="search-1x262144", kind="search", T=1, n=100, na=262144, nb=262144, prec=1,
             red=0),
        # redrawing a large trajectory's clouds from its visible faces with the caller's own words
        dict(name="sample-100x65536", kind="sample", T=100, n=100, na=65536, nb=0, prec=0, red=0),
        # backward with the observed cloud optimised too (a second sort), odd sizes
        dict(name="grad-17x30011x5003", kind="grad", T=17, n=33, na=30011, nb=5003, prec=0, red=0),
        # one calibration query served alone: the latency a client sees
        dict(name="serve-1", kind="serve", requests=1, mix=3, prec=1, red=0),
        # a burst of uneven queries: continuous batching at capacity
        dict(name="serve-24", kind="serve", requests=24, mix=1, prec=1, red=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "calls", "calls", "search", "sample", "grad", "serve"])
    if kind == "serve":
        return dict(kind=kind, requests=_log(rng, 1, 24), mix=rng.randrange(1000),
                    prec=rng.randrange(2), red=rng.randrange(2))
    while True:
        prec = rng.randrange(2)
        T = 1 if kind == "search" and rng.random() < 0.5 else _log(rng, 1, 100)
        top = 262144 if kind == "search" else 65536
        na = _log(rng, 500, top)
        nb = _log(rng, 500, top) if rng.random() < 0.5 else na
        if max(T * na, T * nb) > MOST_POINTS:
            continue
        if T * na * nb > (MOST_PAIRS if prec else MOST_PAIRS_FP32):
            continue
        return dict(kind=kind, T=T, n=rng.randint(7, 100), na=na,
                    nb=0 if kind == "sample" else nb, prec=prec, red=rng.randrange(2))


# ------------------------------------------------------------------ inputs
def _mesh(n):
    lin = torch.arange(n, dtype=torch.float64) / (n - 1) - 0.5
    y, x = torch.meshgrid(lin, lin, indexing="ij")
    j, i = torch.meshgrid(torch.arange(n - 1), torch.arange(n - 1), indexing="ij")
    v = (j * n + i).reshape(-1)
    faces = torch.stack([torch.stack([v, v + 1, v + n + 1], 1),
                         torch.stack([v, v + n + 1, v + n], 1)], 1).reshape(-1, 3)
    return x.reshape(-1), y.reshape(-1), faces.to(torch.int32).contiguous()


def _waves(r):
    return dict(amp=[0.05] * 3, kx=[r.uniform(-3, 3) for _ in range(3)],
                ky=[r.uniform(-3, 3) for _ in range(3)],
                phi=[r.uniform(0, 2 * math.pi) for _ in range(3)],
                omega=[r.uniform(0.05, 0.2) for _ in range(3)], sag=0.1)


def _perturbed(w, r):
    return dict(w, amp=[a * r.uniform(0.9, 1.1) for a in w["amp"]],
                phi=[p + r.uniform(-0.3, 0.3) for p in w["phi"]], sag=0.12)


def _height(w, x, y, T):
    t = torch.arange(T, dtype=torch.float64, device=x.device)[:, None]
    z = -w["sag"] * t / max(T - 1, 1) * (1 - 4 * x * x) * (1 - 4 * y * y)
    for k in range(3):
        z = z + w["amp"][k] * torch.sin(2 * math.pi * (w["kx"][k] * x + w["ky"][k] * y)
                                        + w["phi"][k] + w["omega"][k] * t)
    return z


def _cloth(n, T, nb, seed, dev):
    """(verts [T,n*n,3], faces [F,3], observed [T,nb,3] or None) on `dev`."""
    r = random.Random(seed)
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    x, y, faces = _mesh(n)
    x, y = x.to(dev), y.to(dev)
    w = _waves(r)
    verts = torch.stack([x.expand(T, -1), y.expand(T, -1), _height(w, x, y, T)], 2)
    obs = None
    if nb:
        xy = torch.rand((2, T, nb), generator=g, device=dev, dtype=torch.float64) - 0.5
        obs = torch.stack([xy[0], xy[1], _height(_perturbed(w, r), xy[0], xy[1], T)], 2)
        obs += 0.005 * torch.randn((T, nb, 3), generator=g, device=dev, dtype=torch.float64)
        obs = obs.float().contiguous()
    return verts.float().contiguous(), faces.to(dev), obs


def _cloud(n, T, na, seed, dev):
    """A second cloud on the unperturbed surface of `_cloth(n, T, _, seed)`, without noise."""
    r = random.Random(seed)
    g = torch.Generator(device=dev)
    g.manual_seed(seed + 1)
    w = _waves(r)
    xy = torch.rand((2, T, na), generator=g, device=dev, dtype=torch.float64) - 0.5
    return torch.stack([xy[0], xy[1], _height(w, xy[0], xy[1], T)], 2).float().contiguous()


def _requests(case):
    """Sizes of the requests of a serving case: the range of uneven queries, drawn by `mix`."""
    r = random.Random(case["mix"])
    return [dict(n=r.randint(10, 80), T=r.randint(1, 60), na=_log(r, 512, 32768),
                 nb=_log(r, 512, 32768)) for _ in range(case["requests"])]


_server = []


def _the_server():
    if not _server:  # a program keeps one serving loop for its lifetime
        _server.append(Server())
    return _server[0]


def prepare(case, seed):
    dev = torch.device("cuda")
    s = dict(case, seed=seed)
    if case["kind"] == "serve":
        s["server"] = _the_server()
        s["reqs"] = []
        for k, q in enumerate(_requests(case)):
            verts, faces, obs = _cloth(q["n"], q["T"], q["nb"], seed * 64 + k, dev)
            s["reqs"].append(dict(verts=verts.cpu().numpy(), faces=faces.cpu().numpy(),
                                  observed=obs.cpu().numpy(), n_sim=q["na"], seed=seed * 64 + k))
        return s
    T, n, na, nb = case["T"], case["n"], case["na"], case["nb"]
    s["verts"], s["faces"], s["obs"] = _cloth(n, T, nb, seed, dev)
    g = torch.Generator(device=dev)
    g.manual_seed(seed + 2)
    if case["kind"] == "step":
        s["verts"].requires_grad_(True)
    elif case["kind"] == "search":
        s["a"] = _cloud(n, T, na, seed, dev)
    elif case["kind"] == "sample":
        F = s["faces"].shape[0]
        s["words"] = torch.randint(-2**31, 2**31, (T, na, 4), generator=g, device=dev,
                                   dtype=torch.int32)
        s["mask"] = (torch.rand((T, F), generator=g, device=dev) < 0.7).to(torch.uint8)
    elif case["kind"] == "grad":
        s["weights"] = torch.rand(T, generator=g, device=dev, dtype=torch.float64) + 0.5
        s["pts"], s["fidx"], s["bary"] = dc.sample_surface(s["verts"], s["faces"], na, seed=seed)
        f = dc.chamfer_fwd(s["pts"], s["obs"], precision=1)
        s["ia"], s["ib"] = f["idx_a"], f["idx_b"]
    if case["kind"] == "calls":
        s["one"] = torch.ones(T, dtype=torch.float64, device=dev)
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    kind, prec, red = s["kind"], s["prec"], s["red"]
    if kind == "serve":
        server = s["server"]
        tickets = [server.submit(q["verts"], q["faces"], q["observed"], q["n_sim"], seed=q["seed"],
                                 precision=prec, reduction=red) for q in s["reqs"]]
        out = []
        for t in tickets:
            status, loss, grad, _ = server.wait(t)
            if status != 0:
                raise RuntimeError(f"request failed with status {status}")
            out.append((loss, grad))
        return out
    if kind == "step":
        loss = dc.DiffCloudChamfer.apply(s["verts"], s["faces"], s["obs"], s["na"], s["seed"], prec,
                                         red)
        grad, = torch.autograd.grad(loss.sum(), [s["verts"]])
        return dict(loss=loss, grad=grad)
    if kind == "search":
        return dc.chamfer_fwd(s["a"], s["obs"], precision=prec, reduction=red, b_side=red == 0)
    if kind == "sample":
        pts, fidx, bary = dc.sample_surface(s["verts"], s["faces"], s["na"], uniforms=s["words"],
                                            face_mask=s["mask"])
        return dict(points=pts, face=fidx, bary=bary)
    if kind == "grad":
        ga, gb = dc.chamfer_bwd(s["weights"], s["pts"], s["obs"], s["ia"], s["ib"], reduction=red,
                                want_b=True)
        gv = dc.sample_surface_bwd(ga, s["faces"], s["fidx"], s["bary"], s["verts"].shape[1])
        return dict(grad_a=ga, grad_b=gb, grad_verts=gv)
    pts, fidx, bary = dc.sample_surface(s["verts"], s["faces"], s["na"], seed=s["seed"])
    f = dc.chamfer_fwd(pts, s["obs"], precision=prec, reduction=red, b_side=red == 0)
    ga, _ = dc.chamfer_bwd(s["one"], pts, s["obs"], f["idx_a"], f["idx_b"], reduction=red)
    gv = dc.sample_surface_bwd(ga, s["faces"], fidx, bary, s["verts"].shape[1])
    return dict(f, points=pts, face=fidx, bary=bary, grad_a=ga, grad_verts=gv)


# ------------------------------------------------------------------ what a pass cannot do without
def _work(kind, T, n, na, nb, red):
    """Bytes: each input read and each output written once.  Operations: a point's area draw or
    nearest neighbour cannot be found with fewer comparisons than halving the candidates takes
    (2 operations a halving of the areas, 8 for a distance), and a few tens a point of the rest."""
    V, F = n * n, 2 * (n - 1) ** 2
    two = red == 0
    mesh = T * V * 12 + F * 12
    lg = lambda k: math.log2(max(k, 2))  # noqa: E731
    draws = T * na * (2 * lg(F) + 40) + T * F * 25
    search = 8 * T * (na * lg(nb) + (nb * lg(na) if two else 0)) if nb else 0
    back = T * na * 40
    if kind == "search":
        return T * (na + nb) * 12 + T * (na + (nb if two else 0)) * 8 + T * 8, search
    if kind == "sample":
        return mesh + T * F + T * na * (16 + 28), draws
    if kind == "grad":
        return (T * (na + nb) * 12 * 2 + T * (na + (nb if two else 0)) * 4 + T * na * 16 + F * 12
                + T * V * 12), back
    if kind == "calls":
        return (mesh + T * nb * 12 + T * na * (28 + 8 + 12) + (T * nb * 8 if two else 0)
                + T * V * 12), draws + search + back
    return mesh + T * nb * 12 + T * V * 12 + T * 8, draws + search + back


def work(case):
    if case["kind"] == "serve":
        each = [_work("serve", q["T"], q["n"], q["na"], q["nb"], case["red"])
                for q in _requests(case)]
    else:
        each = [_work(case["kind"], case["T"], case["n"], case["na"], case["nb"], case["red"])]
    return dict(bytes=sum(w[0] for w in each), flops=sum(w[1] for w in each))


# ------------------------------------------------------------------ the same in 64 bits
def _philox(seed, T, N):
    """The sampler's documented words, Philox4x64-10 of counter (point, frame, 0, 0)."""
    out = np.empty((T, N, 4), np.uint64)
    top = 1 << 256
    for t in range(T):
        p = np.random.Philox(counter=((t << 64) - 1) % top, key=seed)
        raw = p.random_raw(4 * N).reshape(N, 4)
        out[t, :, 0] = raw[:, 0]
        out[t, :, 1] = raw[:, 1] >> np.uint64(32)
        out[t, :, 2] = raw[:, 2] >> np.uint64(32)
    return out  # face word (64 bits), then the two 32-bit words of the weights


def _sample64(verts, faces, words, mask=None):
    """(points, face, bary): Eq. 3 in double; words [T,N,>=3] as `_philox` lays them out."""
    v = verts.detach().double()
    f = faces.long()
    dev = v.device
    p1, p2, p3 = (v[:, f[:, c]] for c in range(3))
    area = 0.5 * torch.linalg.cross(p2 - p1, p3 - p1).norm(dim=2)
    if mask is not None:
        area = area * (mask != 0)
    cdf = area.cumsum(1)
    w = torch.from_numpy((words[..., 0] >> np.uint64(11)).astype(np.float64)).to(dev)
    target = w * 2.0 ** -53 * cdf[:, -1:]
    face = torch.searchsorted(cdf, target, right=True).clamp_(max=f.shape[0] - 1)
    r1, r2 = (torch.from_numpy((words[..., k] >> np.uint64(8)).astype(np.float64)).to(dev)
              * 2.0 ** -24 for k in (1, 2))
    s = r1.sqrt()
    bary = torch.stack([1 - s, s * (1 - r2), s * r2], 2)
    corner = [torch.gather(p, 1, face[:, :, None].expand(-1, -1, 3)) for p in (p1, p2, p3)]
    return sum(bary[:, :, c:c + 1] * corner[c] for c in range(3)), face, bary


def _nearest64(q, p):
    """Per frame the squared distance to, and index of, the nearest p of every q, in double."""
    T, nq, np_ = q.shape[0], q.shape[1], p.shape[1]
    idx = torch.empty((T, nq), dtype=torch.int64, device=q.device)
    step = max(1, (1 << 28) // np_)
    for t in range(T):
        pt = p[t].t().contiguous()
        norm = (pt * pt).sum(0)[None]
        for i in range(0, nq, step):
            s = torch.addmm(norm, q[t, i:i + step], pt, alpha=-2.0)  # |p|^2 - 2 q.p
            idx[t, i:i + step] = s.argmin(1)
    near = torch.gather(p, 1, idx[:, :, None].expand(-1, -1, 3))
    return ((q - near) ** 2).sum(2), idx


def _scatter(T, n, idx, val):
    out = torch.zeros((T, n, 3), dtype=torch.float64, device=val.device)
    return out.scatter_add_(1, idx[:, :, None].expand(-1, -1, 3), val)


def _chamfer_grad64(a, b, ia, ib, red, g):
    na, nb = a.shape[1], b.shape[1]
    T = a.shape[0]
    alpha, beta = (1.0, 0.0) if red else (1.0 / na, 1.0 / nb)
    g = g[:, None, None]
    da = 2 * alpha * g * (a - torch.gather(b, 1, ia[:, :, None].expand(-1, -1, 3)))
    ga, gb = da, -_scatter(T, nb, ia, da)
    if beta:
        db = 2 * beta * g * (b - torch.gather(a, 1, ib[:, :, None].expand(-1, -1, 3)))
        ga, gb = ga - _scatter(T, na, ib, db), gb + db
    return ga, gb


def _verts_grad64(ga, faces, face, bary, V):
    T = ga.shape[0]
    corners = faces.long()[face]
    return sum(_scatter(T, V, corners[:, :, c], bary[:, :, c:c + 1] * ga) for c in range(3))


def _chamfer64(a, b, red):
    da, ia = _nearest64(a, b)
    if red:
        return da, ia, None, None, da.sum(1)
    db, ib = _nearest64(b, a)
    return da, ia, db, ib, da.mean(1) + db.mean(1)


def _step64(verts, faces, obs, na, seed, red):
    T, V = verts.shape[0], verts.shape[1]
    a, face, bary = _sample64(verts, faces, _philox(seed, T, na))
    b = obs.double()
    da, ia, db, ib, loss = _chamfer64(a, b, red)
    one = torch.ones(T, dtype=torch.float64, device=a.device)
    ga, _ = _chamfer_grad64(a, b, ia, ib, red, one)
    return dict(dist_a=da, idx_a=None, dist_b=db, idx_b=None, loss=loss, points=a, face=None,
                bary=bary, grad_a=ga, grad_verts=_verts_grad64(ga, faces, face, bary, V))


def exact(case, seed):
    dev = torch.device("cuda")
    kind, red = case["kind"], case["red"]
    s = prepare(case, seed)
    if kind == "serve":
        out = []
        for q in s["reqs"]:
            v, f, o = (torch.from_numpy(q[k]).to(dev) for k in ("verts", "faces", "observed"))
            r = _step64(v, f, o, q["n_sim"], q["seed"], red)
            out.append((r["loss"], r["grad_verts"]))
        return out
    if kind == "step":
        r = _step64(s["verts"], s["faces"], s["obs"], s["na"], seed, red)
        return dict(loss=r["loss"], grad=r["grad_verts"])
    if kind == "calls":
        return _step64(s["verts"], s["faces"], s["obs"], s["na"], seed, red)
    if kind == "search":
        da, _, db, _, loss = _chamfer64(s["a"].double(), s["obs"].double(), red)
        return dict(dist_a=da, idx_a=None, dist_b=db, idx_b=None, loss=loss)
    if kind == "sample":
        w = s["words"].cpu().numpy().view(np.uint32).astype(np.uint64)
        words = np.stack([(w[..., 1] << np.uint64(32)) | w[..., 0], w[..., 2], w[..., 3]], -1)
        pts, _, bary = _sample64(s["verts"], s["faces"], words, s["mask"])
        return dict(points=pts, face=None, bary=bary)
    ga, gb = _chamfer_grad64(s["pts"].double(), s["obs"].double(), s["ia"].long(), s["ib"].long(),
                             red, s["weights"])
    gv = _verts_grad64(ga, s["faces"], s["fidx"].long(), s["bary"].double(), s["verts"].shape[1])
    return dict(grad_a=ga, grad_b=gb, grad_verts=gv)
