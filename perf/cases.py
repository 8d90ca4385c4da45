"""The work that programs have this library do, as measurable cases.

Each case is one call of a public entry point of ``paper_2512_00385_amd.ezsp``
on a synthetic scene that stands in for the clouds such programs hold: indoor
rooms, driving tiles (density falling with the square of the distance from
the sensor), aerial tiles and ring-ordered LiDAR sweeps.  Scenes are drawn on
the GPU from a seed alone; every point carries its primitive's embedding plus
noise, the structure the learned embeddings are trained to have.

listed()          the named cases
draw(rng)         one more case of the same ranges
prepare(case, s)  inputs and reusable handles, made from seed s
run(state)        one pass through the entry point, its whole outputs
work(case)        bytes and operations the pass cannot do without
tolerance(case)   how far two correct implementations may differ
exact(case, s)    the outputs in 64 bits by plain torch, where they have such
"""
import math

import numpy as np
import torch

from paper_2512_00385_amd import ezsp

DEV = "cuda"
NOISE_XYZ = 0.005  # position noise, metres

# The paper's ladder (one strength, growing minimum sizes) and the ladders of
# growing strength of this repository's workloads.
LADDER = "0.05,0.2,0.8"
LADDER_AERIAL = "0.05,0.2,0.8,3.2"
LADDER_PAPER = "0.02,0.02,0.02"


def listed():
    return [
        # one small room: an interactive tool or a unit of a batch of rooms;
        # latency and launches are all there is
        dict(name="room-partition", op="partition", scene="room", n=20_000,
             d=8, k=10, sigma=0.05, lambdas="0.1", min_size="", energy=False,
             link=False),
        # the headline: one mobile-LiDAR tile, kNN to three levels of labels
        dict(name="street-partition", op="partition", scene="street",
             n=3_000_000, d=16, k=10, sigma=0.05, lambdas=LADDER,
             min_size="", energy=False, link=False),
        # a scanned building floor with the paper's own settings (D = 32,
        # k = 8, one lambda, growing minimum sizes)
        dict(name="indoor-partition", op="partition", scene="room",
             n=1_000_000, d=32, k=8, sigma=0.05, lambdas=LADDER_PAPER,
             min_size="5,30,90", energy=False, link=False),
        # the largest single call: an airborne tile, many merge rounds
        dict(name="aerial-partition", op="partition", scene="aerial",
             n=10_000_000, d=16, k=10, sigma=0.1, lambdas=LADDER_AERIAL,
             min_size="", energy=False, link=False),
        # the ladder on a neighbour table the program already has, with the
        # energy of every level (model selection over lambda)
        dict(name="table-partition", op="from_knn", scene="street",
             n=300_007, d=16, k=10, sigma=0.05, lambdas=LADDER, min_size="",
             energy=True, link=False),
        # the neighbour table alone, with distances, a wider neighbourhood
        # and a size that fills no tile
        dict(name="neighbours", op="knn", scene="room", n=150_001, k=16,
             d2=True),
        # the superpoint graph's node attributes from a partition's labels
        dict(name="attributes", op="stats", scene="street", n=3_000_000,
             d=32, sigma=0.05, level=0, xyz=True),
        # what precedes a partition: the raw tile onto a 10 cm grid
        dict(name="subsample", op="grid", scene="street", n=3_000_000,
             h=0.1),
        # a training step of the embedding: loss, affinities, gradient
        dict(name="edge-loss", op="loss", scene="street", n=3_000_000, d=32,
             k=8, sigma=0.05, tau=1.0, rho=0.3),
        # the same for one crop of a training batch
        dict(name="edge-loss-crop", op="loss", scene="room", n=100_003, d=16,
             k=10, sigma=0.05, tau=1.0, rho=0.3),
        # scoring a partition against the ground truth
        dict(name="purity", op="purity", scene="street", n=3_000_000, d=32,
             sigma=0.05, level=0),
        # embedding one 64-beam sweep
        dict(name="embed-sweep", op="mlp", scene="sweep", n=1_265_474, d_in=6,
             d_out=16),
    ]


def _size(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return n | 1 if rng.random() < 0.5 else n


def draw(rng):
    op = rng.choice(["partition"] * 4 + ["from_knn", "knn", "stats", "grid",
                                         "loss", "purity", "mlp"])
    scene = rng.choice(["room", "street", "aerial", "sweep"])
    n = _size(rng, 2_000, 3_000_000)
    c = dict(op=op, scene=scene, n=n)
    if op in ("partition", "from_knn"):
        paper = rng.random() < 0.4
        c.update(d=32 if paper else rng.choice([4, 8, 13, 16, 16, 32, 64]),
                 k=8 if paper else rng.choice([5, 8, 10, 10, 16]),
                 sigma=0.1 if scene == "aerial" else 0.05,
                 lambdas=LADDER_PAPER if paper else
                 rng.choice(["0.1", LADDER, LADDER_AERIAL]),
                 min_size="5,30,90" if paper else "",
                 energy=rng.random() < 0.3,
                 link=paper and op == "partition" and rng.random() < 0.3)
    elif op == "knn":
        c.update(k=rng.choice([4, 8, 10, 16, 20, 32]),
                 d2=rng.random() < 0.5)
    elif op == "stats":
        c.update(d=rng.choice([8, 13, 16, 32]), sigma=0.05,
                 level=rng.choice([0, 1]), xyz=rng.random() < 0.7)
    elif op == "grid":
        c.update(h=rng.choice([0.03, 0.1, 0.25]))
    elif op == "loss":
        c.update(d=rng.choice([8, 16, 20, 32, 64]),
                 k=rng.choice([5, 8, 10, 16]), sigma=0.05,
                 tau=rng.choice([0.5, 1.0]),
                 rho=rng.choice([0.1, 0.3, 1.0]))
    elif op == "purity":
        c.update(d=32, sigma=0.05, level=rng.choice([0, 1]))
    else:
        c.update(d_in=rng.choice([3, 4, 6, 8]), d_out=rng.choice([8, 16, 32]))
    return c


# --------------------------------------------------------------------------
# scenes: rectangles (origin, two edges), a ground and blobs, drawn on the
# GPU; the few hundred primitives come from numpy
# --------------------------------------------------------------------------

def _box(lo, s):
    x, y, z = s
    ex, ey, ez = (x, 0, 0), (0, y, 0), (0, 0, z)
    a = np.asarray(lo, float)
    return [(a + ez, ex, ey), (a, ex, ez), (a + ey, ex, ez), (a, ey, ez),
            (a + ex, ey, ez)]


def _rects(prims):
    """(origins, edges u, edges v, primitive id) of every rectangle."""
    rows = [(o, u, v, i) for i, p in enumerate(prims) for o, u, v in p]
    o, u, v = (torch.tensor(np.array([r[j] for r in rows], np.float64),
                            device=DEV) for j in range(3))
    i = torch.tensor([r[3] for r in rows], device=DEV)
    return o, u, v, i


def _on_rects(g, rects, weight, m):
    """m points on rectangles chosen by weight, with primitive and
    rectangle ids."""
    o, u, v, pid = rects
    cum = torch.cumsum(weight, 0)
    r = torch.rand(m, generator=g, device=DEV, dtype=torch.float64) * cum[-1]
    at = torch.searchsorted(cum, r).clamp_(max=len(cum) - 1)
    a = torch.rand(m, 1, generator=g, device=DEV, dtype=torch.float64)
    b = torch.rand(m, 1, generator=g, device=DEV, dtype=torch.float64)
    return o[at] + a * u[at] + b * v[at], pid[at], at


def _area(rects):
    return torch.linalg.cross(rects[1], rects[2]).norm(dim=1)


def _waves(rng, count, lo, hi, amp):
    th, wl, ph = (rng.uniform(0, 2 * np.pi, count), rng.uniform(lo, hi, count),
                  rng.uniform(0, 2 * np.pi, count))

    def h(x, y):
        z = x * 0
        for t, w, p in zip(th, wl, ph):
            arg = 2 * np.pi * (x * np.cos(t) + y * np.sin(t)) / w + p
            z = z + amp / count * (torch.sin(arg) if torch.is_tensor(arg)
                                   else np.sin(arg))
        return z
    return h


def _room(rng, g, n):
    """A room whose floor area grows with n: shell and boxes, no shuffle."""
    s = min(1.0, max(0.35, (n / 1e6) ** 0.5))
    X, Y, Z = 5 + 5 * s, 5 + 3 * s, 3.0
    prims = [[((0, 0, 0), (X, 0, 0), (0, Y, 0))],
             [((0, 0, Z), (X, 0, 0), (0, Y, 0))],
             [((0, 0, 0), (X, 0, 0), (0, 0, Z))],
             [((0, Y, 0), (X, 0, 0), (0, 0, Z))],
             [((0, 0, 0), (0, Y, 0), (0, 0, Z))],
             [((X, 0, 0), (0, Y, 0), (0, 0, Z))]]
    for _ in range(int(10 + 24 * s)):
        b = rng.uniform(0.3, 1.5, 3)
        prims.append(_box((rng.uniform(0, X - b[0]), rng.uniform(0, Y - b[1]),
                           0.0), b))
    rects = _rects(prims)
    pts, obj, _ = _on_rects(g, rects, _area(rects), n)
    return pts, obj, len(prims)


def _street(rng, g, n):
    """A driving tile of 100 m: ground, cars, posts and facades, density
    1 / max(r, 2 m)^2 around the sensor at the origin."""
    half = 50.0
    h = _waves(rng, 8, 10.0, 50.0, 1.0)
    prims = []
    for _ in range(200):
        s = np.array([4.5, 1.8, 1.5]) * rng.uniform(0.9, 1.1, 3)
        if rng.random() < 0.5:
            s[:2] = s[1::-1]
        c = rng.uniform(-half + 3, half - 3, 2)
        prims.append(_box((c[0] - s[0] / 2, c[1] - s[1] / 2, h(*c)), s))
    for _ in range(300):
        c = rng.uniform(-half + 1, half - 1, 2)
        prims.append(_box((c[0] - 0.13, c[1] - 0.13, h(*c)),
                          (0.26, 0.26, rng.uniform(3.0, 8.0)))[1:])
    for _ in range(40):
        c, w = rng.uniform(-half + 5, half - 5, 2), rng.uniform(10.0, 40.0)
        u = (w, 0, 0) if rng.random() < 0.5 else (0, w, 0)
        o = np.array([c[0], c[1], h(*c)]) - np.array(u) / 2
        prims.append([(o, u, (0, 0, rng.uniform(5.0, 15.0)))])
    rects = _rects(prims)

    def density(x, y):
        return (2.0 / torch.hypot(x, y).clamp(min=2.0)) ** 2

    # rectangles by area and their largest density, thinned by the density
    o, u, v, _ = rects
    lo, hi = torch.minimum(o, o + u + v), torch.maximum(o, o + u + v)
    near = torch.maximum(lo, -hi).clamp(min=0.0)
    pmax = density(near[:, 0], near[:, 1])
    weight = _area(rects) * pmax
    R = half * math.sqrt(2.0)
    ground = 4 * math.pi + 8 * math.pi * math.log(R / 2.0)
    # candidates per unit of weight, with room for what is thinned out
    total = float(weight.sum())
    m_o = int(1.3 * n * total / (ground + total)) + 64
    q, obj, at = _on_rects(g, rects, weight, m_o)
    ok = torch.rand(m_o, generator=g, device=DEV) * pmax[at] \
        < density(q[:, 0], q[:, 1])
    q, obj = q[ok], obj[ok] + 1
    # the ground takes the rest; a tenth of its radial law is off the tile
    m_g = int(1.3 * max(n - q.shape[0], 0)) + 1000
    t = torch.rand(m_g, generator=g, device=DEV, dtype=torch.float64) \
        * (0.5 + math.log(R / 2.0))
    r = torch.where(t < 0.5, torch.sqrt(8 * t), 2 * torch.exp(t - 0.5))
    a = torch.rand(m_g, generator=g, device=DEV, dtype=torch.float64) \
        * (2 * math.pi)
    x, y = r * torch.cos(a), r * torch.sin(a)
    ok = (x.abs() < half) & (y.abs() < half)
    x, y = x[ok], y[ok]
    keep = max(n - q.shape[0], 0)
    x, y = x[:keep], y[:keep]
    pts = torch.cat([q, torch.stack([x, y, h(x, y)], 1)])
    obj = torch.cat([obj, obj.new_zeros(x.shape[0])])
    assert pts.shape[0] >= n, "the street scene fell short of points"
    return pts[:n], obj[:n], len(prims) + 1


def _aerial(rng, g, n):
    """An airborne tile seen from above: terrain, one building in most cells
    of a 20 x 20 grid, a tenth of the points in vegetation blobs; its side
    gives the 40 points per square metre of a 500 m, 10M-point tile."""
    side = math.sqrt(n / 40.0)
    cell = side / 20
    h = _waves(rng, 6, side / 10, side / 2.5, 5.0)
    x, y = (torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * side
            for _ in range(2))
    z, obj = h(x, y), torch.zeros(n, dtype=torch.int64, device=DEV)
    size = torch.tensor(rng.uniform(0.4, 0.85, (400, 2)) * cell, device=DEV)
    at = torch.tensor(rng.uniform(0.0, 0.15, (400, 2)) * cell, device=DEV)
    tall = torch.tensor(rng.uniform(5.0, 30.0, 400), device=DEV)
    c = (x / cell).long().clamp_(max=19) * 20 + (y / cell).long().clamp_(max=19)
    lx, ly = x - (c // 20) * cell - at[c, 0], y - (c % 20) * cell - at[c, 1]
    roof = (lx >= 0) & (ly >= 0) & (lx < size[c, 0]) & (ly < size[c, 1])
    z = torch.where(roof, tall[c] + 5.0, z)
    obj = torch.where(roof, c + 1, obj)
    blobs = max(8, n // 5000)
    m = n // 10
    bc = torch.tensor(rng.uniform(0, side, (blobs, 2)), device=DEV)
    rad = torch.tensor(rng.uniform(0.5, 2.0, blobs), device=DEV)
    b = torch.randint(0, blobs, (m,), generator=g, device=DEV)
    off = torch.randn(m, 3, generator=g, device=DEV, dtype=torch.float64) \
        * rad[b, None]
    x[:m], y[:m] = bc[b, 0] + off[:, 0], bc[b, 1] + off[:, 1]
    z[:m] = h(bc[b, 0], bc[b, 1]) + 3.0 + off[:, 2]
    obj[:m] = 401 + b
    return torch.stack([x, y, z], 1), obj, 401 + blobs


def _sweep(rng, g, n):
    """One revolution of a 64-beam sensor, ring by ring: each ray ends on the
    ground or on the object of its azimuth sector."""
    i = torch.arange(n, device=DEV)
    per = (n + 63) // 64
    ring = i // per
    el = (-24.8 + 26.8 / 63 * ring.double()) * (math.pi / 180)
    az = (i % per).double() / per * (2 * math.pi)
    sectors = 160
    dist = torch.tensor(rng.uniform(4.0, 60.0, sectors), device=DEV)
    tall = torch.tensor(rng.uniform(1.5, 12.0, sectors), device=DEV)
    s = (az / (2 * math.pi) * sectors).long().clamp_(max=sectors - 1)
    to_ground = torch.where(el < -0.015, 1.8 / torch.sin(-el).clamp(min=1e-3),
                            el * 0 + 120.0)
    at = dist[s] / torch.cos(el)
    hit = (at < to_ground) & (1.8 + at * torch.sin(el) < tall[s])
    r = torch.where(hit, at, to_ground)
    pts = torch.stack([r * torch.cos(el) * torch.cos(az),
                       r * torch.cos(el) * torch.sin(az),
                       1.8 + r * torch.sin(el)], 1)
    return pts, torch.where(hit, s + 1, s * 0), sectors + 1


SCENES = dict(room=_room, street=_street, aerial=_aerial, sweep=_sweep)


def _scene(case, seed):
    """xyz [n, 3] fp32, class [n] int32, number of classes, generator.  All
    scenes but the sweep are stored in random order."""
    rng = np.random.default_rng(seed)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    n = case["n"]
    pts, obj, n_obj = SCENES[case["scene"]](rng, g, n)
    pts = pts + NOISE_XYZ * torch.randn(n, 3, generator=g, device=DEV,
                                        dtype=torch.float64)
    if case["scene"] != "sweep":
        order = torch.argsort(torch.rand(n, generator=g, device=DEV,
                                         dtype=torch.float64))
        pts, obj = pts[order], obj[order]
    return (pts.float().contiguous(), obj.to(torch.int32).contiguous(), n_obj,
            g)


def _embed(g, obj, n_obj, d, sigma):
    centre = torch.randn(n_obj, d, generator=g, device=DEV)
    emb = torch.randn(obj.shape[0], d, generator=g, device=DEV)
    return emb.mul_(sigma).add_(centre[obj.long()])


def _numbers(text, kind):
    return [kind(x) for x in text.split(",")] if text else None


def prepare(case, seed):
    xyz, obj, n_obj, g = _scene(case, seed)
    op, s = case["op"], dict(case=case)
    if op == "knn":
        s.update(xyz=xyz)
    elif op == "grid":
        s.update(xyz=xyz)
    elif op == "mlp":
        d_in, d_out = case["d_in"], case["d_out"]
        feat = torch.rand(case["n"], d_in, generator=g, device=DEV)
        c = min(3, d_in)
        feat[:, :c] = xyz[:, :c] / torch.tensor([50.0, 50.0, 5.0],
                                                device=DEV)[:c]
        s["x"] = feat.to(torch.bfloat16)
        for j, (a, b) in enumerate([(d_in, 32), (32, 32), (32, d_out)], 1):
            w, v = (torch.rand(t, generator=g, device=DEV) * 2 - 1
                    for t in ((a, b), (b,)))
            s["w%d" % j] = (w / math.sqrt(a)).to(torch.bfloat16)
            s["b%d" % j] = v / math.sqrt(a)
    else:
        emb = _embed(g, obj, n_obj, case["d"], case["sigma"])
        s.update(emb=emb)
        if op == "partition":
            s.update(xyz=xyz, handle=ezsp.Partitioner(
                case["n"], case["d"], case["k"],
                _numbers(case["lambdas"], float),
                _numbers(case["min_size"], int), energy=case["energy"],
                link=case["link"]))
        elif op == "from_knn":
            s.update(nbr=ezsp.knn(xyz, case["k"]))
        elif op == "loss":
            word = torch.randint(-2**31, 2**31, (case["n"], case["k"]),
                                 generator=g, device=DEV, dtype=torch.int32)
            s.update(nbr=ezsp.knn(xyz, case["k"]), cls=obj, word=word)
        else:  # a partition's labels are what attributes and scores are of
            labels, n_comp, _ = ezsp.partition(xyz, emb, 8, [0.02, 0.02],
                                               [5, 30])
            at = case["level"]
            s.update(labels=labels[at].clone(), n_comp=int(n_comp[at]),
                     cls=obj, n_cls=n_obj,
                     xyz=xyz if case.get("xyz") else None)
            rows = case["n"] // (4 if at == 0 else 24) + 64
            if op == "stats":
                s["size"] = _kept(rows, dtype=torch.int64)
                s["mean"] = _kept(rows, case["d"])
                s["centroid"] = _kept(rows, 3) if case["xyz"] else None
            else:
                s["majority"] = _kept(rows, dtype=torch.int32)
    if op == "grid":
        s["keep"] = _kept(case["n"], dtype=torch.int32)
    return s


# How many rows come back depends on the data; the program keeps them in
# arrays of the largest size (a superpoint has at least 5 or 30 points but
# for a few isolated ones).

def _kept(*shape, dtype=torch.float32):
    return torch.full(shape, -1, dtype=dtype, device=DEV)


def _keep(buf, rows):
    buf[:rows.shape[0]].copy_(rows)
    return buf


def run(s):
    c = s["case"]
    op = c["op"]
    if op == "partition":
        labels, n_comp, energy = s["handle"](s["xyz"], s["emb"])
        out = dict(labels=labels, n_comp=n_comp)
        return dict(out, energy=energy) if c["energy"] else out
    if op == "from_knn":
        labels, n_comp, energy = ezsp.partition_from_knn(
            s["nbr"], s["emb"], _numbers(c["lambdas"], float),
            _numbers(c["min_size"], int), energy=c["energy"])
        out = dict(labels=labels, n_comp=n_comp)
        return dict(out, energy=energy) if c["energy"] else out
    if op == "knn":
        if c["d2"]:
            nbr, d2 = ezsp.knn(s["xyz"], c["k"], want_d2=True)
            return dict(nbr=nbr, d2=d2)
        return dict(nbr=ezsp.knn(s["xyz"], c["k"]))
    if op == "stats":
        size, mean, centroid = ezsp.component_stats(
            s["labels"], s["n_comp"], s["emb"], s["xyz"])
        out = dict(size=_keep(s["size"], size), mean=_keep(s["mean"], mean))
        return dict(out, centroid=_keep(s["centroid"], centroid)) \
            if c["xyz"] else out
    if op == "grid":
        keep = ezsp.grid_subsample(s["xyz"], c["h"])
        return dict(n_keep=keep.shape[0], keep=_keep(s["keep"], keep))
    if op == "loss":
        stats, affinity, grad, sampled = ezsp.edge_loss(
            s["emb"], s["nbr"], s["cls"], s["word"], c["tau"], c["rho"])
        return dict(stats, affinity=affinity, grad=grad, sampled=sampled)
    if op == "purity":
        stats, majority, iou = ezsp.purity(s["labels"], s["n_comp"], s["cls"],
                                           s["n_cls"])
        return dict(stats, majority=_keep(s["majority"], majority), iou=iou)
    return dict(out=ezsp.embed_mlp(s["x"], s["w1"], s["b1"], s["w2"], s["b2"],
                                   s["w3"], s["b3"]))


def work(case):
    """Inputs read once and outputs written once (the few values per
    superpoint and class left out); operations where they are fixed by the
    sizes alone: about 3 D per slot of the loss, two per weight of the MLP."""
    op, n = case["op"], case["n"]
    d, k = case.get("d", 0), case.get("k", 0)
    levels = len(case.get("lambdas", "").split(","))
    flops = 0.0
    if op == "partition":
        nbytes = n * (12.0 + 4 * d + 4 * levels)
    elif op == "from_knn":
        nbytes = n * (4.0 * k + 4 * d + 4 * levels)
    elif op == "knn":
        nbytes = n * (12.0 + 4 * k + (4 * k if case["d2"] else 0))
    elif op == "stats":
        nbytes = n * (4.0 + 4 * d + (12 if case["xyz"] else 0))
        flops = n * (d + (3.0 if case["xyz"] else 0))
    elif op == "grid":
        nbytes = n * 12.0
    elif op == "loss":
        nbytes = n * (8.0 * d + 4 + k * (4 + 4 + 4 + 1.0))
        flops = n * k * 6.0 * d
    elif op == "purity":
        nbytes = n * 8.0
    else:
        nbytes = n * (2.0 * case["d_in"] + 4.0 * case["d_out"])
        flops = 2.0 * n * (case["d_in"] * 32 + 1024 + 32 * case["d_out"])
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    """Labels, neighbours, distances, exact sums and counts are the same on
    every correct implementation.  The loss works in fp32 with a free
    summation order, the MLP in bf16 with fp32 sums: hidden units next to a
    rounding boundary may take the other bf16 value.  The level energies are
    fp64 sums in a free order."""
    if case["op"] == "loss":
        return dict(rel=4e-7)
    if case["op"] == "mlp":
        return dict(rel=5e-5)
    if case.get("energy"):
        return dict(rel=1e-12)
    return "exact"


# --------------------------------------------------------------------------
# the outputs in 64 bits, by plain torch
# --------------------------------------------------------------------------

def _exact_knn(s, c):
    p, k = s["xyz"].double(), c["k"]
    n = p.shape[0]
    if n > 400_000:
        return None
    p = p - p.mean(0)
    sq = (p * p).sum(1)
    out = torch.full((n, k), math.inf, dtype=torch.float64, device=DEV)
    rows = max(1, 400_000_000 // n)
    take = min(k + 5, n)
    for a in range(0, n, rows):
        b = min(a + rows, n)
        # squared distances less each row's own |p|^2; candidates by these,
        # then their distances from the differences
        m = torch.addmm(sq[None, :].expand(b - a, n), p[a:b], p.t(),
                        alpha=-2.0)
        at = torch.topk(m, take, dim=1, largest=False).indices
        d = ((p[at] - p[a:b, None]) ** 2).sum(2)
        d[at == torch.arange(a, b, device=DEV)[:, None]] = math.inf
        d = d.sort(1).values[:, :k]
        out[a:b, :d.shape[1]] = d
    return dict(nbr=None, d2=out) if c["d2"] else None


def _exact_loss(s, c):
    emb, nbr = s["emb"].double(), s["nbr"].long()
    n, k = nbr.shape
    p = torch.arange(n, device=DEV)[:, None].expand(n, k).reshape(-1)
    q = nbr.reshape(-1)
    slot = torch.arange(n * k, device=DEV)
    valid = q >= 0
    # the owner of a pair is the smallest slot that lists it
    lo, hi = torch.minimum(p, q), torch.maximum(p, q)
    key = torch.where(valid & (p != q), lo * n + hi, -1 - slot)
    skey, order = torch.sort(key, stable=True)
    head = torch.ones_like(skey, dtype=torch.bool)
    head[1:] = skey[1:] != skey[:-1]
    owner = torch.zeros(n * k, dtype=torch.bool, device=DEV)
    owner[order] = head & (skey >= 0)
    same = s["cls"][p] == s["cls"][q.clamp(min=0)]
    intra, inter = owner & same, owner & ~same
    n_intra, n_inter = int(intra.sum()), int(inter.sum())
    m = n_intra
    if c["rho"] < 1.0:
        m = min(m, int(math.floor(c["rho"] * n_inter / (1.0 - c["rho"]))))
    at = slot[intra]
    word = s["word"].reshape(-1)[at].long() & 0xffffffff
    taken = at[torch.argsort(word, stable=True)[:m]]
    sampled = inter.clone()
    sampled[taken] = True
    affinity = torch.zeros(n * k, dtype=torch.float64, device=DEV)
    grad = torch.zeros_like(emb)
    loss = 0.0
    step = 4_000_000
    for a in range(0, n * k, step):
        e = slice(a, min(a + step, n * k))
        qq = q[e].clamp(min=0)
        diff = emb[p[e]] - emb[qq]
        dist = diff.norm(dim=1)
        x = dist / c["tau"]
        affinity[e] = torch.where(valid[e], torch.exp(-x), x * 0)
        t = sampled[e]
        diff, dist, x, i = diff[t], dist[t], x[t], same[e][t]
        loss += float(torch.where(i, x, -torch.log(-torch.expm1(-x))).sum())
        coef = torch.where(i, x * 0 + 1, -1.0 / torch.expm1(x)) / c["tau"] \
            / dist
        coef = torch.where(dist > 0, coef, x * 0)
        diff = diff * coef[:, None]
        grad.index_add_(0, p[e][t], diff)
        grad.index_add_(0, qq[t], -diff)
    return dict(loss=loss, n_edges=n_intra + n_inter, n_intra=n_intra,
                n_inter=n_inter, n_intra_kept=m,
                affinity=affinity.reshape(n, k), grad=grad,
                sampled=sampled.reshape(n, k).to(torch.uint8))


def _exact_stats(s, c):
    lab, nc = s["labels"].long(), s["n_comp"]
    size = torch.bincount(lab, minlength=nc)

    # sums of a superpoint's rows as differences of running sums over the
    # rows in label order (its error, 1e-10, is far below fp32's)
    order, end = torch.argsort(lab), torch.cumsum(size, 0)

    def mean(v):
        cols = []
        for col in v.t():
            run = torch.cumsum(col.double()[order], 0)
            total = torch.where(end > 0, run[(end - 1).clamp(min=0)], 0.0)
            cols.append(torch.diff(total, prepend=total.new_zeros(1)))
        return torch.stack(cols, 1) / size[:, None].clamp(min=1)
    def whole(rows, kept):
        return _keep(torch.full_like(kept, -1, dtype=rows.dtype), rows)
    out = dict(size=whole(size, s["size"]),
               mean=whole(mean(s["emb"]), s["mean"]))
    return dict(out, centroid=whole(mean(s["xyz"]), s["centroid"])) \
        if c["xyz"] else out


def _exact_purity(s):
    lab, cls, nc, n_cls = (s["labels"].long(), s["cls"].long(), s["n_comp"],
                           s["n_cls"])
    pair, count = torch.unique(lab * n_cls + cls, return_counts=True)
    comp, y = pair // n_cls, pair % n_cls
    # the largest count, then the smallest class
    best = torch.zeros(nc, dtype=torch.int64, device=DEV).scatter_reduce_(
        0, comp, count * n_cls + (n_cls - 1 - y), "amax")
    major = torch.where(best > 0, n_cls - 1 - best % n_cls, best * 0 - 1)
    pred = major[lab]
    gt, pr = (torch.bincount(v, minlength=n_cls) for v in (cls, pred))
    tp = torch.bincount(cls[pred == cls], minlength=n_cls)
    iou = torch.where(gt > 0, tp.double() / (gt + pr - tp).clamp(min=1),
                      math.nan)
    present = int((gt > 0).sum())
    return dict(miou=float(iou.nansum()) / present,
                purity=int(tp.sum()) / lab.shape[0], n_present=present,
                majority=_keep(s["majority"].long(), major), iou=iou)


def _exact_mlp(s):
    h = s["x"].double()
    for j in (1, 2, 3):
        h = h @ s["w%d" % j].double() + s["b%d" % j].double()
        if j < 3:  # hidden activations are bf16 by definition
            h = h.clamp(min=0).to(torch.bfloat16).double()
    return dict(out=h)


def exact(case, seed):
    op = case["op"]
    if op in ("partition", "from_knn", "grid") or \
            (op == "knn" and (not case["d2"] or case["n"] > 400_000)):
        return None  # whole numbers; a level's energy needs the whole ladder
    s = prepare(case, seed)
    if op == "knn":
        return _exact_knn(s, case)
    if op == "loss":
        return _exact_loss(s, case)
    if op == "stats":
        return _exact_stats(s, case)
    if op == "purity":
        return _exact_purity(s)
    return _exact_mlp(s)
