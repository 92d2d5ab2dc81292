"""Timed cases: what a program that uses this library has it do.

A case names a kind of use, a mesh size, a number of segments and the options of
the call; its inputs follow from the case and a seed.  Meshes are heightfields
over the unit square (four random waves plus noise, as the library's own
workloads use), some with a band folded into an overhang.  Segments are drawn

  box        both ends uniform in the mesh box inflated by 10%
  crossing   half of them from above the surface to below it, the rest on one side
  adversarial  75% box, 20% aimed within 1e-7 of shared edges and vertices, 5%
             within 1e-6 rad of a triangle's plane

Kinds of use:

  query      a mesh that the program keeps, and one call with new segments
  step       a mesh that changes: build, intersect, destroy
  points     a step and then the distances and points of the hits
  one_call   the paper's test(vertices, triangles, from, to) usage
  batch      many meshes and their segments, built and intersected together
  learned    a kept mesh with a trained proposal, segments in proposal order
  train      training of the proposal from new segments

The diagnostic counters that come with every intersection are not among the
outputs here: by their description they may vary from call to call.
"""
import math

import numpy as np
import torch

import paper_2305_01867_amd as rsi


# ------------------------------------------------------------------ cases
def listed():
    return [
        # the smallest calls: a kept mesh asked with a few thousand segments, as
        # an interactive or per-frame caller does; the launches are the cost
        dict(name="tiny_query", kind="query", grid=64, fold=False, rays=10_000, law="crossing", mode="first_hit",
             precision="certified", algorithm="radix_tree", order="input"),
        # the same size through the one-call usage: build, intersect and free
        dict(name="tiny_one_call", kind="one_call", grid=64, fold=False, rays=10_000, law="crossing", mode="boolean",
             precision="certified"),
        # the paper's size and its boolean mode, mesh rebuilt: the headline step
        dict(name="paper_step", kind="step", grid=128, fold=False, rays=10_000_000, law="box", mode="boolean",
             precision="certified", algorithm="restructured", order="input"),
        # the paper's barycentric result: triangles, coordinates, distances and points
        dict(name="paper_points", kind="points", grid=128, fold=False, rays=600_011, law="box",
             mode="barycentric", precision="certified", algorithm="radix_tree", order="input"),
        # the paper's intercept count (inside / outside questions) on a kept mesh
        dict(name="paper_count", kind="query", grid=128, fold=False, rays=4_000_037, law="box",
             mode="intercept_count", precision="certified", algorithm="restructured", order="input"),
        # every option at its default: binary32 decisions, radix tree
        dict(name="plain_defaults", kind="query", grid=128, fold=False, rays=500_009, law="box", mode="barycentric",
             precision="plain", algorithm="radix_tree", order="input"),
        # segments aimed at edges and vertices of a folded surface: many
        # pairs that binary32 cannot decide
        dict(name="precision_nearest", kind="query", grid=256, fold=True, rays=2_500_000, law="adversarial",
             mode="first_hit", precision="certified", algorithm="restructured", order="input"),
        # a large mesh that changes, asked with few segments: the build is the cost
        dict(name="large_build", kind="step", grid=512, fold=False, rays=100_003, law="crossing", mode="first_hit",
             precision="certified", algorithm="restructured", order="input"),
        # 64 uneven meshes with 1e4 .. 1e6 segments each, one build and one launch
        dict(name="batch_full", kind="batch", meshes=64, tri_lo=2_000, tri_hi=200_000, ray_lo=10_000,
             ray_hi=1_000_000, sizes=40, mode="boolean", precision="certified", order="input"),
        # a few small meshes with odd sizes, nearest points wanted
        dict(name="batch_small", kind="batch", meshes=7, tri_lo=200, tri_hi=20_000, ray_lo=100, ray_hi=10_000,
             sizes=5, mode="barycentric", precision="certified", order="input"),
        # a large kept mesh with its trained proposal
        dict(name="learned_query", kind="learned", grid=512, fold=False, rays=2_000_003, law="crossing",
             mode="boolean", precision="certified", algorithm="restructured", order="input"),
        # training of the proposal (labelling, then one epoch of minibatches)
        dict(name="train", kind="train", grid=128, fold=False, rays=600_011, law="box", epochs=1, batch=4096,
             algorithm="radix_tree"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["query", "query", "query", "step", "step", "points", "one_call", "batch", "batch", "learned", "train"])
    if kind == "batch":
        meshes = rng.randint(2, 64)
        ray_hi = _log(rng, 1_000, 500_000)
        tri_hi = _log(rng, 1_000, 100_000)
        return dict(kind=kind, meshes=meshes, tri_lo=max(8, tri_hi // 50), tri_hi=tri_hi, ray_lo=max(1, ray_hi // 100),
                    ray_hi=ray_hi, sizes=rng.randint(0, 9999),
                    mode=rng.choice(["boolean", "first_hit", "barycentric", "intercept_count"]),
                    precision=rng.choice(["certified", "certified", "plain"]),
                    order=rng.choice(["input", "input", "midpoint"]))
    grid = _log(rng, 6, 512)
    rays = _log(rng, 1_000, 4_000_000)
    if kind == "train":
        return dict(kind=kind, grid=_log(rng, 40, 300), fold=False, rays=_log(rng, 20_000, 250_000),
                    law=rng.choice(["box", "crossing"]), epochs=rng.randint(1, 2), batch=rng.choice([2048, 4096, 6000]),
                    algorithm="radix_tree")
    if kind == "learned":
        return dict(kind=kind, grid=_log(rng, 40, 512), fold=rng.random() < 0.3, rays=_log(rng, 2_000, 1_900_000),
                    law=rng.choice(["box", "crossing"]), mode=rng.choice(["boolean", "boolean", "first_hit"]),
                    precision="certified", algorithm="restructured", order="input")
    precision = rng.choice(["certified", "certified", "plain"])
    # plain precision is not for segments that lie in a triangle's plane or on
    # an edge: whether binary32 sees such a pair depends on the boxes around it
    law = rng.choice(["box", "box", "crossing"] + ["adversarial"] * (precision == "certified"))
    case = dict(kind=kind, grid=grid, fold=rng.random() < 0.3, rays=rays, law=law,
                mode=rng.choice(["boolean", "boolean", "first_hit", "barycentric", "intercept_count"]),
                precision=precision)
    if kind == "points":
        case["mode"] = "barycentric"
    elif kind == "one_call" and case["mode"] == "barycentric":
        case["mode"] = "first_hit"  # its compacted barycentric lists have no fixed length: see points
    if kind != "one_call":
        case["algorithm"] = rng.choice(["restructured", "restructured", "radix_tree"])
        case["order"] = rng.choice(["input", "input", "input", "origin_octant"])
    return case


# ------------------------------------------------------------------ inputs
def _heightfield(n, rng, gen, fold):
    """Vertices float32 [n n, 3] and triangles int32 [2 (n-1)^2, 3] of one surface."""
    kw = dict(device="cuda", dtype=torch.float64)
    g = torch.arange(n, **kw) / (n - 1)
    y, x = torch.meshgrid(g, g, indexing="ij")
    z = 0.005 * torch.randn(n, n, generator=gen, **kw)
    for _ in range(4):
        fx, fy, phi = rng.uniform(1.0, 6.0), rng.uniform(1.0, 6.0), rng.uniform(0.0, 2.0 * math.pi)
        z = z + 0.1 * torch.sin(2.0 * math.pi * (fx * x + fy * y) + phi)
    if fold:
        # a band in x runs backwards and the part behind it is lifted: an overhang
        c, w = rng.uniform(0.3, 0.7), 0.05
        u = ((x - c + w) / (2 * w)).clamp(0.0, 1.0)
        z = z + 0.2 * u * u * (3 - 2 * u)
        back = x - 1.5 * w / math.pi * torch.sin(math.pi * (x - c) / w)
        x = torch.where((x - c).abs() < w, back, x)
    V = torch.stack([x, y, z], 2).reshape(-1, 3).float()
    i = torch.arange(n - 1, device="cuda")
    v = (i[:, None] * n + i[None, :]).reshape(-1)
    a, b, c2, d = v, v + 1, v + n + 1, v + n
    F = torch.stack([torch.stack([a, b, c2], 1), torch.stack([a, c2, d], 1)], 1).reshape(-1, 3).int()
    return V.contiguous(), F.contiguous()


def _uniform(gen, *shape):
    return torch.rand(*shape, generator=gen, device="cuda", dtype=torch.float64)


def _box(V, m, gen):
    lo, hi = V.min(0).values.double(), V.max(0).values.double()
    c, h = 0.5 * (lo + hi), 0.55 * (hi - lo)
    return c + h * (2 * _uniform(gen, m, 3) - 1), c + h * (2 * _uniform(gen, m, 3) - 1)


def _crossing(m, gen):
    xy, z, pick = _uniform(gen, m, 4), 0.3 * _uniform(gen, m, 4), _uniform(gen, m, 2) < 0.5
    above0, above1, below0, below1 = 0.5 + z[:, 0], 0.5 + z[:, 1], -z[:, 2], -z[:, 3]
    z0 = torch.where(pick[:, 0] | pick[:, 1], above0, below0)
    z1 = torch.where(~pick[:, 0] & pick[:, 1], above1, below1)
    return torch.cat([xy[:, :2], z0[:, None]], 1), torch.cat([xy[:, 2:], z1[:, None]], 1)


def _adversarial(V, F, m, gen):
    O, E = _box(V, m, gen)
    P, T = V.double(), F.long()
    t = (_uniform(gen, m) * len(T)).long()
    A, B, C = P[T[t, 0]], P[T[t, 1]], P[T[t, 2]]
    u = _uniform(gen, m)
    unit = lambda x: x / x.norm(dim=1, keepdim=True)  # noqa: E731
    g = unit(torch.randn(m, 3, generator=gen, device="cuda", dtype=torch.float64))
    # aimed at a shared edge (the diagonal from A) or, one in four, at a vertex
    lam = 0.05 + 0.9 * _uniform(gen, m)
    on_edge = torch.where((_uniform(gen, m) < 0.25)[:, None], A, A + lam[:, None] * (C - A))
    on_edge = on_edge + g * ((2 * _uniform(gen, m) - 1) * 1e-7 * on_edge.abs().amax(1))[:, None]
    d = unit(torch.randn(m, 3, generator=gen, device="cuda", dtype=torch.float64))
    d[:, 2] = torch.where(d[:, 2].abs() < 0.3, torch.where(d[:, 2] < 0, -0.3, 0.3).double(), d[:, 2])
    d = unit(d)
    h = 0.05 + 0.45 * _uniform(gen, m)[:, None]
    # nearly in the plane of a triangle
    nrm = unit(torch.linalg.cross(B - A, C - A))
    flat = unit(g - nrm * (g * nrm).sum(1, keepdim=True))
    th = 1e-6 * _uniform(gen, m)[:, None]
    w = _uniform(gen, m, 3) + 0.01
    w = w / w.sum(1, keepdim=True)
    inside = w[:, :1] * A + w[:, 1:2] * B + w[:, 2:] * C + nrm * ((2 * _uniform(gen, m) - 1) * 1e-7)[:, None]
    dp = torch.cos(th) * flat + torch.sin(th) * nrm
    hp = 0.01 + 0.09 * _uniform(gen, m)[:, None]
    edge, plane = (u < 0.20)[:, None], ((u >= 0.20) & (u < 0.25))[:, None]
    O = torch.where(edge, on_edge - h * d, torch.where(plane, inside - hp * dp, O))
    E = torch.where(edge, on_edge + h * d, torch.where(plane, inside + hp * dp, E))
    return O, E


def _segments(V, F, m, law, gen, part=1 << 21):
    """Start and end points float32 [m, 3], drawn a part at a time."""
    O = torch.empty(m, 3, device="cuda")
    E = torch.empty(m, 3, device="cuda")
    for s in range(0, m, part):
        k = min(part, m - s)
        o, e = _box(V, k, gen) if law == "box" else _crossing(k, gen) if law == "crossing" else \
            _adversarial(V, F, k, gen)
        O[s:s + k], E[s:s + k] = o, e
    return O, E


def _inputs(case, seed):
    rng = np.random.default_rng([seed, 7])
    gen = torch.Generator("cuda").manual_seed(seed)
    if case["kind"] != "batch":
        V, F = _heightfield(case["grid"], rng, gen, case["fold"])
        return V, F, *_segments(V, F, case["rays"], case["law"], gen)
    grids, rays = _batch_sizes(case)
    parts = []
    for n, m in zip(grids, rays):
        V, F = _heightfield(n, rng, gen, False)
        parts.append((V, F, *_segments(V, F, m, "box", gen)))
    return tuple(torch.cat(p) for p in zip(*parts))


def _batch_sizes(case):
    """Grid size and number of segments of each mesh, spread over their logarithms."""
    rng = np.random.default_rng(case["sizes"])
    spread = lambda lo, hi: np.exp(rng.uniform(np.log(lo), np.log(hi), case["meshes"]))  # noqa: E731
    tris, rays = spread(case["tri_lo"], case["tri_hi"]), spread(case["ray_lo"], case["ray_hi"])
    return [max(2, int(round(math.sqrt(t / 2))) + 1) for t in tris], [max(1, int(round(r))) for r in rays]


def _offsets(case):
    grids, rays = _batch_sizes(case)
    total = lambda x: np.concatenate([[0], np.cumsum(x)]).astype(np.int64)  # noqa: E731
    return total([n * n for n in grids]), total([2 * (n - 1) ** 2 for n in grids]), total(rays)


# ------------------------------------------------------------------ the calls
def prepare(case, seed):
    V, F, O, E = _inputs(case, seed)
    kind = case["kind"]
    s = dict(case, O=O, E=E)
    if kind in ("step", "points", "one_call", "batch"):
        s.update(V=V, F=F)
    if kind in ("query", "learned", "train"):
        s["mesh"] = rsi.rsi_build(V, F, algorithm=case["algorithm"])
    if kind == "learned":
        # trained once, on other segments of the same law
        gen = torch.Generator("cuda").manual_seed(seed + 1_000_003)
        rsi.rsi_proposal_train(s["mesh"], *_segments(V, F, 200_000, case["law"], gen), epochs=1)
    if kind == "batch":
        s["batch"] = rsi.rsi_batch_create(*_offsets(case))
    return s


OUTPUTS = {"boolean": ("hit",), "first_hit": ("tri_id",), "barycentric": ("tri_id", "uvt"),
           "intercept_count": ("count",)}


def run(s):
    kind = s["kind"]
    if kind == "train":
        loss, n = rsi.rsi_proposal_train(s["mesh"], s["O"], s["E"], epochs=s["epochs"], batch=s["batch"], reinit=True)
        return {"loss": loss, "labelled": n, "params": rsi.rsi_proposal_params(s["mesh"])}
    if kind == "one_call":
        return rsi.rsi_test(s["V"], s["F"], s["O"], s["E"], mode=s["mode"], precision=s["precision"])
    opts = dict(mode=s["mode"], precision=s["precision"], ray_sort=s["order"])
    if kind == "batch":
        rsi.rsi_batch_build(s["batch"], s["V"], s["F"])
        r = rsi.rsi_batch_intersect(s["batch"], s["O"], s["E"], **opts)
    elif kind in ("step", "points"):
        with rsi.rsi_build(s["V"], s["F"], algorithm=s["algorithm"]) as mesh:
            r = rsi.rsi_intersect(mesh, s["O"], s["E"], **opts)
        if kind == "points":
            return {k: r[k] for k in OUTPUTS["barycentric"]} | rsi.rsi_derive(s["O"], s["E"], r)
    else:
        r = rsi.rsi_intersect(s["mesh"], s["O"], s["E"], proposal=kind == "learned", **opts)
    return {k: r[k] for k in OUTPUTS[s["mode"]]}


# ------------------------------------------------------------------ what a pass cannot do without
OUT_BYTES = {"boolean": 1, "first_hit": 4, "barycentric": 16, "intercept_count": 4}
NET_FLOPS = 2 * (224 * 256 + 3 * 256 * 256)  # the proposal's four layers, per segment


def work(case):
    """Each segment and each vertex and triangle read once, each result written
    once; per segment its set-up and one triangle test (about 100 operations);
    the network's products where it runs."""
    if case["kind"] == "batch":
        grids, rays = _batch_sizes(case)
        rays = sum(rays)
    else:
        grids, rays = [case["grid"]], case["rays"]
    mesh = sum(12 * n * n + 24 * (n - 1) ** 2 for n in grids)
    flops = 100 * rays
    if case["kind"] == "train":  # forward, and products of the same size for both gradients
        return {"bytes": 24 * rays + mesh + 4 * 254976, "flops": flops + 3 * NET_FLOPS * rays * case["epochs"]}
    if case["kind"] == "learned":
        flops += NET_FLOPS * rays
    out = OUT_BYTES[case["mode"]] + (16 if case["kind"] == "points" else 0)
    return {"bytes": (24 + out) * rays + mesh, "flops": flops}


# ------------------------------------------------------------------ the same in 64 bits
def _nearest(V, F, O, E, pairs=1 << 26):
    """Every segment against every triangle: u, v, t of the nearest hit (NaN on a miss)."""
    V, O, E = V.double(), O.double(), E.double()
    A, B, C = (V[F[:, k].long()] for k in range(3))
    e1, e2 = B - A, C - A
    ids = torch.arange(len(F), device=V.device)
    cross = lambda a, b: (a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0])  # noqa: E731
    dot = lambda a, b: a[0] * b[0] + a[1] * b[1] + a[2] * b[2]  # noqa: E731
    rows = lambda x: [x[None, :, k] for k in range(3)]  # noqa: E731
    found = []
    for o, e in zip(O.split(max(1, pairs // len(F))), E.split(max(1, pairs // len(F)))):
        d = [(e - o)[:, k, None] for k in range(3)]
        s = [o[:, k, None] - A[None, :, k] for k in range(3)]
        p, q = cross(d, rows(e2)), cross(s, rows(e1))
        det = dot(rows(e1), p)
        u, v, t = dot(s, p), dot(d, q), dot(rows(e2), q)
        del s, p, q
        g = det.sign()
        u, v, t, det = g * u, g * v, g * t, g * det
        hit = (det > 0) & (u >= 0) & (v >= 0) & (u + v <= det) & (t >= 0) & (t <= det)
        tt = torch.where(hit, t / det, math.inf)
        best = tt.min(1, keepdim=True).values
        k = torch.where(tt == best, ids, len(F)).min(1).values
        miss = ~torch.isfinite(best[:, 0])
        k = torch.where(miss, 0, k)[:, None]
        uvt = torch.cat([(x / det).gather(1, k) for x in (u, v, t)], 1)
        uvt[miss] = math.nan
        found.append(uvt)
    return torch.cat(found)


def exact(case, seed):
    if case.get("mode") != "barycentric":
        return None  # flags, triangles and counts are whole numbers; training has no such value
    grids, rays = _batch_sizes(case) if case["kind"] == "batch" else ([case["grid"]], [case["rays"]])
    if sum(2 * (n - 1) ** 2 * m for n, m in zip(grids, rays)) > 2.5e10:
        return None
    V, F, O, E = _inputs(case, seed)
    if case["kind"] == "batch":
        v, f, r = _offsets(case)
        parts = [_nearest(V[v[k]:v[k + 1]], F[f[k]:f[k + 1]], O[r[k]:r[k + 1]], E[r[k]:r[k + 1]])
                 for k in range(len(grids))]
        return {"tri_id": None, "uvt": torch.cat(parts)}
    uvt = _nearest(V, F, O, E)
    if case["kind"] != "points":
        return {"tri_id": None, "uvt": uvt}
    d = E.double() - O.double()
    return {"tri_id": None, "uvt": uvt, "distance": uvt[:, 2] * d.norm(dim=1), "point": O + uvt[:, 2:] * d}
