"""What a program asks of this framework, as timed cases.

A case is a dict of plain values; `prepare` makes what the program has in hand
(meshes on the GPU, resident blobs, workspaces) from a seed, and `run` is one
pass through the public entry points.  The shapes are the repository's own
workloads (tiny, pathology, batching, precision stress, serving, mesh
complexity, containment, cubes), drawn on the GPU because inputs are made often.

Kinds of pass:
  join      resident datasets: filter -> refine -> compact, the host reading
            each count (the module's documented use), optionally under a query box
  step      the same chain with the counts handed on inside the device and one
            read at the end, workspaces kept (a program that repeats a join)
  refine    a given candidate list: refine -> compact, workspaces kept
  predicate one join predicate over a given candidate list
  fresh     meshes that have just arrived: build both blobs, then join them
  serve     a burst of query boxes through the continuous-batching server
  dataset   the dataset-level join (one tree per dataset, records deduplicated)
"""
import math

import numpy as np
import torch

import paper_2609_24513_amd as pa
from paper_2609_24513_amd import dataset, serve, synth

# ---------------------------------------------------------------------------
# Meshes, drawn on the GPU
# ---------------------------------------------------------------------------


class Meshes:
    """A dataset: verts f32[V, 3], faces i32[F, 3] (mesh-local), offsets i64[M + 1]."""

    def __init__(self, verts, faces, vert_off, face_off):
        self.verts, self.faces, self.vert_off, self.face_off = verts, faces, vert_off, face_off

    @property
    def n_meshes(self):
        return int(self.vert_off.shape[0] - 1)

    def numpy(self):
        return synth.MeshSet(*(t.cpu().numpy() for t in (self.verts, self.faces, self.vert_off, self.face_off)))


_templates = {}


def _template(kind, *size):
    """A unit surface's vertices (f64) and faces on the GPU; the same for every seed."""
    key = (kind,) + size
    if key not in _templates:
        if kind == "ico":
            v, f = synth.icosphere(*size)
        elif kind == "geo":
            v, f = synth.geodesic_sphere(*size)
        elif kind == "uv":
            v, f = synth.uv_sphere(*size)
        elif kind == "tube":
            line = np.array([[0.0, 0, 0], [1, 0, 0], [2, 0, 0], [3, 0, 0]])
            v, f = synth.capped_tube(line, 1.0, *size)
        else:
            v = [[x, y, z] for x in (0, 1) for y in (0, 1) for z in (0, 1)]
            f = [[0, 1, 3], [0, 3, 2], [4, 6, 7], [4, 7, 5], [0, 4, 5], [0, 5, 1], [2, 3, 7], [2, 7, 6], [0, 2, 6],
                 [0, 6, 4], [1, 5, 7], [1, 7, 3]]
        _templates[key] = (torch.as_tensor(np.asarray(v, np.float64)).cuda(),
                           torch.as_tensor(np.asarray(f, np.int32)).cuda())
    return _templates[key]


def _rng(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _noisy(g, v, r, amp):
    """Spheres of radii r [m] on unit directions v [V, 3]: amp > 0 a low-frequency field of
    eight plane waves, amp < 0 independent radial jitter of that relative deviation."""
    m = r.shape[0]
    if amp < 0:
        rad = r[:, None] * (1.0 - amp * torch.randn(m, v.shape[0], generator=g, device="cuda", dtype=torch.float64))
        return rad[:, :, None] * v
    if amp == 0:
        return r[:, None, None] * v
    k = torch.randn(m, 8, 3, generator=g, device="cuda", dtype=torch.float32)
    k = k / k.norm(dim=2, keepdim=True) * torch.randint(1, 3, (m, 8, 1), generator=g, device="cuda")
    ph = 2 * math.pi * torch.rand(m, 8, generator=g, device="cuda")
    out = torch.empty(m, v.shape[0], 3, dtype=torch.float32, device="cuda")
    v32 = v.float()
    step = max(1, (1 << 25) // (8 * v.shape[0]))
    for a in range(0, m, step):
        b = min(m, a + step)
        n = torch.sin(2 * math.pi * (v32 @ k[a:b].reshape(-1, 3).T).reshape(-1, b - a, 8) + ph[None, a:b]).sum(2).T
        n = n / n.abs().amax(dim=1, keepdim=True)
        out[a:b] = (r[a:b, None].float() * (1.0 + amp * n))[:, :, None] * v32
    return out


def _tubes(g, m, rings, sides, reach):
    """m tubes swept along random cubic Beziers with rotation-minimising frames, centred at 0.
    Every control step goes forward along the tube's direction, so that no ring folds onto another."""
    way = torch.randn(m, 1, 3, generator=g, device="cuda", dtype=torch.float64)
    way = way / way.norm(dim=2, keepdim=True) * _uniform(g, 0.5, 1.0, m, 3, 1)
    steps = reach * (way + _uniform(g, -0.35, 0.35, m, 3, 3))
    ctrl = torch.cat([torch.zeros(m, 1, 3, device="cuda", dtype=torch.float64), steps.cumsum(1)], 1)
    ctrl = ctrl - ctrl.mean(1, keepdim=True)
    rho = _uniform(g, 2.0, 6.0, m)
    t = torch.linspace(0, 1, rings, device="cuda", dtype=torch.float64)
    s = 1 - t
    w = torch.stack([s ** 3, 3 * s * s * t, 3 * s * t * t, t ** 3], 1)
    d = torch.stack([3 * s * s, 6 * s * t, 3 * t * t], 1)
    pts = w @ ctrl
    tan = d @ (ctrl[:, 1:] - ctrl[:, :-1])
    tan = tan / tan.norm(dim=2, keepdim=True)
    axis = torch.eye(3, device="cuda", dtype=torch.float64)[tan[:, 0].abs().argmin(1)]
    r = axis - tan[:, 0] * (axis * tan[:, 0]).sum(1, keepdim=True)
    frames = [r / r.norm(dim=1, keepdim=True)]
    for i in range(rings - 1):
        v1 = pts[:, i + 1] - pts[:, i]
        c1 = (v1 * v1).sum(1, keepdim=True)
        rl = frames[-1] - 2 / c1 * (v1 * frames[-1]).sum(1, keepdim=True) * v1
        tl = tan[:, i] - 2 / c1 * (v1 * tan[:, i]).sum(1, keepdim=True) * v1
        v2 = tan[:, i + 1] - tl
        c2 = (v2 * v2).sum(1, keepdim=True).clamp_min(1e-300)
        rn = rl - 2 / c2 * (v2 * rl).sum(1, keepdim=True) * v2
        rn = rn - tan[:, i + 1] * (rn * tan[:, i + 1]).sum(1, keepdim=True)
        frames.append(rn / rn.norm(dim=1, keepdim=True))
    R = torch.stack(frames, 1)
    Q = torch.linalg.cross(tan, R)
    a = 2 * math.pi * torch.arange(sides, device="cuda", dtype=torch.float64) / sides
    ring = a.cos()[:, None] * R[:, :, None] + a.sin()[:, None] * Q[:, :, None]
    v = (pts[:, :, None] + rho[:, None, None, None] * ring).reshape(m, -1, 3)
    return torch.cat([v, pts[:, :1], pts[:, -1:]], 1)


def _gather(parts, centres, perm):
    """One dataset of `parts` [(verts [m, V, 3], faces [F, 3])], the k-th mesh moved to
    centres[k] and stored at place perm[k]."""
    nv = torch.cat([torch.full((v.shape[0],), v.shape[1], dtype=torch.int64) for v, _ in parts]).cuda()
    nf = torch.cat([torch.full((v.shape[0],), f.shape[0], dtype=torch.int64) for v, f in parts]).cuda()
    M = nv.shape[0]
    zero = torch.zeros(1, dtype=torch.int64, device="cuda")
    vo = torch.cat([zero, torch.empty_like(nv).scatter_(0, perm, nv).cumsum(0)])
    fo = torch.cat([zero, torch.empty_like(nf).scatter_(0, perm, nf).cumsum(0)])
    verts = torch.empty(sum(v.shape[0] * v.shape[1] for v, _ in parts), 3, dtype=torch.float32, device="cuda")
    faces = torch.empty(sum(v.shape[0] * f.shape[0] for v, f in parts), 3, dtype=torch.int32, device="cuda")
    k = 0
    for v, f in parts:
        m, V, F = v.shape[0], v.shape[1], f.shape[0]
        at = perm[k:k + m]
        vi = (vo[at][:, None] + torch.arange(V, device="cuda")).reshape(-1)
        fi = (fo[at][:, None] + torch.arange(F, device="cuda")).reshape(-1)
        verts[vi] = (v.double() + centres[k:k + m, None]).float().reshape(-1, 3)
        faces[fi] = f[None].expand(m, F, 3).reshape(-1, 3)
        k += m
    assert k == M
    return Meshes(verts, faces, vo, fo)


def _plain(verts, faces, centres):
    m = verts.shape[0]
    return _gather([(verts, faces)], centres, torch.arange(m, device="cuda"))


def _boxes(S):
    """Exact mesh boxes f32[M, 6]."""
    n = S.vert_off.diff()
    own = torch.repeat_interleave(torch.arange(S.n_meshes, device="cuda"), n)[:, None].expand(-1, 3)
    out = torch.empty(S.n_meshes, 6, device="cuda")
    lo = torch.full((S.n_meshes, 3), math.inf, device="cuda").scatter_reduce_(0, own, S.verts, "amin")
    hi = torch.full((S.n_meshes, 3), -math.inf, device="cuda").scatter_reduce_(0, own, S.verts, "amax")
    out[:, :3], out[:, 3:] = lo, hi
    return out


def _candidates(a, b):
    """Pairs of boxes that overlap (closed), sorted, int32 [P, 2]."""
    got = []
    for r in range(0, a.shape[0], 1024):
        x = a[r:r + 1024, None]
        ok = ((x[..., :3] <= b[None, :, 3:]) & (b[None, :, :3] <= x[..., 3:])).all(2)
        hit = ok.nonzero()
        hit[:, 0] += r
        got.append(hit)
    return torch.cat(got).to(torch.int32)


def _thin(g, pairs, n):
    """n of the candidate pairs, in order (all of them where there are no more)."""
    if pairs.shape[0] <= n:
        return pairs.contiguous()
    keep = torch.randperm(pairs.shape[0], generator=g, device="cuda")[:n].sort().values
    return pairs[keep].contiguous()


# ---- the datasets ----------------------------------------------------------


def _icospheres(g, n, level, side):
    """Jittered level-`level` icospheres, r~U[0.8, 1.2], in a cube (tiny and serving workloads)."""
    v, f = _template("ico", level)
    return _plain(_noisy(g, v, _uniform(g, 0.8, 1.2, n), -0.02), f, _uniform(g, 0.0, side, n, 3))


def _tissue(g, nuclei, vessels):
    """Nuclei (noise-displaced level-4 icospheres) and vessels (64 x 32 tubes) at the
    pathology workload's density (10,000 x 1,000 in a cube of side 1,000)."""
    side = 1000.0 * (nuclei / 10_000) ** (1 / 3)
    v, f = _template("ico", 4)
    A = _plain(_noisy(g, v, _uniform(g, 3.0, 8.0, nuclei), 0.15), f, _uniform(g, 0.0, side, nuclei, 3))
    _, tf = _template("tube", 64, 32)
    B = _plain(_tubes(g, vessels, 64, 32, 100.0), tf, _uniform(g, 0.0, side, vessels, 3))
    return A, B


def _class_sizes(f_lo, f_hi, classes):
    return [f_lo * (f_hi / f_lo) ** ((k + 0.5) / classes) for k in range(classes)]


def _half_pool(g, n, f_lo, f_hi, classes=10):
    """n surfaces, half displaced geodesic spheres and half tubes, face counts spread over the
    logarithm of [f_lo, f_hi], in mixed order and centred at 0."""
    parts = []
    for k, ft in enumerate(_class_sizes(f_lo, f_hi, classes)):
        m = n * (k + 1) // classes - n * k // classes
        ms = m // 2
        if ms:
            v, f = _template("geo", max(2, round(math.sqrt(ft / 20))))
            parts.append((_noisy(g, v, _uniform(g, 3.0, 8.0, ms), 0.15), f))
        if m - ms:
            sides = max(4, round(math.sqrt(ft / 4)))
            rings = max(2, round(ft / (2 * sides)))
            _, f = _template("tube", rings, sides)
            parts.append((_tubes(g, m - ms, rings, sides, 40.0), f))
    return parts, torch.randperm(n, generator=g, device="cuda")


def _pool(g, meshes, n_pairs, f_lo, f_hi):
    """Batching workload: two half pools in a cube of the side at which a little over n_pairs
    candidates overlap."""
    na = meshes // 2
    pa_, perm_a = _half_pool(g, na, f_lo, f_hi)
    pb_, perm_b = _half_pool(g, meshes - na, f_lo, f_hi)
    ca, cb = _uniform(g, 0.0, 1.0, na, 3), _uniform(g, 0.0, 1.0, meshes - na, 3)

    def place(parts, c):
        lo = torch.cat([v.amin(1).double() for v, _ in parts])
        hi = torch.cat([v.amax(1).double() for v, _ in parts])
        return torch.cat([lo + c, hi + c], 1)

    lo, hi = 1.0, 4096.0
    for _ in range(16):
        side = math.sqrt(lo * hi)
        got = _candidates(place(pa_, ca * side), place(pb_, cb * side)).shape[0]
        if n_pairs * 1.01 + 2 <= got <= n_pairs * 1.1 + 8:
            break
        lo, hi = (side, hi) if got > n_pairs * 1.1 + 8 else (lo, side)
    A, B = _gather(pa_, ca * side, perm_a), _gather(pb_, cb * side, perm_b)
    return A, B, _thin(g, _candidates(_boxes(A), _boxes(B)), n_pairs)


def _touching(g, n):
    """Precision stress: pairs of level-4 icospheres on a 2^-10 grid: 30 % tangent, 20 % with a
    coplanar face, 10 % with a vertex on a face, 40 % at a random distance."""
    step = 2.0 ** -10
    v, f = _template("ico", 4)
    ra, rb = _uniform(g, 0.8, 1.2, n), _uniform(g, 0.8, 1.2, n)
    va = torch.round(ra[:, None, None] * v / step) * step
    vb = torch.round(rb[:, None, None] * v / step) * step
    cls = torch.rand(n, generator=g, device="cuda")
    row = torch.arange(n, device="cuda")
    # tangent: an extreme vertex of B on the opposite extreme vertex of A
    ax = torch.randint(0, 3, (n,), generator=g, device="cuda")
    sg = torch.randint(0, 2, (n,), generator=g, device="cuda").double() * 2 - 1
    along = lambda x: torch.gather(x, 2, ax[:, None, None].expand(-1, x.shape[1], 1))[..., 0] * sg[:, None]  # noqa: E731
    tangent = va[row, along(va).argmax(1)] - vb[row, along(vb).argmin(1)]
    # a face of A: B mirrored through a point of it, or B's extreme vertex put on it
    fv = f[torch.randint(0, f.shape[0], (n,), generator=g, device="cuda")].long()
    a, b, c = (va[row, fv[:, k]] for k in range(3))
    mid = a / 4 + b / 2 + c / 4
    nrm = torch.linalg.cross(b - a, c - a)
    on_face = (2 * a + b + c) / 4 - vb[row, (vb @ nrm[:, :, None])[..., 0].argmin(1)]
    d = torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64)
    d = d / d.norm(dim=1, keepdim=True) * (torch.rand(n, 1, generator=g, device="cuda") * (ra + rb + 0.2)[:, None])
    apart = torch.round(d / step) * step
    shift = torch.where((cls < 0.3)[:, None], tangent, torch.where((cls < 0.6)[:, None], on_face, apart))
    out = vb + shift[:, None]
    out = torch.where(((cls >= 0.3) & (cls < 0.5))[:, None, None], 2 * mid[:, None] - va, out)
    zero = torch.zeros(n, 3, device="cuda", dtype=torch.float64)
    pairs = torch.stack([row, row], 1).to(torch.int32)
    return _plain(va, f, zero), _plain(out, f, zero), pairs


def _sweep(g, n, rings):
    """Mesh complexity: unit UV spheres; A on a jittered lattice, a fifth of B crossing one of
    them, a fifth just apart with overlapping boxes, the rest anywhere."""
    per = math.ceil(n ** (1 / 3))
    cell = torch.arange(per ** 3, device="cuda")[torch.randperm(per ** 3, generator=g, device="cuda")[:n]]
    grid = torch.stack([cell // (per * per), cell // per % per, cell % per], 1).double()
    ca = 6.0 * (grid + 0.5) + _uniform(g, -1.0, 1.0, n, 3)
    u = torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64)
    u = u / u.norm(dim=1, keepdim=True)
    k = n // 5
    near = ca[:k] + u[:k] * _uniform(g, 0.3, 1.0, k, 1)
    apart = ca[k:2 * k] + u[k:2 * k] * _uniform(g, 2.05, 3.2, k, 1)
    rest = _uniform(g, 0.0, 6.0 * per, n - 2 * k, 3)
    v, f = _template("uv", rings, 2 * rings)
    v = v.float()[None].expand(n, -1, -1)
    return _plain(v, f, ca), _plain(v, f, torch.cat([near, apart, rest]))


def _nested(g, n, nu):
    """Containment: displaced spheres r~U[3, 8], and spheres r~U[0.3, 3] inside, across or beside them."""
    v, f = _template("geo", nu)
    ca = _uniform(g, 0.0, 20.0 * n ** (1 / 3), n, 3)
    ra = _uniform(g, 3.0, 8.0, n)
    A = _plain(_noisy(g, v, ra, 0.15), f, ca)
    u = torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64)
    u = u / u.norm(dim=1, keepdim=True)
    B = _plain(_noisy(g, v, _uniform(g, 0.3, 3.0, n), 0.15), f, ca + u * (ra * _uniform(g, 0.0, 1.3, n))[:, None])
    return A, B


def _cubes(g, n, side):
    v, f = _template("cube")
    out = []
    for _ in range(2):
        s = _uniform(g, 1.0, 2.0, n)
        out.append(_plain(s[:, None, None] * v, f, _uniform(g, 0.0, side, n, 3)))
    return out


def _datasets(case, g):
    """(A, B, pairs or None) of a case."""
    what, n = case["data"], case["n"]
    if what == "icospheres":
        # tiny: eight a side in a cube of 4; serving density beyond
        return _icospheres(g, n, 2, case["side"]), _icospheres(g, n, 2, case["side"]), None
    if what == "tissue":
        return (*_tissue(g, n, max(1, n // 10)), None)
    if what == "pool":
        return _pool(g, n, case["pairs"], case["f_lo"], case["f_hi"])
    if what == "touching":
        return _touching(g, n)
    if what == "sweep":
        return (*_sweep(g, n, case["rings"]), None)
    if what == "nested":
        A, B = _nested(g, n, case["nu"])
        return A, B, _thin(g, _candidates(_boxes(A), _boxes(B)), n)
    return (*_cubes(g, n, case["side"]), None)


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------


def listed():
    return [
        # the smallest join anyone makes: 8 x 8 spheres of 320 triangles, all launches and host calls
        {"name": "tiny_join", "kind": "join", "data": "icospheres", "n": 8, "side": 4.0, "width": 4, "leaf": 4},
        # one interactive query on the serving pool: a box that selects a few hundred pairs of 25,000 x 25,000
        {"name": "query_box", "kind": "join", "data": "icospheres", "n": 25_000, "side": 58.5, "query": 7.0,
         "width": 4, "leaf": 4},
        # the server under a burst: 96 query boxes selecting 0 ... 5,000 pairs each, batched 32 to a graph
        {"name": "serving_burst", "kind": "serve", "data": "icospheres", "n": 25_000, "side": 58.5, "requests": 96,
         "width": 4, "leaf": 4},
        # pathology: 10,000 nuclei against 1,000 vessels, the whole chain on the device, repeated
        {"name": "pathology_step", "kind": "step", "data": "tissue", "n": 10_000, "width": 4, "leaf": 4},
        # batching: 50,000 given pairs of a 4,096-mesh pool of 500 ... 100,000 triangles (headline workload)
        {"name": "batching_refine", "kind": "refine", "data": "pool", "n": 4096, "pairs": 50_000, "f_lo": 500.0,
         "f_hi": 100_000.0, "width": 8, "leaf": 1},
        # degenerate contacts: 2,000 pairs that touch exactly, the exact tiers at work
        {"name": "precision_stress", "kind": "refine", "data": "touching", "n": 2000, "width": 4, "leaf": 4},
        # few, very fine meshes: 500 x 500 spheres of 82,368 triangles, 100 crossing
        {"name": "fine_meshes", "kind": "step", "data": "sweep", "n": 500, "rings": 144, "width": 8, "leaf": 2},
        # containment join over an odd number of nested spheres
        {"name": "contains", "kind": "predicate", "data": "nested", "n": 4999, "nu": 13, "predicate": "contains",
         "width": 4, "leaf": 4},
        # a small dataset arriving: build 2 x 173 spheres of 320 triangles and join them
        {"name": "fresh_small", "kind": "fresh", "data": "icospheres", "n": 173, "side": 11.0, "width": 4, "leaf": 4},
        # a tissue sample arriving: build 1,000 nuclei and 100 vessels (5.5 M triangles) and join them
        {"name": "fresh_tissue", "kind": "fresh", "data": "tissue", "n": 1000, "width": 4, "leaf": 4},
        # loading the batching pool: 71 M triangles in meshes of 500 ... 100,000, built and joined
        {"name": "fresh_pool", "kind": "fresh", "data": "pool", "n": 4096, "pairs": 50_000, "f_lo": 500.0,
         "f_hi": 100_000.0, "width": 8, "leaf": 1},
        # the paper's dataset-level join of 50,000 x 50,000 cubes, table sized by the selectivity estimate
        {"name": "dataset_cubes", "kind": "dataset", "data": "cubes", "n": 50_000, "side": 63.0,
         "strategy": "estimated", "width": 4, "leaf": 4},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["join", "join", "serve", "step", "step", "refine", "refine", "predicate", "fresh", "fresh",
                       "dataset"])
    wl = rng.choice([{"width": 4, "leaf": 4}, {"width": 4, "leaf": 4}, {"width": 8, "leaf": 1},
                     {"width": 8, "leaf": 2}])
    if kind == "join" or kind == "serve":
        n = int(_log(rng, 3, 25_000) if kind == "join" else _log(rng, 3000, 25_000))
        c = {"kind": kind, "data": "icospheres", "n": n, "side": 2.0 * n ** (1 / 3), "width": 4, "leaf": 4}
        if kind == "serve":
            c["requests"] = int(_log(rng, 1, 96))
        elif n > 200:
            c["query"] = round(_log(rng, 1.0, 17.0), 3)
        return c
    if kind == "step":
        if rng.random() < 0.5:
            return {"kind": kind, "data": "tissue", "n": int(_log(rng, 300, 10_000)), **wl}
        rings = int(_log(rng, 4, 140))
        return {"kind": kind, "data": "sweep", "n": int(_log(rng, 50, 500)), "rings": rings, **wl}
    if kind == "refine":
        if rng.random() < 0.35:
            return {"kind": kind, "data": "touching", "n": int(_log(rng, 40, 2000)), **wl}
        n = int(_log(rng, 100, 4000))
        return {"kind": kind, "data": "pool", "n": n, "pairs": 12 * n, "f_lo": 500.0,
                "f_hi": round(_log(rng, 5000, 100_000)), **wl}
    if kind == "predicate":
        return {"kind": kind, "data": "nested", "n": int(_log(rng, 100, 8000)), "nu": rng.randint(4, 20),
                "predicate": rng.choice(["contains", "within", "intersection"]), **wl}
    if kind == "fresh":
        if rng.random() < 0.5:
            n = int(_log(rng, 3, 20_000))
            return {"kind": kind, "data": "icospheres", "n": n, "side": 2.0 * n ** (1 / 3), **wl}
        n = int(_log(rng, 60, 2000))
        return {"kind": kind, "data": "pool", "n": n, "pairs": 12 * n, "f_lo": 500.0,
                "f_hi": round(_log(rng, 5000, 100_000)), **wl}
    n = int(_log(rng, 2000, 50_000))
    return {"kind": kind, "data": "cubes", "n": n, "side": round(1.71 * n ** (1 / 3), 2),
            "strategy": rng.choice(["estimated", "two_pass"]), "width": 4, "leaf": 4}


# ---------------------------------------------------------------------------
# Passes
# ---------------------------------------------------------------------------


def _room(case):
    """Pairs that a program makes room for: more than the data's density gives."""
    n = case["n"]
    return {"icospheres": min(n * n, 12 * n + 1024), "tissue": 3 * n + 256, "pool": case.get("pairs", 0) * 5 // 4 + 64,
            "touching": n, "sweep": 2 * n + 256, "nested": n, "cubes": 9 * n}[case["data"]]


def _kept(n_pairs, width):
    """What a program that repeats a refinement keeps: workspace, statistics, status."""
    return {"ws": pa.refine_workspace(n_pairs, width, pa.RefineConfig()),
            "stats": torch.zeros(len(pa.STATS_FIELDS), dtype=torch.int64, device="cuda"),
            "status": torch.zeros(1, dtype=torch.int32, device="cuda")}


def prepare(case, seed):
    g = _rng(seed)
    W, L = case["width"], case["leaf"]
    A, B, pairs = _datasets(case, g)
    kind, room = case["kind"], _room(case)
    s = {"kind": kind, "W": W, "L": L}
    if kind == "dataset":
        hA, hB = A.numpy(), B.numpy()
        s.update(DA=dataset.DatasetBlob.build(hA), DB=dataset.DatasetBlob.build(hB), groups_a=dataset.max_groups(hA),
                 groups_b=dataset.max_groups(hB), strategy=case["strategy"], hits=np.full((room, 2), -1, np.int32))
    else:
        # the program's own result arrays; what a pass does not write stays as it is here
        s.update(flags=torch.zeros(room, dtype=torch.uint8, device="cuda"),
                 hits=torch.full((room, 2), -1, dtype=torch.int32, device="cuda"))
    if kind == "fresh":
        s.update(A=A, B=B)
        return s
    s["a"] = pa.MeshBlob.build(A, width=W, leaf_size=L)
    s["b"] = pa.MeshBlob.build(B, width=W, leaf_size=L)
    s["a"].exp_range(), s["b"].exp_range()
    if kind == "join":
        s["box"] = None
        if "query" in case:
            c = _uniform(g, 0.25, 0.75, 3).cpu().numpy() * case["side"]
            s["box"] = np.concatenate([c - case["query"] / 2, c + case["query"] / 2]).astype(np.float32)
    elif kind == "step":
        s.update(cap=room, **_kept(room, W))
    elif kind == "refine":
        s.update(pairs=pairs, **_kept(pairs.shape[0], W))
        s["flags"] = s["flags"][:pairs.shape[0]].clone()
    elif kind == "predicate":
        s.update(pairs=pairs, predicate=case["predicate"])
        s["flags"] = s["flags"][:pairs.shape[0]].clone()
    elif kind == "serve":
        s["server"] = serve.JoinServer(s["a"], s["b"])
        n, side = case["requests"], case["side"]
        k = torch.exp(_uniform(g, 0.0, math.log(3000.0), n, 1)) ** (1 / 3)
        c = _uniform(g, 0.0, 1.0, n, 3) * side
        s["boxes"] = torch.cat([c - k / 2, c + k / 2], 1).float().cpu().numpy()
        s.update(pairs=np.full((n, 8192, 2), -1, np.int32), flags=np.zeros((n, 8192), np.uint8),
                 counts=np.zeros(n, np.int64))
    return s


def _keep(s, hits):
    """The join's result in the program's own array."""
    s["hits"][:hits.shape[0]].copy_(hits)
    return s["hits"]


def _join(s, a, b, box=None):
    pairs = pa.filter_pairs(a, b, query_box=box)
    _, _, status = pa.refine(a, b, pairs, flags=s["flags"])
    hits = pa.compact(pairs, s["flags"])
    return {"candidates": pairs.shape[0], "flags": s["flags"], "status": status, "n": hits.shape[0],
            "hits": _keep(s, hits)}


def run(s):
    kind = s["kind"]
    if kind == "join":
        return _join(s, s["a"], s["b"], s["box"])
    if kind == "fresh":
        a = pa.MeshBlob.build(s["A"], width=s["W"], leaf_size=s["L"])
        b = pa.MeshBlob.build(s["B"], width=s["W"], leaf_size=s["L"])
        return {"boxes_a": a.boxes(), "boxes_b": b.boxes(), "edges_a": a.edge_counts(), "edges_b": b.edge_counts(),
                **_join(s, a, b)}
    if kind == "step":
        pairs, cnt = pa.filter_pairs(s["a"], s["b"], cap=s["cap"], sync=False)
        pa.refine(s["a"], s["b"], pairs, pa.RefineConfig(n_dev=cnt), ws=s["ws"], flags=s["flags"], stats=s["stats"],
                  status=s["status"])
        hits, n_hits = pa.compact(pairs, s["flags"], n_dev=cnt, sync=False)
        n, m = torch.cat([cnt, n_hits]).tolist()
        return {"candidates": n, "flags": s["flags"], "status": s["status"], "n": m, "hits": _keep(s, hits[:m])}
    if kind == "refine":
        flags, _, status = pa.refine(s["a"], s["b"], s["pairs"], ws=s["ws"], flags=s["flags"], stats=s["stats"],
                                     status=s["status"])
        hits = pa.compact(s["pairs"], flags)
        return {"flags": flags, "status": status, "n": hits.shape[0], "hits": _keep(s, hits)}
    if kind == "predicate":
        flags, _, _, status = pa.predicate(s["a"], s["b"], s["pairs"], s["predicate"], flags=s["flags"])
        hits = pa.compact(s["pairs"], flags)
        return {"flags": flags, "status": status, "n": hits.shape[0], "hits": _keep(s, hits)}
    if kind == "serve":
        done = s["server"].run([serve.Request(k, 0.0, box) for k, box in enumerate(s["boxes"])], realtime=False)
        for k, r in enumerate(done):
            n = r.pairs.shape[0]
            s["counts"][k] = n
            s["pairs"][k, :n] = r.pairs
            s["flags"][k, :n] = r.flags
        return {"counts": s["counts"], "pairs": s["pairs"], "flags": s["flags"]}
    pairs, _ = dataset.join_dataset(s["a"], s["b"], s["DA"], s["DB"], s["groups_a"], s["groups_b"],
                                    strategy=s["strategy"])
    s["hits"][:pairs.shape[0]] = pairs
    return {"n": pairs.shape[0], "hits": s["hits"]}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------


def _faces(case):
    """Triangles of A and of B (a closed surface has half as many vertices and 1.5 times as many edges)."""
    what, n = case["data"], case["n"]
    if what == "icospheres":
        return 320 * n, 320 * n
    if what == "tissue":
        return 5120 * n, 4096 * max(1, n // 10)
    if what == "pool":
        mean = sum(_class_sizes(case["f_lo"], case["f_hi"], 10)) / 10
        return int(mean * (n // 2)), int(mean * (n - n // 2))
    if what == "touching":
        return 5120 * n, 5120 * n
    if what == "sweep":
        per = 4 * case["rings"] * (case["rings"] - 1)
        return per * n, per * n
    if what == "nested":
        return 20 * case["nu"] ** 2 * n, 20 * case["nu"] ** 2 * n
    return 12 * n, 12 * n


def work(case):
    """Bytes: the mesh boxes, 9 B a pair, and where two meshes are compared the part of both
    surfaces that lies in the common box (a triangle is 36 B and its 1.5 edges 36 B; an eighth
    of the triangles of a mesh that has a candidate partner); a build reads 18 B a face
    (vertices and ids) and writes triangles, edges and at least a box and a reference a
    triangle pair (14 B).  Flops: a box test (12) and a segment-triangle test (100) for each edge
    in the common box, and a build's orientation test (30) a face."""
    fa, fb = _faces(case)
    F, n = fa + fb, case["n"]
    kind = case["kind"]
    share = {"icospheres": 1.0, "touching": 0.125, "cubes": 1.0}.get(case["data"], 0.125)
    if case["data"] == "sweep":
        share = 0.05  # two fifths of the meshes have a partner
    if case["data"] == "tissue":
        share = 0.05
    meshes = 2 * n if case["data"] != "tissue" else n + n // 10
    pairs = case.get("pairs", 2 * n)
    if "query" in case:
        vol = min(1.0, (case["query"] + 2.0) ** 3 / case["side"] ** 3)
        share, pairs = share * vol, pairs * vol
    rounds = 1
    if kind == "serve":
        share = min(1.0, case["requests"] * 600 / (4 * n))
        pairs, rounds = 600 * case["requests"], 1
    near = share * F
    bytes_ = rounds * 24 * meshes + 9 * pairs + 72 * near
    flops = 12 * meshes + 112 * 1.5 * near
    if kind == "fresh":
        bytes_ += (18 + 72 + 14) * F
        flops += 30 * F
    return {"bytes": float(bytes_), "flops": float(flops)}


def exact(case, seed):
    """Boxes are the only floating results: the extremes of the vertices.  Flags, pairs and counts
    are whole numbers."""
    if case["kind"] != "fresh":
        return None
    A, B, _ = _datasets(case, _rng(seed))
    return {"boxes_a": _boxes(A).double(), "boxes_b": _boxes(B).double(), "edges_a": None, "edges_b": None,
            "candidates": None, "flags": None, "status": None, "n": None, "hits": None}
