"""The work that programs have this framework do, as cases that can be timed and compared.

A case is a dict of plain values.  Its "kind" says which public entry points one pass calls:

  embed      pipeline.Embedder.embed: all levels of a mesh and the cut links of the finest one; without links
             (links=False) the solid flags and the forest alone
  embed2d    pipeline2d.Embedder2D.embed: a polygon in a quadtree
  gradient   pipeline.cut_link_q and its backward: dL/dvertices of a kept embedding
  shape      pipeline.shape_step with the backward: one step of a moving geometry
  dense      pipeline.links_dense: the table in the layout that a solver reads
  ibb        geo_ibb: interpolated bounce-back of a solver's populations at the links

Geometries are made here, on the GPU: noisy star meshes like scanned surfaces, prisms and boxes like CAD parts,
scenes of spheres, noisy circles and rectangles in 2D, and for the solver's side the links of a sphere.  A case fixes
the body, the seed its pose (a reflection of the domain, and a permutation of its axes where it is cubic) and the
numbering of its vertices and triangles, so that every seed gives other values and the same number of blocks and links.
Coordinates are base cells, n0 the base cells per axis, levels 0..lf.
"""
import math

import numpy as np
import torch

import paper_2512_01251_amd as geo
from paper_2512_01251_amd import pipeline, pipeline2d

VERTS = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # the smallest call: a coarse body in one uniform level (the convex pin of the tests)
        _embed("embed_icosphere64", "icosphere", 1280, (64, 64, 64), 0, 19, "f64", 12.0),
        # a small body with refinement, as in an interactive preview or a unit test of a solver
        _embed("embed_star1792", "star", 1792, (32, 32, 32), 2, 27, "f32", 10.0),
        # a CAD part: few large triangles over many cells (the 256-gon cylinder of the configurations)
        _embed("embed_cylinder256", "prism", 1024, (256, 256, 256), 3, 19, "f64", 30.0),
        # an ordinary scan, double vertices (stands in for the 112k-triangle bunny)
        _embed("embed_star112k", "star", 112000, (128, 128, 128), 3, 19, "f64", 40.0),
        # many bodies, all arithmetic in float64
        _embed("embed_spheres64", "spheres", 1024000, (256, 256, 256), 3, 19, "f64", 8.0, precision="f64"),
        # the largest: stands in for the 7.2M-triangle dragon, the framework's headline workload
        _embed("embed_star7m", "star", 7200000, (256, 256, 256), 4, 27, "f32", 40.0),
        # flags and forest alone (a solver with plain voxel walls), a ragged domain
        _embed("flags_star1m", "star", 1050000, (192, 200, 176), 3, 27, "f32", 44.0, links=False),
        # the 2D cylinder of the configurations
        {"name": "embed2d_circle4096", "kind": "embed2d", "shape": "circle", "edges": 4096, "nx": 512, "ny": 512,
         "lf": 4, "size": 4.0, "d_spec": 2.0},
        # the adjoint of a shape optimisation: the gradient of a functional of q
        {**_embed("gradient_star448k", "star", 448000, (128, 128, 128), 3, 27, "f32", 40.0), "kind": "gradient"},
        # one step of a moving body: rebuild, gradient, uncovered and covered cells
        {**_embed("shape_star112k", "star", 112000, (128, 128, 128), 3, 19, "f64", 40.0), "kind": "shape"},
        # the table of a finished embedding laid out for the solver
        {"name": "dense_384", "kind": "dense", "nx": 384, "ny": 384, "nz": 384, "lf": 1, "lattice": 27},
        # a solver's wall step, each time step
        {"name": "ibb_256", "kind": "ibb", "nx": 256, "ny": 256, "nz": 256, "lf": 1, "lattice": 19, "pops": "f32",
         "interpolate": True, "table": True},
    ]


def draw(rng):
    kind = rng.choice(["embed"] * 9 + ["flags", "embed2d", "embed2d", "gradient", "shape", "dense", "ibb", "ibb"])
    if kind == "embed2d":
        n = [4 * rng.randint(8, 128) for _ in range(2)]
        lf = rng.randint(0, 4)
        while max(n) << lf > 8192:
            lf -= 1
        shape = rng.choice(["circle", "circle", "rectangle"])
        return {"kind": kind, "shape": shape, "edges": 4 if shape == "rectangle" else _log(rng, 16, 8000),
                "nx": n[0], "ny": n[1], "lf": lf, "size": rng.uniform(0.02, 0.3) * min(n),
                "d_spec": rng.choice([2.0, 2.0, 6.0])}
    if kind in ("dense", "ibb"):
        n = 4 * _log(rng, 8, 64)
        c = {"kind": kind, "nx": n + 4 * rng.randint(0, 8), "ny": n + 4 * rng.randint(0, 8), "nz": n,
             "lf": rng.randint(0, 1), "lattice": rng.choice([19, 27])}
        if kind == "ibb":
            c.update(pops=rng.choice(["f32", "f32", "f64"]), interpolate=rng.random() < 0.8,
                     table=rng.random() < 0.7)
        return c
    shape = rng.choice(["star"] * 5 + ["prism", "box", "spheres", "icosphere"]) if kind == "embed" else "star"
    nz = 4 * rng.randint(8, 32)
    n0 = (nz + 4 * rng.randint(0, 8), nz + 4 * rng.randint(0, 8), nz)
    lf = rng.randint(0, 4)
    while max(n0) << lf > 1024:
        lf -= 1
    tris = {"star": _log(rng, 400, 2000000), "prism": 4 * 8 * rng.randint(2, 60), "box": 12,
            "spheres": _log(rng, 8000, 400000), "icosphere": rng.choice([320, 1280, 5120])}[shape]
    c = _embed("", shape, tris, n0, lf, rng.choice([19, 27]), rng.choice(["f32", "f64"]),
               round(nz * (0.03 if shape == "spheres" else 0.28) * rng.uniform(0.55, 1), 3),
               precision=rng.choice(["f32", "f32", "f32", "f64"]), links=kind != "flags",
               d_spec=rng.choice([2.0, 2.0, 2.0, 6.0]))
    del c["name"]
    if kind in ("gradient", "shape"):
        c["kind"] = kind
    return c


def _embed(name, shape, tris, n0, lf, lattice, verts, radius, precision="f32", links=True, d_spec=2.0):
    return {"name": name, "kind": "embed", "shape": shape, "tris": tris, "nx": n0[0], "ny": n0[1], "nz": n0[2],
            "lf": lf, "lattice": lattice, "verts": verts, "radius": radius, "precision": precision, "links": links,
            "d_spec": d_spec}


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _n0(case):
    return tuple(case[k] for k in ("nx", "ny", "nz") if k in case)


# ---------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind == "embed2d":
        V, E = _polygon(case, seed)
        return {"case": case, "V": V, "E": E, "embedder": pipeline2d.Embedder2D("cuda")}
    if kind in ("dense", "ibb"):
        return _prepare_solver(case, seed)
    V, T = _mesh(case, seed)
    s = {"case": case, "V": V, "T": T, "embedder": pipeline.Embedder("cuda")}
    if kind == "gradient":
        s["emb"] = _run_embed(s, V)
        s["w"] = _weights(s["emb"].links.n, seed)
        s["V"] = V.requires_grad_(True)
    if kind == "shape":
        s["prev"] = _run_embed(s, V)
        s["V"] = _mesh(case, seed, 1)[0].requires_grad_(True)
    return s


def _weights(n, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float32) * 2 - 1


def _pose(case, V, P, seed):
    """The body in the seed's pose: axes permuted (cubic domains), reflected, primitives re-ordered cyclically and
    vertices renumbered cyclically.  Coordinates are multiples of a power of two, so that reflections are exact."""
    n0, dim = _n0(case), V.shape[1]
    bits = 24 - math.ceil(math.log2(max(n0))) if case.get("verts") == "f32" else 40
    V = torch.round(V * 2.0 ** bits) / 2.0 ** bits
    flip, turn, rng = seed % 2 ** dim, 0, np.random.default_rng(seed)
    if len(set(n0)) == 1:
        turn = seed // 2 ** dim % (6 if dim == 3 else 2)
        order = [(0, 1, 2), (1, 2, 0), (2, 0, 1), (1, 0, 2), (0, 2, 1), (2, 1, 0)][turn] if dim == 3 else (turn, 1 - turn)
        V = V[:, list(order)]
    odd = turn >= 3 if dim == 3 else turn == 1
    for a in range(dim):
        if flip >> a & 1:
            V = torch.cat([V[:, :a], n0[a] - V[:, a:a + 1], V[:, a + 1:]], 1)
            odd = not odd
    if odd:  # a mirror image: outward orientation restored
        P = P.flip(1)
    k = int(rng.integers(0, V.shape[0]))
    V, P = torch.roll(V, k, 0), (P + k) % V.shape[0]
    P = torch.roll(P, int(rng.integers(0, P.shape[0])), 0)
    return V.to(VERTS[case.get("verts", "f64")]).contiguous(), P.to(torch.int32).contiguous()


def _mesh(case, seed, step=0):
    """The case's body in the seed's pose; step 1: after a small rotation about z and a shift."""
    n0 = np.array(_n0(case), dtype=np.float64)
    shape, tris = case["shape"], case["tris"]
    rng = np.random.default_rng([tris, *_n0(case)])
    r = case["radius"]
    c = n0 / 2 + rng.uniform(-0.4, 0.4, 3)
    if shape == "star":
        nt = max(4, int(round(math.sqrt(tris / 2 / 1.11))))
        V, T = _star(nt, max(4, int(round(tris / 2 / nt))), r, c, rng)
    elif shape == "spheres":
        g = 4 if tris > 100000 else 2
        nt = max(4, int(round(math.sqrt(tris / g ** 3 / 2 / 1.25))))
        npk = max(4, int(round(tris / g ** 3 / 2 / nt)))
        vs, ts, base = [], [], 0
        for k in range(g ** 3):
            cell = n0 / g
            at = (np.array([k % g, k // g % g, k // g // g]) + 0.5) * cell + rng.uniform(-0.12, 0.12, 3) * cell
            v, t = _star(nt, npk, r, at, rng, amplitude=0.15)
            vs.append(v)
            ts.append(t + base)
            base += v.shape[0]
        V, T = torch.cat(vs), torch.cat(ts)
    elif shape == "icosphere":
        V, T = _icosphere(int(round(math.log(tris / 20, 4))), r, c)
    else:
        V, T = _prism(max(8, tris // 4), r, c) if shape == "prism" else _box(r * rng.uniform(0.6, 1, 3), c)
    if step:
        a = 0.002
        X = V - torch.from_numpy(c).cuda()
        V = torch.stack([X[:, 0] * math.cos(a) - X[:, 1] * math.sin(a) + c[0] + 0.031,
                         X[:, 0] * math.sin(a) + X[:, 1] * math.cos(a) + c[1] - 0.017, V[:, 2] + 0.023], 1)
    return _pose(case, V, T, seed)


def _star(n_theta, n_phi, radius, centre, rng, amplitude=0.25, lmax=8):
    """Closed latitude-longitude mesh r = R (1 + A noise), the noise a sum of real spherical harmonics with
    coefficients N(0, 1/l^2), bounded so that r stays in [0.3, 1.5] R.  Rings, single pole vertices, two triangles
    per quad; the triangles that repeat a pole vertex have zero area."""
    dev = "cuda"
    th = torch.arange(0, n_theta + 1, dtype=torch.float64, device=dev) * (math.pi / n_theta)
    ph = torch.arange(n_phi, dtype=torch.float64, device=dev) * (2 * math.pi / n_phi)
    ct, st = torch.cos(th), torch.sin(th)
    ct[0], ct[-1], st[0], st[-1] = 1.0, -1.0, 0.0, 0.0
    f = torch.zeros(n_theta + 1, n_phi, dtype=torch.float64, device=dev)
    pmm = torch.ones_like(ct)
    for m in range(lmax + 1):
        if m:
            pmm = pmm * st * (2 * m - 1)
        rc, rs = torch.zeros_like(ct), torch.zeros_like(ct)
        p0, p1 = torch.zeros_like(ct), pmm
        for l in range(m, lmax + 1):
            if l > m:
                p0, p1 = p1, (ct * p1 * (2 * l - 1) - p0 * (l + m - 1)) / (l - m)
            if l == 0:
                continue
            n = math.sqrt((2 * l + 1) / (4 * math.pi) * math.factorial(l - m) / math.factorial(l + m))
            n *= math.sqrt(2.0) if m else 1.0
            rc += p1 * (n * rng.normal(0, 1 / l))
            rs += p1 * (n * rng.normal(0, 1 / l))
        f += rc[:, None] * torch.cos(m * ph)[None] + (rs[:, None] * torch.sin(m * ph)[None] if m else 0.0)
    r = radius * (1 + amplitude * f).clamp(0.3, 1.5)
    ring = torch.stack([r * st[:, None] * torch.cos(ph)[None], r * st[:, None] * torch.sin(ph)[None],
                        r * ct[:, None]], 2)
    V = torch.cat([ring[0, :1], ring[1:-1].reshape(-1, 3), ring[-1, :1]])
    V = V + torch.tensor(centre, dtype=torch.float64, device=dev)
    i = torch.arange(n_theta, device=dev)[:, None].expand(n_theta, n_phi)
    j = torch.arange(n_phi, device=dev)[None].expand(n_theta, n_phi)

    def vid(a, b):
        v = 1 + (a - 1) * n_phi + b % n_phi
        return torch.where(a == 0, 0, torch.where(a == n_theta, 1 + (n_theta - 1) * n_phi, v))

    a, b, c, d = vid(i, j), vid(i + 1, j), vid(i + 1, j + 1), vid(i, j + 1)
    T = torch.stack([torch.stack([a, b, c], 2), torch.stack([a, c, d], 2)], 2).reshape(-1, 3)
    return V, T


def _icosphere(subdivisions, radius, centre):
    g = (1 + math.sqrt(5)) / 2
    P = np.array([p for a in (-1.0, 1.0) for b in (-g, g) for p in ((0, a, b), (a, b, 0), (b, 0, a))])
    d = np.linalg.norm(P[:, None] - P[None], axis=2)
    F = [(i, j, k) for i in range(12) for j in range(i + 1, 12) for k in range(j + 1, 12)
         if max(d[i, j], d[j, k], d[i, k]) < 2.1]
    F = np.array([t if np.linalg.det(P[list(t)]) > 0 else (t[0], t[2], t[1]) for t in F])
    P /= np.linalg.norm(P, axis=1, keepdims=True)
    for _ in range(subdivisions):
        e = np.sort(np.concatenate([F[:, [0, 1]], F[:, [1, 2]], F[:, [2, 0]]]), axis=1)
        u, inv = np.unique(e, axis=0, return_inverse=True)
        m = (inv.reshape(3, -1) + len(P)).T
        Q = P[u[:, 0]] + P[u[:, 1]]
        P = np.concatenate([P, Q / np.linalg.norm(Q, axis=1, keepdims=True)])
        F = np.concatenate([np.stack([F[:, 0], m[:, 0], m[:, 2]], 1), np.stack([F[:, 1], m[:, 1], m[:, 0]], 1),
                            np.stack([F[:, 2], m[:, 2], m[:, 1]], 1), m])
    return torch.from_numpy(P * radius + centre).cuda(), torch.from_numpy(F).cuda()


def _prism(n, radius, centre):
    """Regular n-gon prism along z, its caps fans around the axis points."""
    k = np.arange(n)
    ring = np.stack([np.cos(2 * np.pi * k / n), np.sin(2 * np.pi * k / n), np.zeros(n)], 1) * radius
    up = np.array([0, 0, radius])
    V = np.concatenate([ring - up, ring + up, [-up], [up]]) + centre
    k1 = (k + 1) % n
    T = np.concatenate([np.stack([k, k1, n + k1], 1), np.stack([k, n + k1, n + k], 1),
                        np.stack([np.full(n, 2 * n), k1, k], 1), np.stack([np.full(n, 2 * n + 1), n + k, n + k1], 1)])
    return torch.from_numpy(V).cuda(), torch.from_numpy(T).cuda()


def _box(half, centre):
    V = np.array([[(1 if k >> a & 1 else -1) * half[a] for a in range(3)] for k in range(8)]) + centre
    Q = [(0, 4, 6, 2), (1, 3, 7, 5), (0, 1, 5, 4), (2, 6, 7, 3), (0, 2, 3, 1), (4, 5, 7, 6)]
    T = np.array([t for a, b, c, d in Q for t in ((a, b, c), (a, c, d))])
    return torch.from_numpy(V).cuda(), torch.from_numpy(T).cuda()


def _polygon(case, seed):
    """Counter-clockwise: a noisy circle of radius "size", or a rectangle of that half height."""
    n = case["edges"]
    rng = np.random.default_rng([n, *_n0(case)])
    c = np.array(_n0(case)) / 2 + rng.uniform(-0.4, 0.4, 2)
    if case["shape"] == "rectangle":
        h = np.array([1.0, rng.uniform(0.7, 1.0)]) * case["size"]
        P = np.array([[-1, -1], [1, -1], [1, 1], [-1, 1]]) * h + c
    else:
        a = 2 * np.pi * np.arange(n) / n
        r = case["size"] * (1 + 0.2 / n * rng.uniform(-1, 1, n) + 0.05 * np.sin(3 * a + rng.uniform(0, 6)))
        P = np.stack([np.cos(a) * r, np.sin(a) * r], 1) + c
    E = np.stack([np.arange(n), (np.arange(n) + 1) % n], 1)
    return _pose(case, torch.from_numpy(P).cuda(), torch.from_numpy(E).cuda(), seed)


def _directions(lattice, dim=3):
    """[(k, c)] of the lattice's moving directions in increasing k; c in axis order."""
    if dim == 2:
        return [(k, (k % 3 - 1, k // 3 - 1)) for k in range(9) if k != 4]
    ks = [(k, (k % 3 - 1, k // 3 % 3 - 1, k // 9 - 1)) for k in range(27) if k != 13]
    return [(k, c) for k, c in ks if lattice == 27 or sum(v * v for v in c) <= 2]


def _sphere_level(case, seed):
    """The finest level of a forest around a sphere, and its cut links, in closed form: level 0 whole, level 1 (lf = 1)
    the children of the blocks within 8 cells of the sphere."""
    dev, n0, L = "cuda", np.array(_n0(case)), case["lf"]
    rng = np.random.default_rng(n0)
    c = np.round((n0 / 2 + rng.uniform(-0.4, 0.4, 3)) * 1024) / 1024
    c = torch.tensor([n0[a] - c[a] if seed >> a & 1 else c[a] for a in range(3)], device=dev)
    r = float(n0.min() * rng.uniform(0.29, 0.31))
    nb = [int(v) // 4 for v in n0]
    z, y, x = torch.meshgrid(*[torch.arange(nb[a], device=dev, dtype=torch.int32) for a in (2, 1, 0)], indexing="ij")
    coord = torch.stack([x, y, z], 3).reshape(-1, 3)
    maps = []
    if L:
        d = ((coord.double() * 4 + 2 - c).square().sum(1).sqrt() - r).abs()
        pick = d < 8
        first = torch.cumsum(pick, 0) - 1
        maps.append(torch.where(pick, 8 * first, -1).to(torch.int32))
        o = torch.arange(8, device=dev, dtype=torch.int32)
        oct_ = torch.stack([o & 1, o >> 1 & 1, o >> 2], 1)
        coord = (2 * coord[pick][:, None] + oct_[None]).reshape(-1, 3)
    coord = coord.contiguous()
    t = torch.arange(64, device=dev)
    tc = torch.stack([t & 3, t >> 2 & 3, t >> 4], 1)
    h = 0.5 ** L
    cell, dr, q, solid = [], [], [], []
    dirs = _directions(case["lattice"])
    cs = torch.tensor([v for _, v in dirs], device=dev, dtype=torch.float64)
    ks = torch.tensor([k for k, _ in dirs], device=dev, dtype=torch.uint8)
    for b0 in range(0, coord.shape[0], 100000):
        X = ((4 * coord[b0:b0 + 100000, None].double() + tc[None] + 0.5) * h - c)  # [b, 64, 3], the centre at 0
        XX = X.square().sum(2)
        inside = XX <= r * r
        solid.append((inside.long() << t[None]).sum(1))
        # of the fluid cells near enough to have a link
        near = (~inside & (XX <= (r + 2 * h) ** 2)).reshape(-1).nonzero()[:, 0]
        Xn = X.reshape(-1, 3)[near]
        Y = Xn[:, None] + h * cs[None]
        dom = ((Y + c > 0) & (Y + c < torch.tensor(n0, device=dev))).all(2)
        i, s = ((Y.square().sum(2) <= r * r) & dom).nonzero(as_tuple=True)
        A, B = (h * cs[s]).square().sum(1), (Xn[i] * cs[s] * h).sum(1)
        q.append((-B - (B * B - A * (Xn[i].square().sum(1) - r * r)).clamp(min=0).sqrt()) / A)
        cell.append(near[i] + 64 * b0)
        dr.append(ks[s])
    q = torch.cat(q).float().clamp(1e-7, 1.0)
    g = torch.Generator(dev).manual_seed(seed)
    tri = torch.randint(0, 1 << 22, (q.numel(),), generator=g, device=dev, dtype=torch.int32)
    return coord, maps, torch.cat(solid), torch.cat(cell).to(torch.int32), torch.cat(dr), q, tri


def _populations(case, nb, seed):
    qf = 19 if case["lattice"] == 19 else 27
    n2 = [sum(v * v for v in c) for _, c in _directions(case["lattice"])]
    n2.insert(qf // 2, 0)
    w = {19: [1 / 3, 1 / 18, 1 / 36], 27: [8 / 27, 2 / 27, 1 / 54, 1 / 216]}[case["lattice"]]
    w = torch.tensor([w[v] for v in n2], device="cuda", dtype=VERTS[case["pops"]])
    g = torch.Generator("cuda").manual_seed(seed)
    f = torch.empty((2, nb, qf, 64), device="cuda", dtype=VERTS[case["pops"]])
    f.uniform_(0.9, 1.1, generator=g).mul_(w[None, None, :, None])
    return f[0], f[1]


def _dense_arrays(case, nb, cell, dr, q, tri):
    """The dense layout of a table (block map, q and hit triangle), -1 where there is no link."""
    dirs = _directions(case["lattice"])
    slot = torch.full((27,), -1, device="cuda", dtype=torch.int64)
    slot[torch.tensor([k for k, _ in dirs], device="cuda")] = torch.arange(len(dirs), device="cuda")
    b = cell.long() >> 6
    has = torch.zeros(nb, device="cuda", dtype=torch.bool)
    has[b] = True
    bmap = torch.where(has, torch.cumsum(has, 0) - 1, -1).to(torch.int32)
    at = (bmap[b].long() * len(dirs) + slot[dr.long()]) * 64 + (cell & 63)
    n = int(has.sum()) * len(dirs) * 64
    dq = torch.full((n,), -1.0, device="cuda", dtype=q.dtype)
    dt = torch.full((n,), -1, device="cuda", dtype=torch.int32)
    dq[at], dt[at] = q, tri
    return bmap, dq.view(-1, len(dirs), 64), dt.view(-1, len(dirs), 64)


def _prepare_solver(case, seed):
    coord, maps, solid, cell, dr, q, tri = _sphere_level(case, seed)
    n0, nb = _n0(case), coord.shape[0]
    if case["kind"] == "dense":
        emb = pipeline.Embedding(n0, case["lf"], case["lattice"])
        for m in maps:
            emb.levels.append(pipeline.Level(len(emb.levels), None, child_map=m))
        emb.levels.append(pipeline.Level(case["lf"], coord, solid=solid))
        emb.links = pipeline.Links(None, cell, dr, q, tri)
        return {"case": case, "emb": emb, "caps": {}}
    bmap, dq, _ = _dense_arrays(case, nb, cell, dr, q, tri)
    level = geo.make_level(n0, case["lf"], coord, maps)
    nbr = None
    if case["table"]:
        nbr = torch.empty((nb, 27), dtype=torch.int32, device="cuda")
        geo.geo_block_neighbours(level, nbr)
    post, new = _populations(case, nb, seed)
    return {"case": case, "level": level, "keep": (coord, maps), "solid": solid, "bmap": bmap, "q": dq, "nbr": nbr,
            "post": post, "new": new}


# ---------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------

def _run_embed(s, V):
    c = s["case"]
    return s["embedder"].embed(V, s["T"], _n0(c), c["lf"], c["lattice"], c["d_spec"], c["precision"],
                               with_links=c["links"])


def _outputs(emb):
    out = {"levels": [[lv.bcoord, lv.solid, lv.bclass, lv.refine, lv.child_map] for lv in emb.levels]}
    k = emb.links
    if k is not None:
        out["links"] = {"cell": k.cell, "dir": k.dir, "q": k.q, "hit": k.edge if hasattr(k, "edge") else k.tri}
    return out


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "embed":
        return _outputs(_run_embed(s, s["V"]))
    if kind == "embed2d":
        return _outputs(s["embedder"].embed(s["V"], s["E"], _n0(c), c["lf"], c["d_spec"]))
    if kind == "gradient":
        q = pipeline.cut_link_q(s["V"], s["T"], s["emb"])
        g, = torch.autograd.grad(q, s["V"], s["w"])
        return {"q": q, "grad": g}
    if kind == "shape":
        emb, q, change = pipeline.shape_step(s["embedder"], s["V"], s["T"], _n0(c), c["lf"], c["lattice"], c["d_spec"],
                                             c["precision"], s["prev"])
        g, = torch.autograd.grad(q.sum(), s["V"])
        return {"embedding": _outputs(emb), "grad": g, "spawned": change.spawned, "covered": change.covered,
                "counts": change.counts}
    if kind == "dense":
        d = pipeline.links_dense(s["emb"], s["caps"])
        return {"block_map": d.block_map, "q": d.q, "tri": d.tri}
    geo.geo_ibb(s["level"], s["solid"], s["bmap"], s["q"], s["q"].shape[0], c["lattice"], c["interpolate"], s["post"],
                s["new"], None, nbr=s["nbr"])
    return s["new"]


# ---------------------------------------------------------------------------------------------------------------
# the work of a pass, from the sizes alone: surface area in cells of the finest level, links per unit of area
# (a quarter of |c| for each direction), blocks of a refined level about 15 layers of the surface
# ---------------------------------------------------------------------------------------------------------------

def work(case):
    kind, n0 = case["kind"], _n0(case)
    links_per_area = sum(math.sqrt(sum(v * v for v in c)) / 4 for _, c in _directions(case.get("lattice", 27)))
    m = min(n0)
    if kind == "embed2d":
        blocks = n0[0] * n0[1] / 16
        per = case["size"] * (8 if case["shape"] == "rectangle" else 2 * math.pi)
        blocks += sum(12 * per * 2 ** l / 4 for l in range(1, case["lf"] + 1))
        links = per * 2 ** case["lf"] * 3 * (1 + math.sqrt(2)) / 4
        return {"bytes": 24 * case["edges"] + 16 * blocks + 13 * links, "flops": 31 * links + 20 * case["edges"]}
    if kind in ("dense", "ibb"):
        area = 4 * math.pi * (0.3 * m * 2 ** case["lf"]) ** 2
        links = area * links_per_area
        total = n0[0] * n0[1] * n0[2] / 64 if not case["lf"] else 1.2 * area
        bnd, dirs = area / 16 * 1.5, len(_directions(case["lattice"]))
        if kind == "dense":
            return {"bytes": 13 * links + 4 * total + 8 * bnd * dirs * 64, "flops": 0}
        size = 8 if case["pops"] == "f64" else 4
        return {"bytes": 4 * total + 4 * bnd * dirs * 64 + (3 if case["interpolate"] else 2) * size * links,
                "flops": 5 * links}
    r = case["radius"]
    g = 4 if case["tris"] > 100000 else 2
    area0 = {"star": 4 * math.pi * r * r, "icosphere": 4 * math.pi * r * r, "prism": 6 * math.pi * r * r,
             "box": 15 * r * r, "spheres": g ** 3 * 4 * math.pi * r * r}[case["shape"]]
    size = 4 if case["verts"] == "f32" else 8
    links = area0 * 4 ** case["lf"] * links_per_area
    mesh = case["tris"] * (12 + 1.5 * size)
    if kind == "gradient":
        return {"bytes": mesh + 17 * links + 1.5 * size * case["tris"], "flops": 100 * links}
    blocks = n0[0] * n0[1] * n0[2] / 64 + sum(15 * area0 * 4 ** l / 16 for l in range(1, case["lf"] + 1))
    out = {"bytes": mesh + 26 * blocks, "flops": 40 * case["tris"]}
    if case["links"]:
        out["bytes"] += 13 * links
        out["flops"] += 31 * links
    if kind == "shape":
        out["bytes"] += 13 * links + 1.5 * size * case["tris"] + 24 * 15 * area0 * 4 ** case["lf"] / 16
        out["flops"] += 100 * links
    return out


# ---------------------------------------------------------------------------------------------------------------
# the floating outputs in float64, by plain definitions on dense grids (grids up to 1024 cells per axis in 3D)
# ---------------------------------------------------------------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind == "embed2d":
        V, E = _polygon(case, seed)
        return {"links": {"q": _table(case, V, E)["q"]}}
    if kind in ("dense", "ibb"):
        coord, maps, solid, cell, dr, q, tri = _sphere_level(case, seed)
        bmap, dq, dt = _dense_arrays(case, coord.shape[0], cell, dr, q.double(), tri)
        if kind == "dense":
            return {"block_map": None, "q": dq, "tri": None}
        return _bounce_back(case, seed, coord, solid, cell, dr, q)
    if max(_n0(case)) << case["lf"] > 1024 or not case["links"]:
        return None
    V, T = _mesh(case, seed, 1 if kind == "shape" else 0)
    t = _table(case, V.double(), T)
    if kind == "embed":
        return {"links": {"q": t["q"]}}
    w = _weights(t["q"].numel(), seed).double() if kind == "gradient" else torch.ones_like(t["q"])
    g = _q_gradient(case, V.double(), T, t, w)
    if kind == "gradient":
        return {"q": t["q"], "grad": g}
    return {"embedding": {"links": {"q": t["q"]}}, "grad": g}


def _chunks(counts, most=1 << 24):
    """Flat enumeration of counts[p] items for each p, in pieces: (p, index within p)."""
    end = torch.cumsum(counts, 0)
    total = int(end[-1]) if end.numel() else 0
    for a in range(0, total, most):
        i = torch.arange(a, min(total, a + most), device=counts.device)
        p = torch.searchsorted(end, i, right=True)
        yield p, i - (end[p] - counts[p])


def _solid(V, P, n):
    """Solid flags of all cells of a level, [nz, ny, nx] or [ny, nx]: parity of the surface crossings to the left.
    V: vertices in the frame where cell centres are integers; P: triangles or edges; n: cells per axis."""
    dim = V.shape[1]
    X = V[P.long()]
    lo = [X[:, :, a].amin(1).ceil().clamp(min=0).long() for a in range(1, dim)]
    hi = [X[:, :, a].amax(1).floor().clamp(max=n[a] - 1).long() for a in range(1, dim)]
    cnt = [(h - l + 1).clamp(min=0) for l, h in zip(lo, hi)]
    rows = n[1] * (n[2] if dim == 3 else 1)
    grid = torch.zeros(rows * n[0], dtype=torch.int8, device=V.device)
    for p, i in _chunks(cnt[0] * (cnt[1] if dim == 3 else 1)):
        y = lo[0][p] + i % cnt[0][p]
        if dim == 3:
            z = lo[1][p] + i // cnt[0][p]
            A, B, C = X[p].unbind(1)
            e1, e2 = B - A, C - A
            N = torch.linalg.cross(e1, e2)
            Q = torch.stack([torch.zeros_like(y), y, z], 1).double()
            ins = N[:, 0] != 0
            for U, W in ((A, B), (B, C), (C, A)):
                e = (U[:, 1] - Q[:, 1]) * (W[:, 2] - Q[:, 2]) - (U[:, 2] - Q[:, 2]) * (W[:, 1] - Q[:, 1])
                ins &= e * N[:, 0] > 0
            x = A[:, 0] - (N[:, 1] * (Q[:, 1] - A[:, 1]) + N[:, 2] * (Q[:, 2] - A[:, 2])) / N[:, 0]
            row = y + n[1] * z
        else:
            A, B = X[p].unbind(1)
            ins = (A[:, 1] > y) != (B[:, 1] > y)
            x = A[:, 0] + (y - A[:, 1]) * (B[:, 0] - A[:, 0]) / (B[:, 1] - A[:, 1])
            row = y
        m = x[ins].ceil().clamp(0, n[0]).long()
        row = row[ins]
        k = m < n[0]
        grid.index_add_(0, row[k] * n[0] + m[k], torch.ones_like(m[k], dtype=torch.int8))
    shape = [n[a] for a in reversed(range(dim))]
    return torch.cumsum(grid.view(shape), dim - 1, dtype=torch.int8).bitwise_and_(1).bool()


def _near(m):
    """True where one of the 3^dim - 1 neighbours is."""
    dim, dev = m.dim(), m.device
    w = torch.zeros([s + 2 for s in m.shape], dtype=torch.bool, device=dev)
    w[(slice(1, -1),) * dim] = m
    out = torch.zeros_like(m)
    for k in range(3 ** dim):
        o = [k // 3 ** a % 3 for a in range(dim)]
        if o != [1] * dim:
            out |= w[tuple(slice(v, v + s) for v, s in zip(o, m.shape))]
    return out


def _finest_blocks(case, V, P):
    """Blocks of the finest level in block order ([nb, dim], slowest axis first) and its dense solid flags."""
    n0, dim, dev = _n0(case), V.shape[1], V.device
    passes = 1 + int(math.floor(case["d_spec"] / (4 * math.sqrt(2.0))))
    there = torch.ones([n0[a] // 4 for a in reversed(range(dim))], dtype=torch.bool, device=dev)
    at = there.nonzero()
    for L in range(case["lf"] + 1):
        S = _solid(V * 2.0 ** L - 0.5, P, [v << L for v in n0])
        if L == case["lf"]:
            return at, S
        v = []
        for s in S.shape:
            v += [s // 4, 4]
        some = S.view(v).any(dim=tuple(range(1, 2 * dim, 2)))
        sol, flu = there & some, there & ~some
        edge = sol & _near(flu)
        ok = there & ~_near(~there)
        mark = ((edge & ok) | _near(edge)) & there
        for k in range(passes):
            mark |= _near(mark) & (flu if k else there)
        mark &= ok
        par = at[mark[tuple(at.T)]]
        o = torch.arange(2 ** dim, device=dev)
        off = torch.stack([o >> a & 1 for a in reversed(range(dim))], 1)
        at = (2 * par[:, None] + off[None]).reshape(-1, dim)
        there = torch.zeros([2 * s for s in there.shape], dtype=torch.bool, device=dev)
        there[tuple(at.T)] = True


def _table(case, V, P):
    """The link table: cell coordinates X [n, dim] (axis order), direction c, q, and a primitive that is hit."""
    dim, dev = V.shape[1], V.device
    at, S = _finest_blocks(case, V, P)
    n = list(reversed(S.shape))
    dirs = _directions(case.get("lattice", 27), dim)
    t = torch.arange(4 ** dim, device=dev)
    tc = torch.stack([t >> 2 * a & 3 for a in range(dim)], 1)
    flat = S.reshape(-1)
    stride = [1, n[0], n[0] * n[1]][:dim]

    def solid_at(Y):
        ins = torch.ones(Y.shape[:-1], dtype=torch.bool, device=dev)
        i = torch.zeros(Y.shape[:-1], dtype=torch.long, device=dev)
        for a in range(dim):
            ins &= (Y[..., a] >= 0) & (Y[..., a] < n[a])
            i += Y[..., a].clamp(0, n[a] - 1) * stride[a]
        return ins & flat[i]

    Xs, ks = [], []
    cs = torch.tensor([c for _, c in dirs], device=dev)
    for b in at.flip(1).split(50000):
        X = 4 * b[:, None] + tc[None]
        fluid = ~solid_at(X)
        m = torch.stack([fluid & solid_at(X + c) for c in cs], 2)
        i, j, s = m.nonzero(as_tuple=True)
        Xs.append(X[i, j])
        ks.append(s)
    X, s = torch.cat(Xs), torch.cat(ks)
    lin = sum(X[:, a] * stride[a] for a in range(dim))
    key, order = torch.sort(lin * len(dirs) + s)
    pos, ts, who = [], [], []
    W = (V * 2.0 ** case["lf"] - 0.5)[P.long()]
    lo = [(W[:, :, a].amin(1) - 1).ceil().clamp(min=0).long() for a in range(dim)]
    cnt = [((W[:, :, a].amax(1) + 1).floor().clamp(max=n[a] - 1).long() - lo[a] + 1).clamp(min=0) for a in range(dim)]
    count = cnt[0] * cnt[1] * (cnt[2] if dim == 3 else 1)
    for p, i in _chunks(count):
        Y = [lo[0][p] + i % cnt[0][p], lo[1][p] + i // cnt[0][p] % cnt[1][p]]
        if dim == 3:
            Y.append(lo[2][p] + i // (cnt[0][p] * cnt[1][p]))
        Y = torch.stack(Y, 1)
        A, B = W[p, 0], W[p, 1]
        N = torch.linalg.cross(B - A, W[p, 2] - A) if dim == 3 else torch.stack([A[:, 1] - B[:, 1], B[:, 0] - A[:, 0]], 1)
        sx = (N * (A - Y)).sum(1)
        k = (sx.abs() <= N.abs().sum(1) * (1 + 1e-9)) & (N.abs().sum(1) > 0) & ~solid_at(Y)
        p, Y, N, sx = p[k], Y[k], N[k], sx[k]
        base = sum(Y[:, a] * stride[a] for a in range(dim)) * len(dirs)
        size = (N * N).sum(1)
        for d in range(len(dirs)):
            c = cs[d].double()
            D = (N * c).sum(1)
            tt = sx / D
            H = Y + tt[:, None] * c
            ok = (D != 0) & (tt >= 0) & (tt <= 1)
            for v in range(dim):
                U, Z = W[p, v], W[p, (v + 1) % dim]
                if dim == 3:
                    ok &= (N * torch.linalg.cross(Z - U, H - U)).sum(1) >= -1e-12 * size
                elif v == 0:
                    e = ((H - U) * (Z - U)).sum(1)
                    ok &= (e >= -1e-12 * size) & (e <= size * (1 + 1e-12))
            kk = (base + d)[ok]
            j = torch.searchsorted(key, kk).clamp(max=key.numel() - 1)
            hit = key[j] == kk
            pos.append(order[j[hit]])
            ts.append(tt[ok][hit])
            who.append(p[ok][hit])
    pos, ts, who = torch.cat(pos), torch.cat(ts), torch.cat(who)
    q = torch.full((X.shape[0],), math.inf, dtype=torch.float64, device=dev)
    q.scatter_reduce_(0, pos, ts, "amin")
    prim = torch.zeros(X.shape[0], dtype=torch.long, device=dev)
    best = ts == q[pos]
    prim[pos[best]] = who[best]
    return {"X": X, "c": cs[s], "q": q, "prim": prim}


def _q_gradient(case, V, T, t, w):
    """dL/dV for L = sum w q: dq/dv_j = lambda_j n / (n . d), lambda the barycentrics of the hit point."""
    h = 0.5 ** case["lf"]
    ids = T.long()[t["prim"]]
    A, B, C = V[ids].unbind(1)
    d = t["c"].double() * h
    N = torch.linalg.cross(B - A, C - A)
    H = (t["X"] + 0.5) * h + t["q"][:, None] * d
    f = (w / (N * d).sum(1))[:, None] * N
    g = torch.zeros_like(V)
    for j, (U, Z) in enumerate(((B, C), (C, A), (A, B))):
        lam = (N * torch.linalg.cross(U - H, Z - H)).sum(1) / (N * N).sum(1)
        g.index_add_(0, ids[:, j], lam[:, None] * f)
    return g


def _bounce_back(case, seed, coord, solid, cell, dr, q):
    """The streamed populations after the wall step, in float64."""
    dev, nb, L = "cuda", coord.shape[0], case["lf"]
    dirs = _directions(case["lattice"])
    post, new = (f.double() for f in _populations(case, nb, seed))
    pslot = torch.full((27,), -1, dtype=torch.long, device=dev)
    pslot[torch.tensor(sorted([k for k, _ in dirs] + [13]), device=dev)] = torch.arange(len(dirs) + 1, device=dev)
    n = [v // 4 << L for v in _n0(case)]
    grid = torch.full((n[0] * n[1] * n[2],), -1, dtype=torch.long, device=dev)
    cl = coord.long()
    grid[cl[:, 0] + n[0] * (cl[:, 1] + n[1] * cl[:, 2])] = torch.arange(nb, device=dev)
    b, t, k = cell.long() >> 6, cell.long() & 63, dr.long()
    fp = post[b, pslot[k], t]
    v = fp
    if case["interpolate"]:
        c = torch.stack([k % 3 - 1, k // 3 % 3 - 1, k // 9 - 1], 1)
        U = 4 * cl[b] + torch.stack([t & 3, t >> 2 & 3, t >> 4], 1) - c
        dom = torch.ones_like(b, dtype=torch.bool)
        i = torch.zeros_like(b)
        for a, s in zip(range(3), (1, n[0], n[0] * n[1])):
            dom &= (U[:, a] >= 0) & (U[:, a] < 4 * n[a])
            i += (U[:, a] >> 2).clamp(0, n[a] - 1) * s
        ub = torch.where(dom, grid[i], -1)
        ut = (U[:, 0] & 3) + 4 * (U[:, 1] & 3) + 16 * (U[:, 2] & 3)
        ok = (ub >= 0) & (solid[ub.clamp(min=0)] >> ut & 1 == 0)
        qq = q.double()
        up = post[ub.clamp(min=0), pslot[k], ut]
        far = fp / (2 * qq) + (1 - 1 / (2 * qq)) * post[b, pslot[26 - k], t]
        v = torch.where(qq >= 0.5, far, torch.where(ok, 2 * qq * fp + (1 - 2 * qq) * up, fp))
    new = new.clone()
    new[b, pslot[26 - k], t] = v
    return new
