"""The work that programs have this library do, as a list of cases to measure.

Scenes are Kuhn grids of the unit cube (6 tets per cell, jittered vertices) in
which the faces between cells inside and outside a union of spheres are the
scene's triangles, as in the library's tests and benchmark: from 16 cells per
axis (24,576 tets) to 128 (12,582,912).  Rays are what renderers trace through
them: camera rays in 8x8 pixel tiles, cosine-weighted ambient-occlusion rays
and shadow rays that leave the camera rays' hits, rays between random points,
and rays aimed through vertices and along edges for the precision variant.

A scene depends on its case alone and stays uploaded, as a program keeps its
scene; camera, light and rays come from the seed.  Scenes, rays and the 64-bit
results (`exact`) are built here with torch and use none of the library: a
plane-test walk in float64, or every triangle against every ray.
"""
import math

import numpy as np
import torch

import paper_2103_02309_amd as tetrt

DEV = torch.device("cuda:0")
PERMS = ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0))
LAYOUTS = ("tet16", "tet20", "tet32", "tet32n")


# ---- the cases -----------------------------------------------------------------------

def listed():
    return [
        # a renderer places its camera: one point located, nothing else to hide the latency
        dict(name="locate_camera", kind="locate", n=128, spheres=20, layout="tet16", rays=1),
        # a preview thumbnail of a small scene, each ray finding its own start, allocating call
        dict(name="camera_thumbnail", kind="camera", n=16, spheres=1, layout="tet20", width=64, height=64,
             own_start=True, tets=False, eps=0.0),
        # a ragged viewport of a mid-size scene that also wants the tets beside each hit
        dict(name="camera_viewport", kind="camera", n=64, spheres=20, layout="tet20", width=500, height=375,
             own_start=False, tets=True, eps=0.0),
        # the benchmark's primary pass: a full-HD frame of the large scene
        dict(name="camera_hd", kind="camera", n=128, spheres=20, layout="tet16", width=1920, height=1080,
             own_start=False, tets=False, eps=0.0),
        # its ambient-occlusion pass: 8 rays per hit (about 10 million), binned by the automatic rule
        dict(name="ao_hd", kind="ao", n=128, spheres=20, layout="tet16", width=1920, height=1080, per_hit=8,
             tmax=0.1, eps=0.0),
        # one occlusion ray per hit of a small window: too few to be binned
        dict(name="ao_window", kind="ao", n=64, spheres=20, layout="tet16", width=403, height=301, per_hit=1,
             tmax=0.1, eps=0.0),
        # shadow rays of a 1024^2 frame towards one light, long and ending at it
        dict(name="shadow_frame", kind="shadow", n=96, spheres=20, layout="tet16", width=1024, height=1024, eps=0.0),
        # visibility queries with no order at all, each ray locating its own origin
        dict(name="random_queries", kind="random", n=64, spheres=20, layout="tet16", rays=1000003, eps=0.0),
        # the precision variant on rays through vertices and along edges
        dict(name="precision_stress", kind="precision", n=16, spheres=1, layout="tet16", rays=300007, eps=1e-6),
        # the precision variant for a whole frame of the large scene
        dict(name="precision_hd", kind="camera", n=128, spheres=20, layout="tet16", width=1280, height=720,
             own_start=False, tets=False, eps=1e-6),
        # many small and mid-size scenes traced by one batched launch, camera and occlusion rays
        dict(name="batch_scenes", kind="batch", n=64, meshes=10, layout="tet16", rays=400000, eps=0.0),
        # a burst of uneven requests to the server: submit, run to completion, collect
        dict(name="serve_burst", kind="serve", n=64, meshes=4, layout="tet16", requests=20, side=1024, eps=0.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["locate", "camera", "camera", "ao", "ao", "shadow", "random", "precision", "batch", "serve"])
    n = _log(rng, 8, 128)
    layout = rng.choice(["tet16", "tet16", "tet16", "tet20", "tet20", "tet32", "tet32n"])
    spheres = rng.choice([1, 5, 20]) if n >= 24 else 1
    eps = rng.choice([0.0, 0.0, 0.0, 1e-6])
    c = dict(kind=kind, n=n, spheres=spheres, layout=layout)
    if kind == "locate":
        c.update(rays=_log(rng, 1, 1000000))
    elif kind == "camera":
        c.update(width=_log(rng, 8, 1920), height=_log(rng, 8, 1080), own_start=rng.random() < 0.5,
                 tets=rng.random() < 0.25, eps=eps)
    elif kind == "ao":
        c.update(width=_log(rng, 16, 1600), height=_log(rng, 16, 900), per_hit=rng.choice([1, 4, 8]),
                 tmax=rng.choice([0.05, 0.1, 0.3]), eps=eps)
    elif kind == "shadow":
        c.update(width=_log(rng, 16, 1600), height=_log(rng, 16, 900), eps=eps)
    elif kind == "random":
        c.update(rays=_log(rng, 100, 1000000), eps=eps)
    elif kind == "precision":
        c.update(n=_log(rng, 8, 24), spheres=1, rays=_log(rng, 1000, 400000), eps=rng.choice([1e-6, 1e-5]))
    elif kind == "batch":
        del c["spheres"]
        c.update(n=min(n, 72), meshes=rng.randint(2, 12), layout=rng.choice(["tet16", "tet20"]),
                 rays=_log(rng, 2000, 500000), eps=eps)
    else:
        del c["spheres"]
        c.update(n=min(n, 72), meshes=rng.randint(1, 4), layout="tet16", requests=rng.randint(1, 20),
                 side=rng.choice([64, 128, 256, 512, 1024]), eps=eps)
    return c


# ---- scenes --------------------------------------------------------------------------

class Scene:
    """A Kuhn grid on the GPU: points [P, 3] float32, tets and nbrs [T, 4] int32, cflag
    [T, 4] uint8, field [T, 4] (the neighbour, -1 at the boundary, -2 - id across
    triangle id) and the triangles: vertices ascending [F, 3], the two tets [F, 2] and
    the face's slot in each."""

    def __init__(self, n, spheres):
        g = torch.Generator(device=DEV).manual_seed(1000 * n + spheres)
        n1 = n + 1
        ax = torch.arange(n1, device=DEV)
        grid = torch.stack(torch.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
        inner = ((grid > 0) & (grid < n)).all(1, keepdim=True)
        jit = (torch.rand(grid.shape, device=DEV, generator=g, dtype=torch.float64) * 0.2 - 0.1) * inner
        self.points = ((grid + jit) / n).float()
        del jit, inner, grid
        ax = torch.arange(n, device=DEV)
        cc = torch.stack(torch.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
        ctr = (cc + 0.5) / n
        if spheres == 1:
            ball = [(0.5, 0.5, 0.5, 0.35)]
        else:
            rs = np.random.default_rng(spheres + 2)
            ball = np.concatenate([rs.uniform(0.15, 0.85, (spheres, 3)), rs.uniform(0.03, 0.12, (spheres, 1))], 1)
        inside = torch.zeros(n ** 3, dtype=torch.bool, device=DEV)
        for x, y, z, r in ball:
            inside |= (ctr[:, 0] - float(x)) ** 2 + (ctr[:, 1] - float(y)) ** 2 + (ctr[:, 2] - float(z)) ** 2 < float(r) ** 2
        del ctr
        at = torch.tensor([n1 * n1, n1, 1], device=DEV)
        vid = (cc * at).sum(1)
        cell = torch.arange(n ** 3, device=DEV)
        step = (n * n, n, 1)
        T = 6 * n ** 3
        self.tets = torch.empty((n ** 3, 6, 4), dtype=torch.int32, device=DEV)
        self.nbrs = torch.empty((n ** 3, 6, 4), dtype=torch.int32, device=DEV)
        flag = torch.zeros((n ** 3, 6, 4), dtype=torch.bool, device=DEV)
        for m, p in enumerate(PERMS):
            odd = m in (1, 2, 5)
            v = [vid, vid + at[p[0]], vid + at[p[0]] + at[p[1]], vid + at.sum()]
            nb, fl = [None] * 4, [torch.zeros_like(inside)] * 4
            # across the cell's face at x[p0] = c + 1, and at x[p2] = c
            for slot, a, sign, to in ((0, p[0], 1, (p[1], p[2], p[0])), (3, p[2], -1, (p[2], p[0], p[1]))):
                ok = (cc[:, a] + sign >= 0) & (cc[:, a] + sign < n)
                other = torch.where(ok, cell + sign * step[a], 0)
                nb[slot] = torch.where(ok, other * 6 + PERMS.index(to), -1)
                fl[slot] = ok & (inside != inside[other])
            nb[1] = cell * 6 + PERMS.index((p[1], p[0], p[2]))
            nb[2] = cell * 6 + PERMS.index((p[0], p[2], p[1]))
            for k, s in enumerate((0, 1, 3, 2) if odd else (0, 1, 2, 3)):
                self.tets[:, m, k], self.nbrs[:, m, k], flag[:, m, k] = v[s].int(), nb[s].int(), fl[s]
        self.tets, self.nbrs, flag = self.tets.view(T, 4), self.nbrs.view(T, 4), flag.view(T, 4)
        self.cflag = flag.to(torch.uint8)
        # triangle ids: flagged faces (t, slot) in order, a face seen before keeps its id
        ts, sl = torch.nonzero(flag, as_tuple=True)
        nb = self.nbrs[ts, sl].long()
        first = (nb < 0) | (ts < nb)
        ft, fs, fn = ts[first], sl[first], nb[first]
        ms = (self.nbrs[fn.clamp(min=0)] == ft[:, None].int()).int().argmax(1)
        ids = torch.arange(ft.numel(), device=DEV)
        self.field = self.nbrs.clone()
        self.field[ft, fs] = (-2 - ids).int()
        has = fn >= 0
        self.field[fn[has], ms[has]] = (-2 - ids[has]).int()
        keep = torch.tensor([[1, 2, 3], [0, 2, 3], [0, 1, 3], [0, 1, 2]], device=DEV)
        self.tri = self.tets[ft].long().gather(1, keep[fs]).sort(1).values
        self.tri_tets, self.tri_slots = torch.stack([ft, fn], 1), torch.stack([fs, ms], 1)
        self.n, self.tri_count = n, int(ft.numel())

    def upload(self, layout):
        return tetrt.upload(self.points.cpu().numpy(), self.tets.cpu().numpy(), self.nbrs.cpu().numpy(),
                            self.cflag.cpu().numpy(), layout=layout)


_scenes, _meshes = {}, {}


def scene(n, spheres):
    if (n, spheres) not in _scenes:
        _scenes[n, spheres] = Scene(n, spheres)
    return _scenes[n, spheres]


def mesh(n, spheres, layout):
    if (n, spheres, layout) not in _meshes:
        _meshes[n, spheres, layout] = scene(n, spheres).upload(layout)
    return _meshes[n, spheres, layout]


def parts(c):
    """The scenes of a case with several: cells per axis and spheres of each."""
    r = np.random.default_rng(77 + c["n"])
    out = [(c["n"], 20 if c["n"] >= 24 else 1)]
    while len(out) < c["meshes"]:
        n = int(round(math.exp(r.uniform(math.log(8), math.log(c["n"] + 1)))))
        out.append((n, 5 if n >= 24 else 1))
    return out


# ---- float64 reference ---------------------------------------------------------------

def _exit(S, o, d, cur, jin):
    """Slot of the face through which the line leaves each tet, and its parameter."""
    P = [S.points[S.tets[cur, k].long()].double() - o for k in range(4)]
    best = torch.full(o.shape[:1], math.inf, dtype=torch.float64, device=DEV)
    slot = torch.zeros_like(cur)
    for j, (a, b, e) in enumerate(((1, 3, 2), (0, 2, 3), (0, 3, 1), (0, 1, 2))):
        nrm = torch.linalg.cross(P[b] - P[a], P[e] - P[a])
        nd = -(nrm * d).sum(1)
        s = -(nrm * P[a]).sum(1) / nd
        take = (nd > 0) & (jin != j) & (s < best)
        best = torch.where(take, s, best)
        slot = torch.where(take, torch.full_like(slot, j), slot)
    return slot, best


def locate(S, p):
    """The tet that holds each point (float64 [m, 3]): a walk from the cell's own tets."""
    c = (p * S.n).long().clamp(0, S.n - 1)
    cur = ((c[:, 0] * S.n + c[:, 1]) * S.n + c[:, 2]) * 6
    s0 = S.points[S.tets[cur].long()].double().mean(1)
    d = p - s0
    jin, act = torch.full_like(cur, -1), torch.arange(cur.numel(), device=DEV)
    for _ in range(64):
        if not act.numel():
            break
        j, s = _exit(S, s0[act], d[act], cur[act], jin[act])
        nb = S.nbrs[cur[act], j].long()
        go = (s < 1.0) & (nb >= 0)
        act, nb, old = act[go], nb[go], cur[act[go]]
        jin[act] = (S.nbrs[nb] == old[:, None].int()).int().argmax(1)
        cur[act] = nb
    return cur


def on_triangle(S, o, d, tri):
    """t and the weights of the 2nd and 3rd vertex where rays meet their triangles' planes."""
    A, B, C = (S.points[S.tri[tri, k]].double() for k in range(3))
    e1, e2, s = B - A, C - A, o - A
    p, q = torch.linalg.cross(d, e2), torch.linalg.cross(s, e1)
    det = (e1 * p).sum(1)
    return (e2 * q).sum(1) / det, torch.stack([(s * p).sum(1) / det, (d * q).sum(1) / det], 1)


def walk(S, o, d, cur, jin, tmax):
    """Closest triangle along each ray from tet to tet (float64): tri, t, bary."""
    m = o.shape[0]
    tri = torch.full((m,), -1, dtype=torch.long, device=DEV)
    act = torch.arange(m, device=DEV)
    cur, jin = cur.clone(), jin.clone()
    for _ in range(40 * S.n + 100):
        if not act.numel():
            break
        j, s = _exit(S, o[act], d[act], cur, jin)
        f = S.field[cur, j].long()
        hit = f < -1
        tri[act[hit]] = -2 - f[hit]
        go = (f >= 0) & (s <= tmax[act])
        act, f, old = act[go], f[go], cur[go]
        jin, cur = (S.nbrs[f] == old[:, None].int()).int().argmax(1), f
    return _result(S, o, d, tri, tmax)


def closest_of_all(S, o, d, tmax):
    """The same from every triangle against every ray: the lowest id within 1e-12 of the nearest."""
    tri = torch.full(o.shape[:1], -1, dtype=torch.long, device=DEV)
    A, B, C = (S.points[S.tri[:, k]].double()[None] for k in range(3))
    e1, e2 = B - A, C - A
    rows = max(1, (1 << 25) // S.tri_count)
    for i in range(0, o.shape[0], rows):
        O, D = o[i:i + rows, None], d[i:i + rows, None]
        p = torch.linalg.cross(D.expand(-1, S.tri_count, -1), e2.expand(O.shape[0], -1, -1))
        s = O - A
        q = torch.linalg.cross(s, e1.expand(O.shape[0], -1, -1))
        det = (e1 * p).sum(2)
        u, v, t = (s * p).sum(2) / det, (D * q).sum(2) / det, (e2 * q).sum(2) / det
        ok = (det != 0) & (u >= 0) & (v >= 0) & (u + v <= 1) & (t > 0) & (t <= tmax[i:i + rows, None])
        t = torch.where(ok, t, math.inf)
        near = t.min(1).values
        k = (t <= near[:, None] + 1e-12).int().argmax(1)
        tri[i:i + rows] = torch.where(torch.isfinite(near), k, -1)
    return _result(S, o, d, tri, tmax)


def _result(S, o, d, tri, tmax):
    hit = tri >= 0
    t = torch.full(tri.shape, math.nan, dtype=torch.float64, device=DEV)
    bary = torch.full((tri.numel(), 2), math.nan, dtype=torch.float64, device=DEV)
    t[hit], bary[hit] = on_triangle(S, o[hit], d[hit], tri[hit])
    late = t > tmax
    t[late], bary[late], tri[late] = math.nan, math.nan, -1
    return tri, t, bary


# ---- rays ----------------------------------------------------------------------------

def _unit(v):
    return v / torch.linalg.vector_norm(v, dim=-1, keepdim=True)


def _pose(rs):
    """A camera near the cube's front face that looks roughly along +z."""
    eye = np.array([rs.uniform(0.4, 0.6), rs.uniform(0.4, 0.6), rs.uniform(0.02, 0.06)])
    return eye, np.array([rs.uniform(-0.15, 0.15), rs.uniform(-0.15, 0.15), 1.0])


def camera(eye, fwd, W, H, fov=60.0):
    """Float32 origins and directions of a pinhole camera, pixels in 8x8 tiles."""
    f = fwd / np.linalg.norm(fwd)
    r = np.cross(f, (0.0, 1.0, 0.0) if abs(f[1]) < 0.9 else (1.0, 0.0, 0.0))
    r /= np.linalg.norm(r)
    u = np.cross(r, f)
    f, r, u = (torch.tensor(x, device=DEV) for x in (f, r, u))
    ar = lambda k: torch.arange(k, device=DEV)  # noqa: E731
    ty, tx, iy, ix = torch.meshgrid(ar((H + 7) // 8), ar((W + 7) // 8), ar(8), ar(8), indexing="ij")
    py, px = (ty * 8 + iy).reshape(-1), (tx * 8 + ix).reshape(-1)
    keep = (py < H) & (px < W)
    py, px = py[keep].double(), px[keep].double()
    th = math.tan(math.radians(fov) / 2)
    d = _unit(f + ((2 * (px + 0.5) / W - 1) * th)[:, None] * r + ((1 - 2 * (py + 0.5) / H) * th * (H / W))[:, None] * u)
    o = torch.tensor(eye, device=DEV).float().expand(d.shape[0], 3).contiguous()
    return o, d.float()


def camera_hits(S, o, d):
    """The first hits of camera rays in image order, in float64, 6 for every 10 rays (from the
    start again where the image has fewer): triangle, point, facing normal."""
    O, D = o.double(), d.double()
    cur = locate(S, O[:1]).expand(O.shape[0])
    far = torch.full(O.shape[:1], math.inf, dtype=torch.float64, device=DEV)
    tri, t, _ = walk(S, O, D, cur, torch.full_like(cur, -1), far)
    p = O + t[:, None] * D
    if not (tri >= 0).any():   # nothing in view: the triangles' centres
        tri = torch.arange(O.shape[0], device=DEV) % S.tri_count
        p = S.points[S.tri[tri]].double().mean(1)
    hit = torch.nonzero(tri >= 0).reshape(-1)
    hit = hit[torch.arange(hit_count(O.shape[0]), device=DEV) % hit.numel()]
    tri = tri[hit]
    A, B, C = (S.points[S.tri[tri, k]].double() for k in range(3))
    nrm = _unit(torch.linalg.cross(B - A, C - A))
    nrm = torch.where(((nrm * D[hit]).sum(1) > 0)[:, None], -nrm, nrm)
    return tri, p[hit], nrm


def hit_count(rays):
    return max(1, (6 * rays) // 10)


def hemisphere(nrm, k, gen):
    """k cosine-weighted directions about each normal."""
    m = nrm.shape[0]
    u1, u2 = torch.rand((2, m, k, 1), device=DEV, generator=gen, dtype=torch.float64)
    a = torch.where((nrm[:, :1].abs() < 0.9), torch.tensor([[1.0, 0, 0]], device=DEV, dtype=torch.float64),
                    torch.tensor([[0, 1.0, 0]], device=DEV, dtype=torch.float64))
    t1 = _unit(torch.linalg.cross(a, nrm))
    t2 = torch.linalg.cross(nrm, t1)
    ph = 2 * math.pi * u2
    return _unit(u1.sqrt() * (ph.cos() * t1[:, None] + ph.sin() * t2[:, None]) + (1 - u1).sqrt() * nrm[:, None])


def rays_of(S, c, seed):
    """The rays of a case with one scene: orig, dirs and the optional arrays."""
    rs, gen = np.random.default_rng(seed), torch.Generator(device=DEV).manual_seed(int(seed))
    kind = c["kind"]
    if kind in ("camera", "ao", "shadow"):
        eye, fwd = _pose(rs)
        o, d = camera(eye, fwd, c["width"], c["height"])
        if kind == "camera":
            a = dict(orig=o, dirs=d)
            if not c["own_start"]:   # the camera's tet, located once by the program
                a["start_tet"] = locate(S, o[:1].double()).int().expand(o.shape[0]).contiguous()
            return a
        tri, p, nrm = camera_hits(S, o, d)
        if kind == "ao":
            k = c["per_hit"]
            d = hemisphere(nrm, k, gen).reshape(-1, 3)
            tm = torch.full((d.shape[0],), c["tmax"], device=DEV)
            return dict(orig=p.float().repeat_interleave(k, 0), dirs=d.float(), tmax=tm,
                        start_face=tri.int().repeat_interleave(k))
        light = torch.tensor([rs.uniform(0.1, 0.9), rs.uniform(0.8, 0.97), rs.uniform(0.05, 0.5)], device=DEV)
        o = p.float()
        return dict(orig=o, dirs=(light.float() - o).contiguous(), tmax=torch.ones(o.shape[0], device=DEV),
                    start_face=tri.int())
    m = c["rays"]
    o = torch.rand((m, 3), device=DEV, generator=gen, dtype=torch.float64) * 0.998 + 0.001
    d = _unit(torch.randn((m, 3), device=DEV, generator=gen, dtype=torch.float64))
    if kind == "precision":
        k = m // 10
        v = torch.randint(S.points.shape[0], (k,), device=DEV, generator=gen)
        d[:k] = _unit(S.points[v].double() - o[:k])
        # along tet edges that are no edge of a scene triangle
        P = S.points.shape[0]
        e = torch.cat([S.tri[:, [0, 1]], S.tri[:, [1, 2]], S.tri[:, [0, 2]]])
        e = (e[:, 0] * P + e[:, 1]).unique()
        t = torch.randint(S.tets.shape[0], (4 * k + 64,), device=DEV, generator=gen)
        s = torch.rand((t.numel(), 4), device=DEV, generator=gen).argsort(1)
        ab = S.tets[t].long().gather(1, s[:, :2])
        ab = ab[~torch.isin(ab.min(1).values * P + ab.max(1).values, e)][:k]
        k2 = ab.shape[0]
        A, B = S.points[ab[:, 0]].double(), S.points[ab[:, 1]].double()
        w = torch.rand((k2, 1), device=DEV, generator=gen, dtype=torch.float64) * 0.8 + 0.1
        o[k:k + k2], d[k:k + k2] = A + w * (B - A), _unit(B - A)
    return dict(orig=o.float(), dirs=d.float())


def batch_rays(S, count, seed):
    """Camera rays and occlusion rays of one scene of a batch, about half each."""
    rs, gen = np.random.default_rng(seed), torch.Generator(device=DEV).manual_seed(int(seed))
    side = max(4, int(math.sqrt(count / 2.2)))
    eye, fwd = _pose(rs)
    o, d = camera(eye, fwd, side, side)
    tri, p, nrm = camera_hits(S, o, d)
    k = 2
    ad = hemisphere(nrm, k, gen).reshape(-1, 3).float()
    return [dict(orig=o, dirs=d), dict(orig=p.float().repeat_interleave(k, 0), dirs=ad,
                                       tmax=torch.full((ad.shape[0],), 0.1, device=DEV),
                                       start_face=tri.int().repeat_interleave(k))]


def batch_jobs(c, seed):
    r = np.random.default_rng(5 + c["n"])
    out = []
    for i, (n, spheres) in enumerate(parts(c)):
        count = int(c["rays"] * math.exp(r.uniform(math.log(0.02), 0.0)))
        out += [(n, spheres, a) for a in batch_rays(scene(n, spheres), max(64, count), 100 * seed + i)]
    return out


def requests_of(c, seed):
    rs = np.random.default_rng(seed)
    shape = np.random.default_rng(9 + c["requests"])   # what is asked for: the case's; from where: the seed's
    out = []
    for i in range(c["requests"]):
        kind = ("primary", "primary", "shadow", "ao")[shape.integers(4)]
        side = max(64, c["side"] >> int(shape.integers(3)))
        fwd = rs.normal(size=3)
        fwd /= np.linalg.norm(fwd)
        up = (0.0, 1.0, 0.0) if abs(fwd[1]) < 0.9 else (1.0, 0.0, 0.0)
        out.append(dict(mesh=int(shape.integers(c["meshes"])), kind=kind, width=side, height=side,
                        eye=tuple(rs.uniform(0.05, 0.95, 3)), forward=tuple(fwd), up=up, fov_h_deg=60.0,
                        light=tuple(rs.uniform(0.1, 0.9, 3)), ao_tmax=0.1, seed=int(rs.integers(1 << 31))))
    return out


# ---- prepare, run --------------------------------------------------------------------

def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "batch":
        # every job writes its own part of three result arrays
        parts_in = batch_jobs(c, seed)
        sizes = [a["orig"].shape[0] for _, _, a in parts_in]
        out = tetrt.outputs(sum(sizes), DEV)
        views = {k: v.split(sizes) for k, v in out.items()}
        jobs = [dict(a, mesh=mesh(n, spheres, c["layout"]), out={k: v[i] for k, v in views.items()})
                for i, (n, spheres, a) in enumerate(parts_in)]
        b = tetrt.Batch(len(jobs), sum(sizes))
        b.set(jobs, eps=c["eps"])
        return dict(kind=kind, batch=b, out=out)
    if kind == "serve":
        ms = [mesh(n, s, c["layout"]) for n, s in parts(c)]
        reqs = [dict(r, out=None) for r in requests_of(c, seed)]
        outs = [tetrt.outputs(r["width"] * r["height"], DEV) for r in reqs]
        srv = tetrt.Server(ms, max_rays=1 << 22, eps=c["eps"])
        return dict(kind=kind, server=srv, reqs=[tetrt.Server.prepare(**r) for r in reqs], outs=outs)
    m = mesh(c["n"], c["spheres"], c["layout"])
    a = rays_of(scene(c["n"], c["spheres"]), c, seed)
    st = dict(kind=kind, mesh=m, a=a, opts=dict(eps=c["eps"]) if c.get("eps") else {})
    if kind != "locate":
        n = a["orig"].shape[0]
        # small calls let the library allocate; frames are traced into buffers that the program keeps
        st["out"] = None if n <= 1 << 14 else tetrt.outputs(n, DEV, want_tets=c.get("tets", False))
        need = m.workspace_bytes(n, "tmax" in a, **st["opts"])
        st["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV) if need and st["out"] is not None else None
        st["tets"] = c.get("tets", False)
    return st


def run(st):
    kind = st["kind"]
    if kind == "locate":
        return st["mesh"].locate(st["a"]["orig"])
    if kind == "batch":
        st["batch"].launch()
        return st["out"]
    if kind == "serve":
        s = st["server"]
        for r, out in zip(st["reqs"], st["outs"]):
            s.submit_prepared(r, out)
        s.drain()
        s.poll()
        return st["outs"]
    if st["out"] is None:
        return st["mesh"].trace(want_tets=st["tets"], **st["a"], **st["opts"])
    return st["mesh"].trace_into(st["out"], workspace=st["ws"], **st["a"], **st["opts"])


# ---- what a pass cannot do without ---------------------------------------------------

def work(case):
    """Rays in, results out, and for each ray the triangle it ends on (three ids, three
    points) and one ray-triangle intersection (about 100 operations).  What a walk reads
    on the way there depends on the method and is not counted."""
    c, kind = case, case["kind"]
    if kind == "locate":
        return dict(bytes=c["rays"] * (12 + 4 + 64), flops=c["rays"] * 100)
    per = 24 + 16 + 48
    if kind == "camera":
        rays, per = c["width"] * c["height"], per + (0 if c["own_start"] else 4) + (8 if c["tets"] else 0)
    elif kind == "ao":
        rays, per = hit_count(c["width"] * c["height"]) * c["per_hit"], per + 8
    elif kind == "shadow":
        rays, per = hit_count(c["width"] * c["height"]), per + 8
    elif kind == "batch":
        r = np.random.default_rng(5 + c["n"])
        rays = sum(max(64, c["rays"] * math.exp(r.uniform(math.log(0.02), 0.0))) for _ in range(c["meshes"]))
    elif kind == "serve":
        px = [(r["width"] * r["height"], r["kind"]) for r in requests_of(c, 0)]
        rays = sum(p * (1 if k == "primary" else 2) for p, k in px)
    else:
        rays = c["rays"]
    return dict(bytes=rays * per, flops=rays * 100)


# ---- 64-bit results ------------------------------------------------------------------

def _exact_rays(S, c, a):
    O, D = a["orig"].double(), a["dirs"].double()
    tmax = a["tmax"].double() if "tmax" in a else torch.full(O.shape[:1], math.inf, dtype=torch.float64, device=DEV)
    if c["kind"] == "precision":
        tri, t, bary = closest_of_all(S, O, D, tmax)
    else:
        jin = torch.full(O.shape[:1], -1, dtype=torch.long, device=DEV)
        if "start_face" in a:
            # the tet on the side of the face that the ray points into
            f = a["start_face"].long()
            cent = S.points[S.tets[S.tri_tets[f, 0]].long()].double().mean(1)
            A, B, C = (S.points[S.tri[f, k]].double() for k in range(3))
            nrm = torch.linalg.cross(B - A, C - A)
            side = (((nrm * (cent - A)).sum(1) > 0) != ((nrm * D).sum(1) > 0)).long()
            cur = S.tri_tets[f].gather(1, side[:, None])[:, 0]
            jin = S.tri_slots[f].gather(1, side[:, None])[:, 0]
        elif "start_tet" in a:
            cur = a["start_tet"].long()
        else:
            cur = locate(S, O)
        tri, t, bary = walk(S, O, D, cur, jin, tmax)
    return dict(tri=tri.int(), t=t, bary=bary)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "locate":
        return locate(scene(c["n"], c["spheres"]), rays_of(scene(c["n"], c["spheres"]), c, seed)["orig"].double()).int()
    if kind == "batch":
        got = [_exact_rays(scene(n, s), c, a) for n, s, a in batch_jobs(c, seed)]
        return {k: torch.cat([g[k] for g in got]) for k in got[0]}
    if kind == "serve":
        # camera requests; shadow and occlusion rays leave float32 hit points of the server's own
        out, at = [], parts(c)
        for r in requests_of(c, seed):
            if r["kind"] != "primary":
                out.append(None)
                continue
            eye = np.array(r["eye"], np.float32).astype(np.float64)
            o, d = camera(eye, np.array(r["forward"], np.float32).astype(np.float64), r["width"], r["height"])
            out.append(_exact_rays(scene(*at[r["mesh"]]), c, dict(orig=o, dirs=d)))
        return out
    S = scene(c["n"], c["spheres"])
    out = _exact_rays(S, c, rays_of(S, c, seed))
    if c.get("tets"):
        out["hit_tets"] = None
    return out
