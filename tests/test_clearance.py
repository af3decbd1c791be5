"""The clearance grid that an upload builds (CPU): which cells triangles touch, the
distances, and the meshes that get none."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from synth import kuhn_mesh

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2103_02309_amd", "csrc")


@pytest.fixture(scope="module")
def grid_of(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    tmp = tmp_path_factory.mktemp("clear")
    out = str(tmp / "driver")
    subprocess.run([gxx, "-std=c++17", "-O1", "-pthread", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "clear_driver.cpp"), os.path.join(CSRC, "pack.cpp"), "-o", out],
                   check=True)

    def run(points, tets, nbrs, cflag):
        path = str(tmp / "mesh.bin")
        with open(path, "wb") as fh:
            fh.write(np.array([len(points), len(tets)], np.int64).tobytes())
            for a, dt in ((points, np.float32), (tets, np.int32), (nbrs, np.int32), (cflag, np.uint8)):
                fh.write(np.ascontiguousarray(a, dt).tobytes())
        r = subprocess.run([out, path], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout + r.stderr
        lines = r.stdout.splitlines()
        h = lines[0].split()
        R = tuple(int(x) for x in h[1:4])
        if int(h[0]) == 0:
            return None, R, None
        return np.array(lines[1].split(), np.int64).reshape(R), R, np.array([float(x) for x in h[4:7]])

    return run


def _triangles(m):
    t, j = np.nonzero(m.cflag)
    return np.stack([np.delete(m.tets[a], b) for a, b in zip(t, j)])


@pytest.mark.parametrize("n,scale", [(1, (1, 1, 1)), (5, (1, 1, 1)), (9, (1, 1, 1)), (6, (4, 1, 0.5))])
def test_cells_and_distances(grid_of, n, scale):
    spheres = [[0.5, 0.5, 0.5, 0.3], [0.2, 0.3, 0.7, 0.2]]
    m = kuhn_mesh(n, jitter=0.1, seed=n, spheres=spheres)
    pts = (m.points * np.array(scale, np.float32)).astype(np.float32)
    D, R, inv = grid_of(pts, m.tets, m.nbrs, m.cflag)
    assert D is not None and D.min() >= 0
    if not m.cflag.any():
        assert (D == 255).all()
        return
    tri = pts[_triangles(m)].astype(np.float64) * inv          # cell coordinates (the box starts at 0)
    # points of every triangle lie in touched cells, whichever side of a border they fall on
    rng = np.random.default_rng(0)
    w = rng.dirichlet([0.5, 0.5, 0.5], size=400)
    p = np.einsum("kc,tca->tka", w, tri).reshape(-1, 3)
    for off in ([0, 0, 0], [3e-3, 3e-3, 3e-3], [-3e-3, -3e-3, -3e-3], [3e-3, -3e-3, 0]):
        c = np.floor(p + np.array(off)).astype(int)
        ok = ((c >= 0) & (c < np.array(R))).all(1)
        assert (D[tuple(c[ok].T)] == 0).all()
    # and touched cells have a triangle near: samples within half a cell of the box
    touched = np.argwhere(D == 0)
    for c in touched[:: max(1, len(touched) // 60)]:
        d = np.maximum(np.maximum(c - p, p - (c + 1)), 0).max(1)
        assert d.min() < 0.5
    # distances: Chebyshev, in cells
    grid = np.argwhere(np.ones(R, bool))
    for g in grid[:: max(1, len(grid) // 300)]:
        assert D[tuple(g)] == np.abs(touched - g).max(1).min()


def test_meshes_without_a_grid(grid_of):
    m = kuhn_mesh(4, jitter=0.1, seed=1)
    assert grid_of(m.points, m.tets, m.nbrs, m.cflag)[0] is not None
    # a hole inside: its faces bound the mesh away from the box
    gone = 6 * ((1 * 4 + 2) * 4 + 1)
    keep = np.array([t for t in range(m.n_tets) if t != gone])
    new = np.full(m.n_tets, -1)
    new[keep] = np.arange(len(keep))
    nbrs = np.where(m.nbrs[keep] >= 0, new[m.nbrs[keep]], -1)
    cflag = np.where(nbrs >= 0, m.cflag[keep], 0)
    assert grid_of(m.points, m.tets[keep], nbrs, cflag)[0] is None
    # a corner pulled in: the boundary leaves the box's planes
    pts = m.points.copy()
    pts[0] += 0.05
    assert grid_of(pts, m.tets, m.nbrs, m.cflag)[0] is None
    # two grids on top of each other: the volumes add up to twice the box
    T, P = m.n_tets, m.n_points
    assert grid_of(np.concatenate([m.points, m.points]), np.concatenate([m.tets, m.tets + P]),
                   np.concatenate([m.nbrs, np.where(m.nbrs >= 0, m.nbrs + T, -1)]),
                   np.concatenate([m.cflag, m.cflag]))[0] is None
    # far from the origin: float32 positions too coarse for the cells
    assert grid_of(np.round(m.points * 64) / 64 + 4096.0, m.tets, m.nbrs, m.cflag)[0] is None
