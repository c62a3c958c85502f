"""Volumes, surfaces and centroid sums recounted on the GPU against their
definition, at the edges of the reductions' bricks and runs: ragged and tiny
sides, more labels in a brick than its map holds, cells across the periodic
boundary, rows that are not whole vectors; single lattices and batches."""
import numpy as np
import pytest

from paper_2312_09317_amd import cpm, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    cpm.load()
    return torch


def _expected(lat, n):
    """lat: (z, y, x)."""
    ndim = 3 if lat.shape[0] > 1 else 2
    V = np.bincount(lat[lat > 0], minlength=n + 1)
    S = np.zeros(n + 1, dtype=np.int64)
    for dz in (-1, 0, 1) if ndim == 3 else (0,):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                unlike = (np.roll(lat, (dz, dy, dx), (0, 1, 2)) != lat) & (lat > 0)
                S += np.bincount(lat[unlike], minlength=n + 1)
    C = np.zeros((n + 1, ndim), dtype=np.int64)
    flat = lat.reshape(-1)
    dims = lat.shape[::-1]
    sites = np.flatnonzero(flat > 0)
    labels = flat[sites]
    ref = np.full(n + 1, 2 ** 31 - 1, dtype=np.int64)
    np.minimum.at(ref, labels, sites)
    pitch = 1
    for d in range(ndim):
        L = dims[d]
        p, r = sites // pitch % L, ref[labels] // pitch % L
        diff = p - r
        diff = np.where(diff > L // 2, diff - L, diff)
        diff = np.where(diff < -((L - 1) // 2), diff + L, diff)
        np.add.at(C[:, d], labels, r + diff)
        pitch *= L
    return V, S, C


LATTICES = [
    # dims, cells, lattice
    ((2, 2), 3, "noise"), ((6, 34), 5, "noise"), ((66, 70), 2000, "noise"), ((130, 64), 12, "blobs"),
    ((256, 258), 300, "blobs"), ((2, 4, 6), 4, "noise"), ((18, 16, 34), 3000, "noise"), ((16, 48, 16), 20, "blobs"),
    ((50, 14, 30), 40, "blobs"), ((32, 32, 32), 1, "all"),
]


def _make(case):
    dims, n, kind = LATTICES[case]
    shape = tuple(dims) + (1,) * (3 - len(dims))
    if kind == "all":
        lat = np.ones(shape[::-1], dtype=np.int32)
    elif kind == "noise":
        lat = inputs.random_labels(shape, n, 5 + case, p_obstacle=0.05)
    else:
        lat = inputs.random_blobs(shape, n, seed=5 + case, fill=0.7, p_obstacle=0.02)
    p = cpm.Params(ndim=len(dims), dims=dims, J=np.zeros((3, 3)), lambda_volume=[0, 1, 0], volume_target=[0, 10, 0],
                   obstacle_type=2, sub=1)
    return p, np.ascontiguousarray(lat.reshape(shape[::-1])), n


@pytest.mark.parametrize("case", range(len(LATTICES)))
def test_cell_stats(torch_cuda, case):
    p, lat, n = _make(case)
    print(f"cell stats of {LATTICES[case]}", flush=True)
    sim = cpm.Simulation(p, lat, np.array([0] + [1] * n, dtype=np.int32))
    V, S, C = _expected(lat, n)
    for centroids in (True, False):
        v, s, c = sim.cell_stats(centroids)
        np.testing.assert_array_equal(v.cpu().numpy()[1:], V[1:])
        np.testing.assert_array_equal(s.cpu().numpy()[1:], S[1:])
        if centroids:
            np.testing.assert_array_equal(c.cpu().numpy()[1:], C[1:])


@pytest.mark.parametrize("ndim", [2, 3])
def test_batch_cell_stats(torch_cuda, ndim):
    made = [m for m in map(_make, range(len(LATTICES))) if m[0].c.ndim == ndim]
    print(f"batch cell stats, {len(made)} lattices", flush=True)
    b = cpm.Batch([m[0] for m in made], [m[1] for m in made], [np.array([0] + [1] * m[2], dtype=np.int32) for m in made])
    v, s, c = (t.cpu().numpy() for t in b.cell_stats())
    c = c.reshape(-1, ndim)
    for i, (_, lat, n) in enumerate(made):
        lo = int(b.label_off[i])
        V, S, C = _expected(lat, n)
        np.testing.assert_array_equal(v[lo + 1:lo + n + 1], V[1:])
        np.testing.assert_array_equal(s[lo + 1:lo + n + 1], S[1:])
        np.testing.assert_array_equal(c[lo + 1:lo + n + 1], C[1:])
