"""GPU checks of the summary statistics and the directional autocorrelation on
sample buffers written directly, at the edges of the reductions' work split:
cells per chunk, lags per thread, several workgroups per lattice, and series
too long for the step buffer of a full chunk."""
import numpy as np
import pytest

from oracle import summary as ref_summary
from paper_2312_09317_amd import cpm

pytestmark = pytest.mark.gpu


def _batch(ndim, n_cells):
    L = 8
    dims = (L,) * ndim
    params = [cpm.Params(ndim=ndim, dims=dims, J=np.zeros((2, 2)), lambda_volume=[0.0, 1.0], volume_target=[0, 10],
                         lattice_id=i) for i in range(len(n_cells))]
    lats = [np.zeros((L if ndim == 3 else 1, L, L), dtype=np.int32) for _ in n_cells]
    return cpm.Batch(params, lats, [np.array([0] + [1] * c, dtype=np.int32) for c in n_cells]), dims


def _samples(rng, K, n_cells, ndim, L):
    """(K, C + 1, 5): persistent walks, some cells resting or dead at times."""
    C = n_cells + 1
    rec = np.zeros((K, C, 5))
    rec[..., 0] = rng.integers(5, 40, (K, C))
    rec[..., 1] = rng.integers(20, 90, (K, C))
    drift = rng.normal(size=(1, C, ndim))
    hop = 0.4 * drift + 0.5 * rng.normal(size=(K, C, ndim))
    hop[rng.random((K, C)) < 0.1] = 0.0
    rec[..., 2:2 + ndim] = np.mod(rng.random((1, C, ndim)) * L + np.cumsum(hop, axis=0), L)
    dead = rng.random((K, C)) < 0.05
    rec[dead] = 0.0
    return rec


@pytest.mark.parametrize("ndim,K,n_cells", [
    (2, 1, (1, 3)),                # a single sample: no steps
    (2, 2, (1, 63)),               # one step, one lag
    (2, 5, (64, 0, 65)),           # kLags steps; chunk edges; a lattice without cells
    (2, 6, (128, 129)),            # one lag past a thread's
    (2, 41, (200, 7)),             # the emulator's plan
    (3, 41, (70,)),
    (2, 150, (33, 2)),             # chunks of 16 cells
    (3, 260, (9, 3)),              # smaller ones
])
def test_statistics_match_reference(ndim, K, n_cells):
    import torch
    rng = np.random.default_rng(K * 100 + ndim)
    b, dims = _batch(ndim, n_cells)
    recs = [_samples(rng, K, c, ndim, dims[0]) for c in n_cells]
    buf = torch.as_tensor(np.concatenate([r.reshape(-1) for r in recs])).cuda()
    out = b.summary(buf, K, 3.0)
    ac = b.autocorrelation(buf, K) if K > 1 else None
    again = b.summary(buf, K, 3.0)
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    for i, r in enumerate(recs):
        ref = ref_summary.summary(r[..., 0], r[..., 1], r[..., 2:2 + ndim], dims, 3.0)
        # sums of at most 1e6 terms of like size: a relative 1e6 * 2^-53, and
        # variances as differences of such sums
        np.testing.assert_allclose(out[i].cpu().numpy(), ref, rtol=1e-9, atol=1e-9)
        if ac is not None:
            s, n = ref_summary.autocorrelation(r[..., 0], r[..., 2:2 + ndim], dims)
            np.testing.assert_allclose(ac[i, :, 0].cpu().numpy(), s, rtol=1e-9, atol=1e-9)
            np.testing.assert_array_equal(ac[i, :, 1].cpu().numpy(), n)
    b.close()


def _autocorrelation(V, pos, dims):
    """ref_summary.autocorrelation of long series, by np.correlate."""
    d = np.diff(pos[:, 1:], axis=0)
    L = np.asarray(dims, dtype=np.float64)[:pos.shape[2]]
    d -= L * np.rint(d / L)
    norm = np.sqrt((d * d).sum(-1))
    ok = (V[:-1, 1:] > 0) & (V[1:, 1:] > 0) & (norm > 0)
    u = np.where(ok[..., None], d / np.where(ok, norm, 1.0)[..., None], 0.0)
    m = len(d)
    lags = lambda x: np.correlate(x, x, "full")[m - 1:]
    cells = range(d.shape[1])
    return (sum(lags(u[:, c, e]) for c in cells for e in range(d.shape[2])),
            np.rint(sum(lags(ok[:, c].astype(np.float64)) for c in cells)))


@pytest.mark.parametrize("ndim,K,n_cells,autocorrelation", [
    (2, 5200, (2, 1), False),  # one cell's steps no longer fit the LDS: the general kernels
    (3, 4100, (1,), False),
    (3, 3610, (1,), True),     # (met by one thread per cell: some seconds)
])
def test_series_beyond_the_step_buffer(ndim, K, n_cells, autocorrelation):
    import torch
    print(f"{ndim}D, {K} samples", flush=True)
    rng = np.random.default_rng(K + ndim)
    b, dims = _batch(ndim, n_cells)
    recs = [_samples(rng, K, c, ndim, dims[0]) for c in n_cells]
    for r in recs:  # no drift: the search for the persistence time ends early (one thread per cell)
        r[..., 2:2 + ndim] = rng.random(r[..., 2:2 + ndim].shape) * dims[0]
    buf = torch.as_tensor(np.concatenate([r.reshape(-1) for r in recs])).cuda()
    out = b.summary(buf, K, 3.0).cpu().numpy()
    for i, r in enumerate(recs):
        ref = ref_summary.summary(r[..., 0], r[..., 1], r[..., 2:2 + ndim], dims, 3.0)
        # sums of at most 1e4 terms of size 1: 1e4 * 2^-53, as above
        np.testing.assert_allclose(out[i], ref, rtol=1e-9, atol=1e-9)
    ac = b.autocorrelation(buf, K).cpu().numpy() if autocorrelation else None
    for i, r in enumerate(recs if autocorrelation else []):
        s, n = _autocorrelation(r[..., 0], r[..., 2:2 + ndim], dims)
        np.testing.assert_allclose(ac[i, :, 0], s, rtol=1e-9, atol=1e-9)
        np.testing.assert_array_equal(ac[i, :, 1], n)
    b.close()


def test_variances_of_one_value_and_of_like_values():
    # one cell: its persistence time has no variance, whatever the rounding of
    # its square; cells that move alike: no variance falls below zero
    import torch
    K, cells = 41, (1, 1, 1, 1, 3, 64, 70)
    b, dims = _batch(2, cells)
    rng = np.random.default_rng(9)
    recs = []
    for i, c in enumerate(cells):
        rec = np.repeat(_samples(rng, K, 1, 2, dims[0])[:, 1:], c + 1, axis=1)
        rec[rec[..., 0] == 0] = rec[0, 0]
        recs.append(rec)
    buf = torch.as_tensor(np.concatenate([r.reshape(-1) for r in recs])).cuda()
    out = b.summary(buf, K, 1.0 / 3.0).cpu().numpy()
    assert (out[:4, 7] == 0.0).all()
    assert (out[:, [1, 3, 5, 7]] >= 0.0).all()
    for i, r in enumerate(recs):
        ref = ref_summary.summary(r[..., 0], r[..., 1], r[..., 2:4], dims, 1.0 / 3.0)
        np.testing.assert_allclose(out[i], ref, rtol=1e-9, atol=1e-9)
    b.close()
