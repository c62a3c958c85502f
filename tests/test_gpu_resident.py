"""Sweeps of lattices kept in LDS (the library's own choice of tiling) against
the same sweeps by one launch per activation (an explicit layout), bit for
bit, where the resident kernel can go wrong: rows that are not whole vectors,
s from 1 up, several attempts per activation, lists and queues that overflow,
lattices cut into parts (with every term that reads across a cut), and calls
of both kinds in turn."""
import numpy as np
import pytest

from paper_2312_09317_amd import cpm, inputs

pytestmark = pytest.mark.gpu

J3 = np.array([[0, 3, 5, 1.5], [3, 7, 1.25, -2], [5, 1.25, 9, 0.5], [1.5, -2, 0.5, 0]])


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    cpm.load()
    return torch


def _params(dims, types=1, T=8.0, **kw):
    """One cell type, or two and obstacles."""
    if types == 1:
        base = dict(J=np.array([[0.0, 6.0], [6.0, 9.0]]), lambda_volume=[0, 2.0], volume_target=[0, 40],
                    lambda_surface=[0, 0.25], surface_target=[0, 90])
    else:
        base = dict(J=J3, lambda_volume=[0, 2.5, 1.0, 0], volume_target=[0, 30, 40, 0], lambda_surface=[0, 0.5, 0.25, 0],
                    surface_target=[0, 90, 120, 0], obstacle_type=3)
    base.update(kw)
    return cpm.Params(ndim=len(dims), dims=dims, temperature=T, seed=11, **base)


def _lattice(kind, dims, n, seed, obstacles):
    shape = tuple(dims) + (1,) * (3 - len(dims))
    p = 0.03 if obstacles else 0.0
    if kind == "noise":
        return inputs.random_labels(shape, n, seed, p_obstacle=p), n
    return inputs.random_blobs(shape, n, seed=seed, fill=0.4, p_obstacle=p), n


def _same(torch, p, lattice, types, explicit, n_mcs):
    """The library's choice against `explicit`, in two calls."""
    out = []
    for q in (p, p.replace(layout=explicit)):
        sim = cpm.Simulation(q, lattice, types)
        sim.sweep(1)
        sim.sweep(n_mcs - 1)
        torch.cuda.synchronize()
        assert sim.check_invariants()
        out.append([sim.lattice.cpu().numpy(), sim.act.cpu().numpy() if sim.act is not None else np.zeros(1)] +
                   [c.cpu().numpy()[1:] for c in sim.counters()] + [np.array([int(x) for x in sim.attempt_stats()])])
        sim.close()
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


SINGLE = [
    # dims, lattice, cells, types, s, k, T, act
    ((24, 24), "blobs", 5, 1, 2, 1, 8.0, False),
    ((30, 42), "blobs", 9, 2, 3, 1, 8.0, False),      # rows of 30 words: no whole vectors
    ((34, 18), "noise", 300, 1, 1, 1, 30.0, False),   # s = 1, rows of 34
    ((200, 200), "noise", 3000, 1, 2, 1, 40.0, False),  # every attempt nontrivial: queue and lists overflow
    ((96, 64), "noise", 500, 2, 4, 8, 40.0, False),   # several attempts per area, many accepted
    ((64, 64), "blobs", 40, 1, 2, 4, 8.0, True),
    ((44, 40), "blobs", 20, 2, 2, 1, 8.0, True),
    ((208, 16), "blobs", 12, 1, 2, 2, 8.0, False),
    ((180, 180), "noise", 2000, 1, 2, 1, 30.0, True),  # 32-bit words
    ((16, 24, 20), "blobs", 12, 2, 2, 1, 8.0, False),
    ((40, 40, 40), "noise", 600, 1, 2, 1, 30.0, False),
    ((16, 16, 24), "blobs", 9, 2, 2, 1, 8.0, True),
    ((12, 6, 18), "blobs", 5, 1, 3, 1, 8.0, False),
]


@pytest.mark.parametrize("case", range(len(SINGLE)))
def test_single_lattice(torch_cuda, case):
    dims, kind, n, types, s, k, T, act = SINGLE[case]
    print(f"resident case {SINGLE[case]}", flush=True)
    lat, n = _lattice(kind, dims, n, 20 + case, types == 2)
    kw = dict(sub=s, attempts=k)
    if act:
        kw.update(lambda_act=[0, 60.0] + ([0.0, 0.0] if types == 2 else []), max_act=[0, 20] + ([0, 0] if types == 2 else []))
    ct = np.array([0] + [1 + (i % types) for i in range(n)], dtype=np.int32)
    _same(torch_cuda, _params(dims, types, T, **kw), lat, ct, "in_place" if k == 1 else "box", 5)


@pytest.mark.parametrize("incremental", [False, True])
def test_persistence(torch_cuda, incremental):
    dims = (24, 20, 28)
    lat, n = _lattice("blobs", dims, 10, 3, False)
    p = _params(dims, lambda_persistence=[0, 40.0], persistence_mu=[0, 0.9], persistence_dt=2,
                persistence_centroids="incremental" if incremental else "recount")
    print(f"resident persistence incremental={incremental}", flush=True)
    _same(torch_cuda, p, lat, np.array([0] + [1] * n, dtype=np.int32), "in_place", 6)


def _batches_same(torch, params, lats, types, explicit, n_mcs, mode_between=None):
    out = []
    for lay in ("auto", explicit):
        b = cpm.Batch([q.replace(layout=lay) for q in params], lats, types)
        b.sweep(2)
        if mode_between and lay == "auto":
            b.launch_mode(mode_between)  # a launch per activation, then resident again
            b.sweep(1)
            b.launch_mode("graph")
        else:
            b.sweep(1)
        b.sweep(n_mcs - 3)
        torch.cuda.synchronize()
        assert all(b.check_invariants())
        out.append([b.lattices.cpu().numpy(), b.act.cpu().numpy() if b.act is not None else np.zeros(1)] +
                   [c.cpu().numpy() for c in b.counters()] + [np.asarray(b.attempt_stats()).astype(np.int64)])
    labels = np.cumsum([0] + [len(t) for t in types])[:-1]
    for v in out:
        for c in v[2:4]:
            c[labels] = 0
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


BATCH = [
    # lattices (dims), kind, cells, types, s, k, act, chemotaxis
    ([(640, 512), (288, 300), (64, 48)] * 2, "blobs", 700, 1, 2, 1, True, False),   # cut into parts, and not; 16-bit words
    ([(640, 600), (512, 528)] * 2, "noise", 900, 1, 2, 1, False, False),
    ([(640, 600), (480, 528)] * 3, "noise", 900, 2, 2, 1, True, False),             # 32-bit words
    ([(576, 576)] * 5, "blobs", 500, 1, 4, 8, False, True),
    ([(1024, 800), (900, 1000)], "noise", 400, 1, 1, 1, False, True),
    ([(64, 72, 80)] * 6, "blobs", 300, 2, 2, 1, False, False),                      # cut across y and z
    ([(64, 64, 68), (64, 60, 64)] * 4, "blobs", 300, 2, 2, 1, True, False),
]


@pytest.mark.parametrize("case", range(len(BATCH)))
def test_batch_with_cut_lattices(torch_cuda, case):
    dims, kind, n, types, s, k, act, chem = BATCH[case]
    print(f"resident batch case {BATCH[case]}", flush=True)
    params, lats, cts = [], [], []
    for i, d in enumerate(dims):
        lat, m = _lattice(kind, d, n, 50 + i, types == 2)
        kw = dict(sub=s, attempts=k, lattice_id=i)
        if act:
            kw.update(lambda_act=[0, 60.0] + ([0.0, 0.0] if types == 2 else []), max_act=[0, 20] + ([0, 0] if types == 2 else []))
        if chem:
            rng = np.random.default_rng(i)
            kw.update(lambda_chemotaxis=[0, 9.0], chemotaxis_field=torch_cuda.as_tensor(
                rng.integers(-16000, 16000, int(np.prod(d)) * len(d)).astype(np.int16)).cuda())
        params.append(_params(d, types, 8.0 + i, **kw))
        lats.append(lat)
        cts.append(np.array([0] + [1 + (j % types) for j in range(m)], dtype=np.int32))
    _batches_same(torch_cuda, params, lats, cts, "in_place" if k == 1 else "box", 5, mode_between="eager" if case % 2 == 0 else None)


@pytest.mark.parametrize("s,k", [(1, 1), (2, 1), (2, 4), (4, 2)])
def test_hot_lists_grow_while_drawn_ahead(torch_cuda, s, k):
    # many small lattices of a few fast cells: areas turn hot in every step,
    # while the other half of the workgroup draws the next one's attempts from
    # the same lists
    print(f"growing hot lists s={s} k={k}", flush=True)
    params, lats, cts = [], [], []
    for i in range(192):
        d = (64 + 16 * (i % 3), 48 + 16 * (i % 2))
        lat, m = _lattice("blobs", d, 4, 400 + i, False)
        params.append(_params(d, 1, 25.0 + i % 7, sub=s, attempts=k, lattice_id=i))
        lats.append(lat)
        cts.append(np.array([0] + [1] * m, dtype=np.int32))
    _batches_same(torch_cuda, params, lats, cts, "in_place" if k == 1 else "box", 14)


# batches that the default keeps in LDS in parts
CUT = [
    ([(640, 512), (288, 300), (64, 48)] * 2, "blobs", 700, 1, 2, 1, True, False),  # 16-bit label-activity words
    ([(512, 512), (480, 528)] * 2, "blobs", 700, 2, 2, 4, True, False),            # 32-bit words, several types
    ([(512, 512)] * 2, "blobs", 700, 1, 2, 2, True, True),                         # 32-bit words, one type
    ([(576, 576)] * 18, "blobs", 500, 1, 4, 8, False, True),
    ([(512, 528), (640, 600)] * 10, "noise", 900, 2, 2, 1, False, False),
    ([(640, 700)] * 3, "noise", 400, 1, 1, 1, False, True),
]


def _cut_batch(torch, case):
    """Parameters, lattices and types of CUT[case]."""
    return _batch_of(torch, CUT[case])


def _batch_of(torch, spec):
    dims, kind, n, types, s, k, act, chem = spec
    params, lats, cts, made = [], [], [], {}
    for i, d in enumerate(dims):
        if d not in made:  # lattices of one shape start alike
            made[d] = _lattice(kind, d, n, 80 + i, types == 2)
        lat, m = made[d]
        kw = dict(sub=s, attempts=k, lattice_id=i)
        if act:
            kw.update(lambda_act=[0, 60.0] + ([0.0, 0.0] if types == 2 else []), max_act=[0, 20] + ([0, 0] if types == 2 else []))
        if chem:
            kw.update(lambda_chemotaxis=[0, 9.0], chemotaxis_field=torch.as_tensor(
                np.random.default_rng(i).integers(-16000, 16000, int(np.prod(d)) * len(d)).astype(np.int16)).cuda())
        params.append(_params(d, types, 8.0 + i % 6, **kw))
        lats.append(lat)
        cts.append(np.array([0] + [1 + (j % types) for j in range(m)], dtype=np.int32))
    return params, lats, cts


def _assert_same(a, b):
    assert a.torch.equal(a.lattices, b.lattices)
    assert a.act is None or a.torch.equal(a.act, b.act)
    for x, y in zip(a.counters(), b.counters()):
        for lo, hi in zip(a.label_off[:-1], a.label_off[1:]):
            assert a.torch.equal(x[lo + 1:hi], y[lo + 1:hi])
    np.testing.assert_array_equal(a.attempt_stats(), b.attempt_stats())


@pytest.mark.parametrize("case", range(len(CUT)))
def test_parts_that_do_not_come_together(torch_cuda, case):
    # no poll allowed: every lattice cut into parts is marked as not together,
    # and one workgroup sweeps the lattice; then the parts meet again
    params, lats, cts = _cut_batch(torch_cuda, case)
    print(f"parts apart, case {case}", flush=True)
    b, ref = cpm.Batch(params, lats, cts), cpm.Batch(params, lats, cts)
    ref.use_graph(False)
    cpm.cpm_batch_set_barrier_spin_limit(b.handle, 0)
    b.sweep(2)
    ref.sweep(2)
    _assert_same(b, ref)
    apart = cpm.cpm_batch_alone_count(b.handle, b.stream)
    assert apart > 0
    cpm.cpm_batch_set_barrier_spin_limit(b.handle, 1 << 21)
    b.sweep(2)
    ref.sweep(2)
    _assert_same(b, ref)
    assert cpm.cpm_batch_alone_count(b.handle, b.stream) == apart
    assert all(b.check_invariants())


@pytest.mark.parametrize("case", [0, 3])
def test_captured_sweeps_replay(torch_cuda, case):
    # a captured sweep of lattices cut into parts, replayed with eager work
    # and a synchronisation in between
    torch = torch_cuda
    params, lats, cts = _cut_batch(torch, case)
    print(f"captured resident sweeps, case {case}", flush=True)
    b, ref = cpm.Batch(params, lats, cts), cpm.Batch(params, lats, cts)
    ref.use_graph(False)
    b.sweep(1)
    ref.sweep(1)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b.sweep(2)
    for _ in range(3):
        g.replay()
        ref.mcs = 1
        ref.sweep(2)
        torch.cuda.synchronize()
        assert torch.equal(b.lattices, ref.lattices)
        assert b.act is None or torch.equal(b.act, ref.act)
        b.mcs = ref.mcs = 7
        b.sweep(1)
        ref.sweep(1)
        for x, y in zip(b.cell_stats(), ref.cell_stats()):
            assert torch.equal(x, y)
    assert all(b.check_invariants())


def test_graph_mode_replays_the_graph(torch_cuda):
    # a batch that the default keeps in LDS: "graph" replays the MCS graph
    # (no lattice is in parts, so none is swept alone), with read-outs and
    # serial MCS between replays, and the modes may follow each other
    params, lats, cts = _cut_batch(torch_cuda, 0)
    b, ref = cpm.Batch(params, lats, cts), cpm.Batch(params, lats, cts)
    ref.launch_mode("eager")
    cpm.cpm_batch_set_barrier_spin_limit(b.handle, 0)
    for step, mode in enumerate(("graph", "graph", "auto", "eager", "auto", "graph", "auto")):
        print(f"step {step}: {mode}", flush=True)
        b.launch_mode(mode)
        before = cpm.cpm_batch_alone_count(b.handle, b.stream)
        for x in (b, ref):
            x.sweep(1 + step % 2)
        assert (cpm.cpm_batch_alone_count(b.handle, b.stream) > before) == (mode == "auto")
        for u, v in zip(b.cell_stats(), ref.cell_stats()):
            assert torch_cuda.equal(u, v)
        _assert_same(b, ref)
        if step in (1, 4):
            b.sweep_serial(1)
            ref.sweep_serial(1)
    assert all(b.check_invariants())
    with pytest.raises(cpm.CpmError) as e:
        b.launch_mode(4)
    assert e.value.code == cpm.CPM_EINVAL


@pytest.mark.parametrize("case", range(1, len(CUT)))
def test_default_mode_after_others(torch_cuda, case):
    # resident, by launches, and resident again
    params, lats, cts = _cut_batch(torch_cuda, case)
    b, ref = cpm.Batch(params, lats, cts), cpm.Batch(params, lats, cts)
    ref.launch_mode("eager")
    for mode in ("auto", "graph", "auto", "eager", "auto"):
        b.launch_mode(mode)
        b.sweep(2)
        ref.sweep(2)
        _assert_same(b, ref)
    assert all(b.check_invariants())


@pytest.mark.parametrize("s,k", [(2, 1), (4, 8)])
def test_batch_tuner_times_the_default(torch_cuda, s, k):
    ws = inputs.config3(n_lattices=6, L_min=64, L_max=128, seed=5, n_mcs=0)
    for w in ws:
        side = w.dims[0] // (2 * s) * (2 * s)
        w.lattice = w.lattice.reshape(w.dims[1], w.dims[0])[:side, :side].copy().reshape(-1)
        w.dims = (side, side, 1)
    params = [cpm.Params.from_workload(w, sub=s, attempts=k) for w in ws]
    r = cpm.autotune_batch(params, [w.lattice for w in ws], [w.cell_type for w in ws], trial_mcs=2)
    print(r["times"], flush=True)
    assert next(iter(r["times"])) == "auto" and len(r["times"]) >= 2
    b = cpm.Batch(cpm.batch_params(params, r["best"]), [w.lattice for w in ws], [w.cell_type for w in ws])
    b.launch_mode(r["best"]["mode"])
    b.sweep(1)
    assert all(b.check_invariants())


@pytest.mark.parametrize("spec", [
    ([(64, 72, 80)] * 2, "blobs", 300, 2, 2, 1, False, False),   # 3D lattices in parts
    ([(512, 512)] * 2, "blobs", 700, 2, 2, 1, True, False),      # 32-bit words, one attempt
    ([(576, 576)] * 2, "blobs", 500, 1, 4, 8, False, True),      # too few parts for the CUs
    ([(512, 528)] * 2, "noise", 900, 1, 2, 1, False, False),
])
def test_batches_swept_faster_by_launches(torch_cuda, spec):
    # these leave the LDS path to the graph: no lattice of theirs is in parts
    params, lats, cts = _batch_of(torch_cuda, spec)
    b, ref = cpm.Batch(params, lats, cts), cpm.Batch(params, lats, cts)
    ref.launch_mode("eager")
    cpm.cpm_batch_set_barrier_spin_limit(b.handle, 0)
    b.sweep(2)
    ref.sweep(2)
    _assert_same(b, ref)
    assert cpm.cpm_batch_alone_count(b.handle, b.stream) == 0


def test_many_attempts_per_area_uncut(torch_cuda):
    # eight attempts per area, nearly all of them evaluated and many accepted
    spec = ([(96, 64)] * 100, "noise", 500, 2, 4, 8, False, False)
    params, lats, cts = _batch_of(torch_cuda, spec)
    params = [p.replace(temperature=40.0) for p in params]
    _batches_same(torch_cuda, params, lats, cts, "box", 4)


def test_lattices_of_two_sizes_swept_by_two_threads(torch_cuda):
    # one kernel launched with different amounts of LDS from two threads, each
    # on a stream of its own
    import threading
    torch = torch_cuda
    dims = ((176, 176), (208, 208))
    sims, streams, want, errors = [], [], [], []
    for d in dims:
        lat, n = _lattice("blobs", d, 30, 90, False)
        ct = np.array([0] + [1] * n, dtype=np.int32)
        ref = cpm.Simulation(_params(d).replace(layout="in_place"), lat, ct)
        ref.sweep(40)
        want.append(ref.lattice.clone())
        sims.append(cpm.Simulation(_params(d), lat, ct))
        streams.append(torch.cuda.Stream())
    torch.cuda.synchronize()

    def run(i):
        try:
            with torch.cuda.stream(streams[i]):
                for _ in range(40):
                    sims[i].sweep(1)
        except Exception as e:  # reported by the test
            errors.append(e)

    threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors
    for s, w in zip(sims, want):
        assert torch.equal(s.lattice, w)
