"""GPU parity of the serial CPM at the edges of its rounds of drawn attempts:
lattices of less than one round, exactly one, a few attempts more, and several,
with every attempt hot (random labels, high temperature) so that most rounds
hold commits that later attempts of the round must see."""
import numpy as np
import pytest

import oracle
from paper_2312_09317_amd import cpm, inputs
from tests.test_gpu_chemotaxis import _batch, _batch_check
from tests.test_gpu_parity import _multi, oracle_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndim,dims,act,labels", [
    (2, (8, 8, 1), False, 3), (2, (8, 8, 1), True, 2), (2, (32, 32, 1), False, 4), (2, (32, 32, 1), True, 5),
    (2, (44, 24, 1), True, 9), (3, (12, 8, 8), True, 6), (3, (16, 16, 12), False, 30),
])
def test_serial_rounds(ndim, dims, act, labels):
    import torch
    ws = []
    for i in range(3):
        w = _multi(dims, ndim, seed=40 + i, act=act, obstacles=0.02, T=40.0)
        n = min(labels, w.n_cells + 1)
        w.lattice = inputs.random_labels(dims, n, 90 + i, p_obstacle=0.02)
        if act:
            w.act = np.random.default_rng(i).integers(0, 6, w.lattice.shape).astype(np.uint8)
        w.lattice_id = 3 * i
        ws.append(w)
    states = [oracle.State(oracle_model(w), w.lattice, w.cell_type, w.act) for w in ws]
    b = _batch(ws)
    for step, n in (("serial", 3), ("dcs", 1), ("serial", 1)):
        print(f"serial rounds: dims={dims} act={act} {step} {n}", flush=True)
        for st in states:
            st.serial_sweep(n) if step == "serial" else st.sweep(n)
        b.sweep_serial(n) if step == "serial" else b.sweep(n)
    torch.cuda.synchronize()
    _batch_check(torch, ws, b, states)
    assert all(b.check_invariants())
    b.close()
