"""GPU checks of the emulator's row kernel and gradient split at the sizes
where their work split changes: a single row, rows per workgroup, one split of
the batch and several, and the changes of kernel variant."""
import numpy as np
import pytest

from paper_2312_09317_amd import emu, inputs

pytestmark = pytest.mark.gpu


def _setup(n, seed=0):
    rng = np.random.default_rng(seed + n)
    W, b = inputs.mlp_weights(3)
    b = [0.1 * rng.standard_normal(v.shape) for v in b]
    x = rng.standard_normal((n, 6)).astype(np.float32)
    t = rng.standard_normal((n, 8)).astype(np.float32)
    return W, b, x, t


def _exact_grads(W, b, x, t):
    import torch
    p = [torch.tensor(v, dtype=torch.float64, requires_grad=True) for pair in zip(W, b) for v in pair]
    a = torch.as_tensor(x, dtype=torch.float64)
    for i in range(4):
        a = a @ p[2 * i].T + p[2 * i + 1]
        if i < 3:
            a = torch.nn.functional.gelu(a)
    loss = ((a - torch.as_tensor(t, dtype=torch.float64)) ** 2).mean()
    g = torch.autograd.grad(loss, p)
    return a.detach().numpy(), loss.item(), np.concatenate([v.numpy().reshape(-1) for v in g])


# bf16 operands (unit roundoff 2^-9): two rounded operands per product over
# four layers forward, one more per layer backward
@pytest.mark.parametrize("n", [1, 3, 4, 5, 15, 17, 64, 65, 1023, 1024, 1025, 2049, 8192, 8193, 8257])
def test_rows_and_gradients(n):
    import torch
    W, b, x, t = _setup(n)
    y_ref, loss_ref, g_ref = _exact_grads(W, b, x, t)
    net = emu.Emulator(max(n, 64))
    net.set_params(emu.pack(W, b))
    y = net.forward(x).cpu().numpy()
    g, loss = net.grads(x, t)
    torch.cuda.synchronize()
    g = g.cpu().numpy()
    assert np.linalg.norm(y - y_ref) <= 8 * 2.0 ** -9 * np.linalg.norm(y_ref)
    assert np.linalg.norm(g - g_ref) <= 16 * 2.0 ** -9 * np.linalg.norm(g_ref)
    assert abs(float(loss) - loss_ref) <= 16 * 2.0 ** -9 * loss_ref
    # a step is those gradients, then Adam
    ref = emu.Emulator(max(n, 64))
    ref.set_params(emu.pack(W, b))
    ref.adam(1e-3, g)
    step_loss = net.train_step(torch.as_tensor(x).cuda(), torch.as_tensor(t).cuda(), 1e-3)
    assert torch.equal(net.params(), ref.params())
    assert float(step_loss) == float(loss)
    y2, y3 = net.forward(x), ref.forward(x)
    assert torch.equal(y2, y3)  # the operand copies follow the parameters
    net.close(), ref.close()
