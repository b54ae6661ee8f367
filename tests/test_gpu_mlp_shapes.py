"""The training kernels of the dense network where their forms meet: batches about the 16-sample tile
and the 256-sample range, layers that are no multiple of 4 or 16, parameters off the 16-byte
boundary, and a network too large for the fused form.  Tolerances as for the 140-128-128-20 network:
outputs 1e-5 of the largest, loss 1e-5, gradient blocks 1e-4 (relative L2), against the FP64 oracle."""
import numpy as np
import pytest

import oracle as O
from paper_1602_09079_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dgm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1602_09079_amd import dg
    dg.lib()
    return dg


@pytest.mark.parametrize("shape,batch,shift", [
    ((140, 128, 128, 20), 1, 0), ((140, 128, 128, 20), 15, 0), ((140, 128, 128, 20), 257, 1),
    ((140, 100, 72, 20), 48, 0), ((7, 5, 3, 2), 33, 0), ((16, 17, 65, 1), 513, 0), ((900, 500, 300, 40), 40, 0)])
def test_loss_grad_at_shape_edges(dgm, shape, batch, shift):
    rng = np.random.default_rng(1)
    p = synth.xavier_params(shape, seed=4)
    p = (p + 0.05 * rng.standard_normal(p.size)).astype(np.float32)
    x = rng.standard_normal((batch + 9, shape[0])).astype(np.float32)
    t = rng.standard_normal((batch + 9, shape[3])).astype(np.float32)
    rows = rng.permutation(batch + 9)[:batch].astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    pd = torch.cat([torch.zeros(shift, device="cuda"), dev(p)])[shift:]
    net = dgm.MLP(shape, batch + 20)  # a workspace for more than the batch
    y = net.forward(pd, dev(x), rows=dev(rows)).cpu().double().numpy()
    f = lambda a: a.astype(np.float64)
    want = O.mlp_forward(f(p), f(x[rows]), shape)[2]
    assert np.abs(y - want).max() <= 1e-5 * np.abs(want).max()
    g, loss = net.loss_grad(pd, dev(x), dev(t), rows=dev(rows))
    loss_ref, g_ref = O.mlp_loss_grad(f(p), f(x[rows]), f(t[rows]), shape)
    assert abs(loss.item() - loss_ref) <= 1e-5 * loss_ref
    nin, h1, h2, no = shape
    at = np.cumsum([h1 * nin, h1, h2 * h1, h2, no * h2])
    for gb, rb in zip(np.split(g.cpu().double().numpy(), at), np.split(g_ref, at)):
        assert np.linalg.norm(gb - rb) <= 1e-4 * np.linalg.norm(rb)
