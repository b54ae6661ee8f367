"""Loss gradients over batches past 8192 samples, where the weight gradients' 32 ranges grow beyond 256
samples and the last ones may be short or empty: 9001 (ranges of 288, the last of 80), 8193 (ranges of 272,
one of 48 and the last empty) and 16384 (32 ranges of 512), against the FP64 oracle.  Tolerances as for the smaller batches: loss 1e-5, gradient blocks 1e-4 (relative L2)."""
import numpy as np
import pytest

import oracle as O
from paper_1602_09079_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape,batch", [((140, 128, 128, 20), 9001), ((140, 128, 128, 20), 16384), ((37, 29, 17, 5), 8193)])
def test_loss_grad_of_large_batches(shape, batch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1602_09079_amd import dg
    rng = np.random.default_rng(1)
    p = synth.xavier_params(shape, seed=4)
    p = (p + 0.05 * rng.standard_normal(p.size)).astype(np.float32)
    x = rng.standard_normal((batch + 9, shape[0])).astype(np.float32)
    t = rng.standard_normal((batch + 9, shape[3])).astype(np.float32)
    rows = rng.permutation(batch + 9)[:batch].astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    g, loss = dg.MLP(shape, batch).loss_grad(dev(p), dev(x), dev(t), rows=dev(rows))
    f = lambda a: a.astype(np.float64)
    loss_ref, g_ref = O.mlp_loss_grad(f(p), f(x[rows]), f(t[rows]), shape)
    assert abs(loss.item() - loss_ref) <= 1e-5 * loss_ref
    nin, h1, h2, no = shape
    at = np.cumsum([h1 * nin, h1, h2 * h1, h2, no * h2])
    for gb, rb in zip(np.split(g.cpu().double().numpy(), at), np.split(g_ref, at)):
        assert np.linalg.norm(gb - rb) <= 1e-4 * np.linalg.norm(rb)
