"""Infinite parameters of the dense network: a saturated unit is +-1 and an output its infinity, whatever
lies beside them.  Layer widths that end inside a group of 16 (140, 100, 72, 20: the products' padding),
in the reads of four weights and of one (37, 29, 5), against plain torch in 64 bits."""
import pytest

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


def _split(p, shape):
    out, at = [], 0
    for i, o in zip(shape[:-1], shape[1:]):
        out.append((p[at:at + i * o].view(o, i), p[at + i * o:at + i * o + o]))
        at += i * o + o
    return out


@pytest.mark.parametrize("shape", [(140, 128, 128, 20), (140, 100, 72, 20), (37, 29, 17, 5)])
def test_forward_with_infinite_weights(dgm, shape):
    batch = 33
    p = torch.from_numpy(synth.xavier_params(shape, seed=2)).float().cuda()
    (w1, _), (w2, _), (w3, _) = _split(p, shape)
    w1[3, -1] = float("inf")    # the last input, the last hidden unit: where the padding begins
    w1[5, 0] = -float("inf")
    w2[2, -1] = float("inf")
    w3[1, -1] = -float("inf")
    g = torch.Generator(device="cuda").manual_seed(1)
    x = 0.5 + torch.rand(batch, shape[0], generator=g, device="cuda")
    h = x.double()
    for j, (w, b) in enumerate(_split(p.double(), shape)):
        h = (h[:, None, :] * w).sum(2) + b  # (a sum of products: no library product between it and infinity)
        h = torch.tanh(h) if j < 2 else h
    y = dgm.MLP(shape, batch).forward(p, x).double()
    inf = torch.isinf(h)
    assert inf.any() and not torch.isnan(h).any()
    assert torch.equal(y[inf], h[inf])
    assert (y[~inf] - h[~inf]).abs().max() <= 1e-5 * h[~inf].abs().max()


@pytest.mark.parametrize("shape", [(140, 128, 128, 20), (37, 29, 17, 5)])
def test_gradient_with_a_saturated_unit(dgm, shape):
    """A first-layer unit held at +1 by an infinite weight: its own gradient rows are zero, the rest of the
    gradient is finite."""
    batch = 40
    p = torch.from_numpy(synth.xavier_params(shape, seed=2)).float().cuda()
    _split(p, shape)[0][0][3, -1] = float("inf")
    g = torch.Generator(device="cuda").manual_seed(1)
    x = 0.5 + torch.rand(batch, shape[0], generator=g, device="cuda")
    t = torch.randn(batch, shape[3], generator=g, device="cuda")
    q = p.double()
    leaves = [(w.clone().requires_grad_(True), b.clone().requires_grad_(True)) for w, b in _split(q, shape)]
    h = x.double()
    for j, (w, b) in enumerate(leaves):
        h = (h[:, None, :] * w).sum(2) + b
        h = torch.tanh(h) if j < 2 else h
    ((h - t) ** 2).mean().backward()
    grad, loss = dgm.MLP(shape, batch).loss_grad(p, x, t)
    assert torch.isfinite(loss)
    for (gw, gb), (w, b) in zip(_split(grad.double(), shape), leaves):
        for got, want in ((gw, w.grad), (gb, b.grad)):
            assert torch.isfinite(want).all()
            assert (got - want).norm() <= 1e-4 * want.norm()
