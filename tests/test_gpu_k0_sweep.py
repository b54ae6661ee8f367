"""The k = 0 sweep and the CFL reduction at the edges of their work items: z chunks of several planes
with a ragged last one, ragged tiles, a slab with halo planes, planes of 2 GiB and more; rows shorter
than, equal to and longer than a workgroup.  Against the FP64 oracle: R in FP64 to 1e-12 of the largest
field norm; dt to 1e-13 on the stored state.  In FP32 the slab, whose chunks start at other planes, is
compared with the whole mesh."""
import numpy as np
import pytest

import oracle as O
from tests.layout import from_abi, to_abi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

G = 5.0 / 3.0


@pytest.fixture(scope="module")
def dgm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1602_09079_amd import dg
    dg.lib()
    return dg


def state(k, n, dtype, seed=5):
    rng = np.random.default_rng(seed)
    N = (k + 1) * (k + 2) * (k + 3) // 6
    y = 0.01 * rng.standard_normal((5, N, n[2], n[1], n[0]))
    y[:, 0] += np.array([1.0, 0.2, -0.3, 0.1, 2.5])[:, None, None, None]
    return torch.from_numpy(to_abi(y)).to("cuda", dtype)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [(130, 62, 101), (256, 64, 129)])
def test_chunks_of_several_planes(dgm, prec, n):
    s = dgm.Solver(0, n, gamma=G, precision=prec)
    y = state(0, n, s.dtype)
    r = s.rhs(y)
    if prec == "fp64":
        want = O.rhs(O.make_cfg(0, n, gamma=G), from_abi(y.cpu().numpy())).reshape(5, -1)
        d = from_abi(r.cpu().numpy()).reshape(5, -1) - want
        err = np.linalg.norm(d, axis=1) / np.linalg.norm(want, axis=1).max()
        assert np.all(err <= 1e-12), err
    # a slab of it, its other neighbours in halo planes: the same to rounding (its box over its planes is
    # not exactly the whole mesh's cell height)
    part = dgm.Solver(0, (n[0], n[1], 40), box=(1.0, 1.0, 40 / n[2]), gamma=G, precision=prec, zhalo=True)
    part.set_halo(y[6].clone(), y[47].clone())
    got, ref = part.rhs(y[7:47].clone()), r[7:47]
    assert (got - ref).abs().max() <= {"fp64": 1e-13, "fp32": 1e-5}[prec] * ref.abs().max()


def test_planes_past_two_gib(dgm):
    n, rep = (64, 48, 2), (150, 240)
    s = dgm.Solver(0, n, gamma=G, precision="fp32")
    y = state(0, n, s.dtype)
    want = s.rhs(y)
    big = dgm.Solver(0, (n[0] * rep[0], n[1] * rep[1], 2), box=(150.0, 240.0, 1.0), gamma=G, precision="fp32")
    assert 20 * n[0] * n[1] * rep[0] * rep[1] >= 2 ** 31
    got = big.rhs(y.repeat(1, rep[1], 1, 1, rep[0]))
    for j in (0, 239):
        for i in (0, 149):
            part = got[:, j * n[1]:(j + 1) * n[1], :, :, i * n[0]:(i + 1) * n[0]]
            assert (part - want).abs().max() <= 1e-5 * want.abs().max(), (i, j)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("k,n", [(0, (3, 5, 2)), (1, (341, 7, 2)), (0, (512, 3, 2)), (0, (1024, 2, 2)), (0, (1025, 3, 2)),
                                 (2, (64, 30, 9)), (0, (100, 300, 40))])
def test_dt_over_rows(dgm, prec, k, n):
    s = dgm.Solver(k, n, box=(1.0, 0.7, 1.3), gamma=G, precision=prec)
    y = state(k, n, s.dtype)
    cfg = O.make_cfg(k, n, box=(1.0, 0.7, 1.3), gamma=G)
    for cell in ((0, 0, 0), (n[2] - 1, n[1] - 1, n[0] - 1), (n[2] // 2, n[1] // 2, n[0] // 2)):
        z = y.clone()
        z[cell[0], cell[1], 1, 0, cell[2]] += 3.0  # the fastest cell
        z[cell[0], cell[1], 4, 0, cell[2]] += 9.0
        want = O.dt(cfg, from_abi(z.cpu().double().numpy()))
        assert abs(s.dt(z) - want) <= 1e-13 * want, cell
