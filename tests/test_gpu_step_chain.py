"""A call of several steps equals the same steps in calls of one, bit for bit: on small meshes the last
stage of a step forms the next step's CFL rate, in a run of one-step calls the reduction kernel does.

Both take the same maximum of the same values, so no tolerance.  Planes of one cell tile, of several
with ragged edges, and the largest that the chained form takes (16 tiles); driving, the exact Riemann
solver and the closure's correction beside it; and the rate slots as they are left for the next call.
"""
import numpy as np
import pytest

from paper_1602_09079_amd import synth
from tests.test_gpu_closure import SHAPE, dgm  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _solver(dg, k, n, prec, kind):
    s = dg.Solver(k, n, precision=prec, forcing=kind == "driven", riemann="exact" if kind == "exact" else "hllc",
                  closure=kind == "closure")
    if kind == "driven":
        rng = np.random.default_rng(4)
        s.set_forcing(np.array([[1, 0, 0], [0, 1, 1], [2, 0, 1]]), 0.05 * rng.standard_normal((3, 3, 2)))
    if kind == "closure":
        s.set_closure(synth.xavier_params(SHAPE, seed=3), np.zeros(140), np.ones(140), np.full(20, 1e-3), np.full(20, 1e30))
    return s


def _state(s, k, n, seed):
    rng = np.random.default_rng(seed)
    N = (k + 1) * (k + 2) * (k + 3) // 6
    y = 0.02 * rng.standard_normal((n[2], n[1], 5, N, n[0]))
    y[:, :, 0, 0] += 1.0
    y[:, :, 4, 0] += 1.5
    return torch.from_numpy(y).to(device="cuda", dtype=s.dtype).reshape(s.state_shape())


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("k,n,kind", [(1, (5, 3, 3), "plain"), (1, (16, 16, 16), "closure"), (1, (33, 21, 4), "driven"),
                                      (2, (17, 9, 5), "driven"), (2, (32, 32, 3), "exact")])
def test_steps_in_one_call_and_in_several(dgm, k, n, kind, prec):  # noqa: F811
    s, t = _solver(dgm, k, n, prec, kind), _solver(dgm, k, n, prec, kind)
    y, z = _state(s, k, n, 1), _state(t, k, n, 1)
    for calls in (5, 2, 3):  # odd and even: each slot is the one that a call leaves behind
        s.step(y, calls)
        for _ in range(calls):
            t.step(z, 1)
        torch.testing.assert_close(y, z, rtol=0, atol=0)
        assert torch.isfinite(y).all()
        assert s.dt(y) == t.dt(z)
