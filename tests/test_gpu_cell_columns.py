"""Columns of cells (one x-block of 14, two rows) at k = 2 in FP64, on both sides of the length where they go
to the matrix kernel (256 planes), and the columns beside them that do not (a third row, a 15th cell):
R and a stage against the FP64 oracle, ||R_gpu,i - R_orc,i|| / max_j ||R_orc,j|| <= 1e-12; driving, the exact
solver; slabs of the column against the whole, to rounding."""
import numpy as np
import pytest

import oracle as O
from paper_1602_09079_amd import synth
from tests.layout import from_abi
from tests.test_gpu_cell_stage import G, dgm, state  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,riemann", [((14, 2, 256), "hllc"), ((14, 2, 257), "hllc"), ((2, 2, 400), "exact"),
                                       ((15, 2, 257), "hllc"), ((14, 3, 257), "hllc"), ((9, 2, 1030), "hllc")])
def test_columns_against_the_oracle(dgm, n, riemann):  # noqa: F811
    s = dgm.Solver(2, n, box=(1.0, 0.5, 20.0), gamma=G, precision="fp64", forcing=True, riemann=riemann)
    nvec = synth.forcing_modes(1.0, 3.0)
    ah = 0.05 * synth.ou_stationary_start(7, len(nvec))
    s.set_forcing(nvec, ah)
    y = state(s, n)
    cfg = O.make_cfg(2, n, box=(1.0, 0.5, 20.0), gamma=G, riemann=riemann)
    want = O.rhs(cfg, from_abi(y.cpu().numpy()), O.ForcingTable(nvec, ah))
    r = s.rhs(y)
    d = (from_abi(r.cpu().numpy()) - want).reshape(5, -1)
    err = np.linalg.norm(d, axis=1) / np.linalg.norm(want.reshape(5, -1), axis=1).max()
    assert np.all(err <= 1e-12), err
    # a stage is its combination, and the z chunk length does not change a bit
    out, h = torch.empty_like(y), 1e-4
    s.stage(y, y, out, 0.75, 0.25, h)
    ref = 0.75 * y + 0.25 * (y - h * r)
    assert (out - ref).abs().max() <= 1e-14 * ref.abs().max()
    for zl in (1, 7, n[2]):
        s.set_zchunk(zl)
        assert torch.equal(s.rhs(y), r), zl


def test_slabs_of_a_column(dgm):  # noqa: F811
    n = (6, 2, 300)
    whole = dgm.Solver(2, n, box=(1.0, 1.0, 300.0), gamma=G, precision="fp64")
    y = state(whole, n)
    r = whole.rhs(y)
    for lo, hi in ((0, 20), (20, 300)):
        s = dgm.Solver(2, (6, 2, hi - lo), box=(1.0, 1.0, float(hi - lo)), gamma=G, precision="fp64", zhalo=True)
        s.set_slab(lo, 300)
        s.set_halo(y[lo - 1].clone(), y[hi % 300].clone())
        assert (s.rhs(y[lo:hi].clone()) - r[lo:hi]).abs().max() <= 1e-13 * r.abs().max()


def test_steps_of_a_column(dgm):  # noqa: F811
    """Several steps in a call equal one-step calls (the rate is formed by the reduction here)."""
    n = (4, 2, 300)
    s, t = (dgm.Solver(2, n, gamma=G, precision="fp64") for _ in range(2))
    y = state(s, n)
    z = y.clone()
    s.step(y, 3)
    for _ in range(3):
        t.step(z, 1)
    assert torch.isfinite(y).all() and torch.equal(y, z)
