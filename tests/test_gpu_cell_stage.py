"""The one-cell-per-lane stage kernel (k = 1, 2 in FP64 and FP32) on small and ragged meshes (its tiles
are 16 x 4 cells; these meshes take the form whose tiles are split over waves by task), against the FP64
oracle, and the properties its dispatch keeps: the z chunk length and a z slab do not change a bit, and
planes of 2 GiB and more (64-bit addresses) get the same result.

Tolerances on R as for the other stage kernels: ||R_gpu,i - R_orc,i|| / max_j ||R_orc,j|| <= 1e-12
(FP64), 2e-5 (FP32)."""
import numpy as np
import pytest

import oracle as O
from paper_1602_09079_amd import synth
from tests.layout import from_abi, to_abi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

G = 5.0 / 3.0
TOL = {"fp64": 1e-12, "fp32": 2e-5}


@pytest.fixture(scope="module")
def dgm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1602_09079_amd import dg
    dg.lib()
    return dg


def state(s, n, seed=3):
    """Random weights about a uniform flow, decaying with the mode's degree."""
    rng = np.random.default_rng(seed)
    y = np.zeros((5, s.N, n[2], n[1], n[0]))
    for l in range(s.N):
        amp = 0.05 if l == 0 else 0.03 if l < 4 else 0.01
        y[:, l] = amp * rng.standard_normal(y[:, l].shape)
    y[:, 0] += np.array([1.0, 0.2, -0.3, 0.1, 2.5])[:, None, None, None]
    return torch.from_numpy(to_abi(y)).to("cuda", s.dtype)


# fewer cells than a tile along x; exact tiles and ragged ones; axes of 2 cells
@pytest.mark.parametrize("n", [(8, 8, 2), (9, 7, 3), (32, 32, 2), (40, 32, 3), (33, 33, 2), (2, 130, 2), (131, 2, 3)])
@pytest.mark.parametrize("k", [1, 2])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_rhs_at_tile_edges(dgm, prec, k, n):
    box, force, riemann = (1.0, 0.9, 1.1), n[2] == 3, "exact" if n[0] == 33 else "hllc"
    s = dgm.Solver(k, n, box=box, gamma=G, precision=prec, forcing=force, riemann=riemann)
    frc = None
    if force:
        nvec = synth.forcing_modes(1.0, 3.0)
        ah = 0.05 * synth.ou_stationary_start(7, len(nvec))
        s.set_forcing(nvec, ah)
        frc = O.ForcingTable(nvec, ah)
    y = state(s, n)
    r = s.rhs(y)
    want = O.rhs(O.make_cfg(k, n, box=box, gamma=G, riemann=riemann), from_abi(y.cpu().double().numpy()), frc)
    d = (from_abi(r.cpu().double().numpy()) - want).reshape(5, -1)
    err = np.linalg.norm(d, axis=1) / np.linalg.norm(want.reshape(5, -1), axis=1).max()
    print(f"k={k} {prec} {n}: {err}")
    assert np.all(err <= TOL[prec]), err


@pytest.mark.parametrize("n", [(41, 33, 6), (16, 24, 6)])
@pytest.mark.parametrize("k", [1, 2])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_chunks_and_slabs_do_not_change_a_bit(dgm, prec, k, n):
    s = dgm.Solver(k, n, gamma=G, precision=prec)
    y = state(s, n)
    whole = s.rhs(y)
    for zl in (6, 4, 1):
        s.set_zchunk(zl)
        assert torch.equal(s.rhs(y), whole), zl
    for lo, hi in ((0, 2), (2, 6)):
        part = dgm.Solver(k, (n[0], n[1], hi - lo), box=(1.0, 1.0, (hi - lo) / n[2]), gamma=G, precision=prec, zhalo=True)
        part.set_halo(y[lo - 1].clone(), y[hi % n[2]].clone())
        assert torch.equal(part.rhs(y[lo:hi].clone()), whole[lo:hi]), (lo, hi)


def test_planes_past_two_gib(dgm):
    """A mesh whose z plane takes 2.3 GB is a small periodic mesh repeated: the same result, repeated."""
    k, n, rep = 2, (48, 40, 2), (60, 50)
    s = dgm.Solver(k, n, gamma=G, precision="fp64")
    y = state(s, n)
    want = s.rhs(y)
    big = dgm.Solver(k, (n[0] * rep[0], n[1] * rep[1], n[2]), box=(60.0, 50.0, 1.0), gamma=G, precision="fp64")
    assert 8 * big.N * 5 * n[0] * n[1] * rep[0] * rep[1] >= 2 ** 31
    yb = y.repeat(1, rep[1], 1, 1, rep[0])
    got = big.rhs(yb)
    del yb
    # the cell widths of the two meshes agree to rounding only
    for j in (0, 17, 49):
        for i in (0, 23, 59):
            part = got[:, j * n[1]:(j + 1) * n[1], :, :, i * n[0]:(i + 1) * n[0]]
            assert (part - want).abs().max() <= 1e-12 * want.abs().max(), (i, j)
