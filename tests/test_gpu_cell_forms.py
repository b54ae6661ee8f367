"""The one-cell-per-lane stage kernel (k = 1, 2 in FP64 and FP32) on both sides of its form rule: tiles of
16 x 4 cells times planes of the whole mesh, split over waves by task up to 1536 (k = 1) or 768 (k = 2; in
FP32 512), one wave a tile and chunk beyond.  Meshes just inside and just past the rule, one exact tile and one cell
more, against the FP64 oracle; the form a z slab takes; the production form of four waves a workgroup;
and the form's time where the other one takes well over half as long again.

Tolerance on R as for the other stage kernels: ||R_gpu,i - R_orc,i|| / max_j ||R_orc,j|| <= 1e-12 (FP64),
2e-5 (FP32)."""
import numpy as np
import pytest

import oracle as O
from paper_1602_09079_amd import synth
from tests.layout import from_abi
from tests.test_gpu_cell_stage import G, TOL, dgm, state  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LIMIT = {1: 1536, 2: 768}


def tiles(n):
    return -(-n[0] // 16) * -(-n[1] // 4)


def driven(dg, k, n, prec, **kw):
    s = dg.Solver(k, n, gamma=G, precision=prec, forcing=True, **kw)
    nvec = synth.forcing_modes(1.0, 3.0)
    ah = 0.05 * synth.ou_stationary_start(7, len(nvec))
    s.set_forcing(nvec, ah)
    return s, O.ForcingTable(nvec, ah)


def check(s, k, n, prec, y, r, frc, riemann="hllc"):
    want = O.rhs(O.make_cfg(k, n, gamma=G, riemann=riemann), from_abi(y.cpu().double().numpy()), frc).reshape(5, -1)
    d = from_abi(r.cpu().double().numpy()).reshape(5, -1) - want
    err = np.linalg.norm(d, axis=1) / np.linalg.norm(want, axis=1).max()
    assert np.all(err <= TOL[prec]), err


# one exact tile, one cell more, one fewer; thin meshes of many tiles; long meshes of few tiles; on the
# limit (32 x 32, 16 tiles, 48 or 96 planes) and one plane past it
@pytest.mark.parametrize("k,n", [(1, (16, 4, 3)), (2, (16, 4, 3)), (1, (17, 5, 3)), (2, (17, 5, 3)), (2, (15, 3, 3)),
                                 (1, (80, 70, 2)), (2, (80, 70, 2)), (1, (20, 6, 385)), (2, (20, 6, 193)),
                                 (1, (32, 32, 96)), (1, (32, 32, 97)), (2, (32, 32, 48)), (2, (32, 32, 49))])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_rhs_about_the_form_rule(dgm, prec, k, n):  # noqa: F811
    s, frc = driven(dgm, k, n, prec)
    y = state(s, n)
    check(s, k, n, prec, y, s.rhs(y), frc)


@pytest.mark.parametrize("n", [(32, 32, 32), (32, 32, 33), (16, 3, 512), (5, 4, 513)])
def test_rhs_about_the_line_of_k2_fp32(dgm, n):  # noqa: F811
    s, frc = driven(dgm, 2, n, "fp32")
    y = state(s, n)
    check(s, 2, n, "fp32", y, s.rhs(y), frc)


@pytest.mark.parametrize("k,nz", [(1, 90), (2, 45)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_placed_slabs_take_the_form_of_the_whole_mesh(dgm, prec, k, nz):  # noqa: F811
    """The mesh is past the limit and its slabs are not: placed by set_slab they give its bits, with and
    without driving.  (Cells of height 1: the slab's box over its planes is exactly the whole mesh's.)"""
    n, dz = (40, 24, nz), nz // 3
    assert tiles(n) * dz <= LIMIT[k] < tiles(n) * nz
    whole, _ = driven(dgm, k, n, prec, box=(1.0, 1.0, float(nz)))
    plain = dgm.Solver(k, n, box=(1.0, 1.0, float(nz)), gamma=G, precision=prec)
    y = state(whole, n)
    want, want_plain = whole.rhs(y), plain.rhs(y)
    nvec = synth.forcing_modes(1.0, 3.0)
    ah = 0.05 * synth.ou_stationary_start(7, len(nvec))
    for lo in range(0, nz, dz):
        hi = lo + dz
        for ref, force in ((want, True), (want_plain, False)):
            s = dgm.Solver(k, (n[0], n[1], dz), box=(1.0, 1.0, float(dz)), gamma=G, precision=prec, forcing=force,
                           zhalo=True)
            s.set_slab(lo, nz)
            if force:
                s.set_forcing(nvec, ah)
            s.set_halo(y[lo - 1].clone(), y[hi % nz].clone())
            assert torch.equal(s.rhs(y[lo:hi].clone()), ref[lo:hi]), (lo, force)


@pytest.mark.parametrize("k,prec,riemann", [(1, "fp64", "hllc"), (1, "fp32", "exact"), (2, "fp64", "hllc"),
                                            (2, "fp32", "hllc")])
def test_four_waves_a_workgroup(dgm, k, prec, riemann):  # noqa: F811
    """More than 1024 items of two planes, one of them alone in the last workgroup, ragged tiles in x and y:
    the form of the large meshes (32-bit plane offsets, four waves of a workgroup with their own LDS regions).
    Chunks of other lengths, with fewer items than a workgroup of four is used for, give the same bits."""
    n = (70, 43, 61)
    items = tiles(n) * -(-n[2] // 2)
    assert items > 1024 and items % 4 == 1 and tiles(n) * n[2] > LIMIT[k]
    assert tiles(n) * -(-n[2] // 4) < 1024
    s, frc = driven(dgm, k, n, prec, riemann=riemann)
    y = state(s, n)
    s.set_zchunk(2)
    r = s.rhs(y)
    check(s, k, n, prec, y, r, frc, riemann)
    for zl in (4, 61, 1):
        s.set_zchunk(zl)
        assert torch.equal(s.rhs(y), r), zl


def stage_time(dg, k, n, prec):
    s, _ = driven(dg, k, n, prec)
    y = state(s, n)
    out = torch.empty_like(y)
    best = 1e9
    for _ in range(8):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record()
        for _ in range(10):
            s.stage(y, y, out, 0.75, 0.25, 1e-6)
        ev[1].record()
        torch.cuda.synchronize()
        best = min(best, ev[0].elapsed_time(ev[1]))
    return best


@pytest.mark.parametrize("k,prec,n,like,most", [(2, "fp32", (32, 32, 256), (64, 64, 64), 1.4),
                                                (2, "fp64", (64, 64, 2), (16, 16, 16), 1.6)])
def test_form_of_long_and_of_thin_meshes(dgm, k, prec, n, like, most):  # noqa: F811
    """A long mesh of small planes takes the time of a compact one of as many cells (measured 0.95 of it in
    the unsplit form, 1.76 split); a thin mesh of few tiles that of a small mesh (1.03 split, 2.3 unsplit)."""
    assert stage_time(dgm, k, n, prec) <= most * stage_time(dgm, k, like, prec)
