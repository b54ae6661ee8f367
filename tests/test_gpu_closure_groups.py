"""Closure inference where its groups of 16 cells end: fewer cells than one workgroup's waves take, a
ragged last group, and more groups than a full grid of 256 x 8 waves holds at once, so that some waves
take a second group and prefetch past their last one.

Against the FP64 oracle, at the bounds of the FP32 network: 1e-5 of the largest field norm (FP64
storage), 3e-5 with FP32 storage, whose plain operator is bounded at 2e-5.  A repeated call gives the
same bits: the mean rows are summed in a fixed order.
"""
import numpy as np
import pytest

import oracle as O
from tests.layout import from_abi, to_abi
from tests.test_gpu_closure import _network, dev, dgm, rhs_err, turb  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [(3, 3, 3), (5, 7, 3), (43, 29, 27)])
def test_closure_groups(dgm, n, prec):  # noqa: F811
    cfg, y = turb(1, n, seed=31)
    p, fmean, fstd, scale = _network(cfg, y, np.random.default_rng(17))
    bound = np.full(20, 1e30)
    corr, nfb = O.closure_correction(cfg, y, O.ClosureParams(p, fmean, fstd, scale, bound))
    assert nfb == 0
    s = dgm.Solver(1, n, precision=prec, closure=True)
    s.set_closure(p, fmean, fstd, scale, bound)
    yd = dev(to_abi(y), s.dtype)
    r = s.rhs(yd)
    assert s.closure_fallbacks() == 0
    err = rhs_err(from_abi(r.cpu().double().numpy()), O.rhs(cfg, y) - corr)
    assert np.all(err <= {"fp64": 1e-5, "fp32": 3e-5}[prec]), err
    torch.testing.assert_close(s.rhs(yd), r, rtol=0, atol=0)
    # a second network replaces the first one's layout on the device
    p2, *rest = _network(cfg, y, np.random.default_rng(18))
    corr2, _ = O.closure_correction(cfg, y, O.ClosureParams(p2, *rest, bound))
    s.set_closure(p2, *rest, bound)
    err = rhs_err(from_abi(s.rhs(yd).cpu().double().numpy()), O.rhs(cfg, y) - corr2)
    assert np.all(err <= {"fp64": 1e-5, "fp32": 3e-5}[prec]), err
