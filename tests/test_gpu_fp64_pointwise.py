"""The FP64 reciprocal and square root of the pointwise physics over the whole range of their operands:
the ends (zeros, infinities, not a number, a quotient past the largest double) exactly as 1 / x and
sqrt(x), everything else to two units in the last place (subnormal results: of the subnormals')."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pointwise():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1602_09079_amd import dg
    f = dg.lib().dgmi_pointwise64
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]

    def run(x):
        d = torch.from_numpy(x).cuda()
        r, q = torch.empty_like(d), torch.empty_like(d)
        assert f(d.data_ptr(), d.numel(), r.data_ptr(), q.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
        return r.cpu().numpy(), q.cpu().numpy()
    return run


def test_ends_of_the_range(pointwise):
    # 1e-300: the smallest pressure of the exact Riemann solver; 1 / 5.5e-309 is past the largest double
    x = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 5e-324, -5e-324, 1e-310, -1e-310, 5.5e-309])
    with np.errstate(all="ignore"):
        rcp, root = 1.0 / x, np.sqrt(x)
    got_rcp, got_root = pointwise(x)
    np.testing.assert_array_equal(got_rcp, rcp)
    np.testing.assert_array_equal(np.signbit(got_rcp[:4]), np.signbit(rcp[:4]))
    ends = np.array([0, 1, 2, 3, 4, 6, 8])
    np.testing.assert_array_equal(got_root[ends], root[ends])
    np.testing.assert_array_equal(np.signbit(got_root[:2]), np.signbit(root[:2]))


def test_between_the_ends(pointwise):
    rng = np.random.default_rng(0)
    x = np.concatenate([10.0 ** rng.uniform(-300, 300, 20000), rng.uniform(0.25, 4.0, 20000),
                        [1e-300, 5.6e-309, 2.2250738585072014e-308, 1e-308, 1.0, 4.0, 1e307, 1.7976931348623157e308]])
    got_rcp, got_root = pointwise(x)
    for got, want in ((got_rcp, 1.0 / x), (got_root, np.sqrt(x))):
        assert np.all(np.abs(got - want) <= 2 * np.spacing(want)), x[np.abs(got - want) > 2 * np.spacing(want)]
    got_rcp, _ = pointwise(-x)
    assert np.all(np.abs(got_rcp + 1.0 / x) <= 2 * np.spacing(1.0 / x))


@pytest.mark.parametrize("k", [0, 1, 2, 3])
def test_flux_at_a_cell_of_the_largest_density(k):
    """Beside a column of gas too heavy to move, HLLC's momentum difference overflows and its reciprocal
    is zero: the contact stands still and the flux is the wall's.  R before the column is then that of any
    other immovable one: at 1e280 the contact's speed is 1e-280 and R differs by rounding only.  (On its far
    side the column's own star state is formed, infinity times zero.)"""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1602_09079_amd import dg
    n = (8, 5, 4)
    s = dg.Solver(k, n, precision="fp64")
    r = []
    # (an infinite mean at k >= 1: the matrix kernels multiply it by the zeros of their tables)
    for heavy in (1e280, 1.7e308) + ((float("inf"),) if k == 0 else ()):
        y = s.empty_state().zero_()
        y[:, :, 0, 0] = 1.0
        y[:, :, 1, 0] = 0.2
        y[:, :, 4, 0] = 2.5
        y[:, :, 0, 0, 3] = heavy
        y[:, :, 1, 0, 3] = 0.0
        r.append(s.rhs(y)[..., [0, 1, 2, 5, 6, 7]])
    assert r[0].abs().max() > 1.0
    for got in r[1:]:
        assert (got - r[0]).abs().max() <= 1e-14 * r[0].abs().max()
