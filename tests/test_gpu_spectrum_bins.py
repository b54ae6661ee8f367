"""A spectrum of few shells is the head of the full one, bit for bit (rows and parts of rows past the last
shell asked for are not read): grids of even and odd side, shorter and longer than the 64 elements a wave
takes at a time."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("k,n,S", [(1, 5, 1), (1, 6, 2), (2, 33, 4), (0, 75, 3)])
def test_few_shells(prec, k, n, S):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1602_09079_amd import dg
    s = dg.Solver(k, (n, n, n), precision=prec)
    rng = np.random.default_rng(2)
    y = 0.05 * rng.standard_normal(s.state_shape())
    y[:, :, 0, 0] += 1.0
    y[:, :, 4, 0] += 2.0
    y = torch.from_numpy(y).to("cuda", s.dtype)
    M = n * S
    full = s.velocity_spectrum(y, S, nbins=M + 7)  # past the corner's shell: zeros
    last = int(np.floor(np.sqrt(3.0) * (M // 2) + 0.5))
    assert np.all(full[:last] > 0) and np.all(full[last + 1:] == 0)
    for nb in (1, 2, 3, M // 2, M // 2 + 1, M):
        np.testing.assert_array_equal(s.velocity_spectrum(y, S, nbins=nb), full[:nb])
