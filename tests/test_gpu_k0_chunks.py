"""k = 0 in FP32 over z chunks of several planes, with ragged tiles and a ragged last chunk, against the FP64
oracle: ||R_gpu,i - R_orc,i|| / max_j ||R_orc,j|| <= 2e-5, as for the other stage kernels; and a slab of it,
whose chunks start at other planes, bit for bit (cells of height 1, so both have the same widths)."""
import numpy as np
import pytest

import oracle as O
from tests.layout import from_abi
from tests.test_gpu_k0_sweep import G, dgm, state  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [(130, 62, 101), (256, 64, 129)])
def test_chunks_against_the_oracle(dgm, prec, n):  # noqa: F811
    box = (1.0, 1.0, float(n[2]))
    s = dgm.Solver(0, n, box=box, gamma=G, precision=prec)
    y = state(0, n, s.dtype)
    r = s.rhs(y)
    want = O.rhs(O.make_cfg(0, n, box=box, gamma=G), from_abi(y.cpu().double().numpy())).reshape(5, -1)
    d = from_abi(r.cpu().double().numpy()).reshape(5, -1) - want
    err = np.linalg.norm(d, axis=1) / np.linalg.norm(want, axis=1).max()
    assert np.all(err <= {"fp64": 1e-12, "fp32": 2e-5}[prec]), err
    part = dgm.Solver(0, (n[0], n[1], 40), box=(1.0, 1.0, 40.0), gamma=G, precision=prec, zhalo=True)
    part.set_halo(y[6].clone(), y[47].clone())
    assert torch.equal(part.rhs(y[7:47].clone()), r[7:47])
