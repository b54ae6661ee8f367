"""dg_mlp_workspace_bytes: what the form that a shape takes lays out, and enough for every smaller batch (a
workspace made for one batch serves the smaller ones)."""
import pytest


@pytest.mark.parametrize("shape", [(140, 128, 128, 20), (7, 5, 3, 300), (16, 17, 65, 1), (900, 500, 300, 40)])
def test_workspace_of_one_form(shape):
    from paper_1602_09079_amd import dg
    nb = [dg.lib().dg_mlp_workspace_bytes(dg._shape_arr(shape), b) for b in (1, 15, 16, 17, 4096, 9001, 65536)]
    assert nb == sorted(nb)
    # activations and signals of every sample; in the separate products' form the outputs and targets too
    nin, h1, h2, no = shape
    fused = nin < 900
    for b, n in zip((1, 15, 16, 17, 4096, 9001, 65536), nb):
        bp = -(-b // 16) * 16
        if fused:  # at most 32 shares of the gradient beside them
            np_ = dg.mlp_nparams(shape)
            splits = min(32, -(-bp // 256))
            most = 4 * (bp * (nin + 2 * h1 + 2 * h2 + no) + splits * (np_ + 3)) + 8 * (splits * (h1 + h2 + no) + bp // 16) + 64
            assert 4 * bp * (nin + 2 * h1 + 2 * h2 + no) < n <= most, (b, n, most)
        else:
            assert n == 4 * b * (nin + 2 * h1 + 2 * h2 + 3 * no) + 64
