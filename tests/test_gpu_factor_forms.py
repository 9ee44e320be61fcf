"""The ILU(0) factorisation by x lines and the one with a row per thread give the
same factors in every bit: on a mesh whose spacings and time step are no powers
of two, a box of 54 nodes along x is factored by lines where its neighbour has
54 nodes too, and row by row where the neighbour has 55."""
from types import SimpleNamespace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def st():
    import paper_1508_06103_amd as st_mod
    assert torch.cuda.is_available()
    return st_mod


def _problem(nx, h, variant, reg):
    """Elements of the last 53 along x are alike on every such mesh: one spacing, coefficients constant along x."""
    n, M = (nx, 4, 3), 5
    length = (nx * h, n[1] * h, n[2] * h)
    assert length[0] / nx == h
    a = np.random.default_rng(1).uniform(0.5, 2.0, (n[2], n[1], 1))
    node = np.array([nx - 3 + (nx + 1) * (2 + (n[1] + 1) * 1)], dtype=np.int32)
    return SimpleNamespace(n=n, M=M, a_elem=np.broadcast_to(a, (n[2], n[1], nx)).ravel(), v=(1.0, 0.5, 0.25),
                           beta1=1e-4, beta2=1e-3, sensor_node=node, data=np.zeros((M + 1, 1)), length=length, T=1.0,
                           dirichlet_faces=0b000011, variant=variant, reg=reg)


@pytest.mark.parametrize("variant,reg", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("h", [1 / 20, 1 / 24])
def test_factors_of_both_forms_in_bits(st, h, variant, reg):
    print(f"case h {h:.4f} variant {variant} regularisation {reg}", flush=True)
    got = []
    for nx, dims in ((107, (54, 54)), (108, (55, 54))):
        op = st.KKTOperator(_problem(nx, h, variant, reg))
        pre = st.RAS(op, (2, 1, 1, 1), 0)
        b = pre.boxes()
        assert tuple(b[:, 12] - b[:, 8]) == dims
        got.append(pre.export_factors(1))
    assert np.isfinite(got[0]).all()
    assert np.array_equal(got[0].view(np.uint64), got[1].view(np.uint64))
