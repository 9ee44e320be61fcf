"""The restriction's forms against the oracle: x and y in one launch or an axis
at a time, z and t in one launch or an axis at a time, and both mixtures, for
one vector and for more than one group of vectors."""
import numpy as np
import pytest

from oracle import twolevel
from workloads.generate import make_custom

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# few wide planes: by axes; many planes with long windows in z and t: x and y (or one of them) together, then z and t
# by axes (or one of them); neither x nor y, long windows; few wide planes and long windows
FORMS = [((40, 40, 4), 4, (20, 20, 2, 2)), ((4, 4, 24), 24, (2, 2, 12, 12)), ((2, 4, 24), 24, (1, 2, 24, 8)),
         ((4, 2, 36), 8, (2, 1, 36, 1)), ((4, 2, 4), 40, (2, 1, 1, 40)), ((4, 4, 24), 24, (1, 1, 12, 8)),
         ((60, 20, 10), 10, (20, 20, 10, 10))]


@pytest.fixture(scope="module")
def st():
    import paper_1508_06103_amd as st_mod
    assert torch.cuda.is_available()
    return st_mod


@pytest.mark.parametrize("n,M,fac", FORMS)
def test_correction_of_every_form(st, n, M, fac):
    print(f"case {n} x {M} factor {fac}", flush=True)
    nn = [k + 1 for k in n]
    # a coarse node off the Dirichlet faces x = 0 and x = 1
    ix = fac[0] if fac[0] < n[0] else 0
    node = np.array([ix], dtype=np.int32)
    prob = make_custom(n, M, 51, sensors=node, faces=0b000011 if ix else 0)
    op = st.KKTOperator(prob)
    tl = twolevel.TwoLevel(prob, None, None, fac, coarse="lu")
    X = np.random.default_rng(52).standard_normal((5, prob.unknowns))
    Xd = torch.from_numpy(X).cuda()
    ref = np.stack([tl.coarse_correction(v) for v in X])
    size = np.linalg.norm(ref, axis=1)
    C = st.Coarse(op, fac)
    one = C.apply(Xd[0].contiguous()).cpu().numpy()
    all5 = C.apply_multi(Xd).cpu().numpy()
    assert np.linalg.norm(one - ref[0]) <= 1e-9 * size[0]
    assert (np.linalg.norm(all5 - ref, axis=1) <= 1e-9 * size).all()
    assert np.array_equal(one, all5[0])   # the same form whatever the number of vectors
