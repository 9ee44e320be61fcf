"""The correction of one vector on both sides of the block size where its chunk
sums get a launch of their own: against the oracle, and in bits against the
same vector among several."""
import numpy as np
import pytest

from oracle import twolevel
from workloads.generate import make_custom

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def st():
    import paper_1508_06103_amd as st_mod
    assert torch.cuda.is_available()
    return st_mod


# blocks of 1176 and 1344 rows (the line of the matrix-core form), 2430 and 2700 (of the FP32 GEMV), three levels
@pytest.mark.parametrize("c", [(6, 6, 7), (7, 6, 7), (8, 8, 9), (8, 9, 9)])
def test_one_vector_against_several(st, c):
    n = tuple(2 * k for k in c)
    print(f"case {n}, {3 * (c[0] + 1) * (c[1] + 1) * (c[2] + 1)} rows", flush=True)
    node = np.array([6 + (n[0] + 1) * (6 + (n[1] + 1) * 6)], dtype=np.int32)
    prob = make_custom(n, 4, 41, sensors=node)
    op = st.KKTOperator(prob)
    tl = twolevel.TwoLevel(prob, None, None, (2, 2, 2, 2), coarse="lu")
    X = np.random.default_rng(42).standard_normal((17, prob.unknowns))
    Xd = torch.from_numpy(X).cuda()
    ref = [tl.coarse_correction(X[i]) for i in (0, 16)]
    for prec, tol in ((st.F64, 1e-9), (st.F32, 1e-4)):
        C = st.Coarse(op, (2, 2, 2, 2), precision=prec)
        one = C.apply(Xd[0].contiguous()).cpu().numpy()
        few = C.apply_multi(Xd[:2].contiguous()).cpu().numpy()
        many = C.apply_multi(Xd).cpu().numpy()   # the last one alone in its pass
        last = C.apply_multi(Xd[15:].contiguous()).cpu().numpy()
        for got, want in ((one, ref[0]), (many[16], ref[1])):
            assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)
        if prec == st.F64:   # one FP64 vector takes the products of several
            assert np.array_equal(one, few[0])
        assert np.array_equal(many[16], last[1]) and np.array_equal(many[0], few[0])
        for q in (3, 5):   # vectors in fours, with a remainder
            assert np.array_equal(C.apply_multi(Xd[:q].contiguous()).cpu().numpy(), many[:q])
