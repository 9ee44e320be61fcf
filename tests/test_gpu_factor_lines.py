"""The ILU(0) factorisation by x lines at the edges of its workgroups: lines of
1, 2, 7 and 8 nodes (one or two wavefronts), 27 and 28 (the narrower and the
wider workgroup), 54 (the widest) and 56 (rows in parallel instead), boxes of
one line, of one level and of several workgroups per line level, FP32 factors."""
import sys

import numpy as np
import pytest

from oracle import kkt, ras as oras
from workloads.generate import make_custom

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = [((6, 4, 4), 5, (7, 1, 1, 1), 0), ((7, 5, 4), 4, (7, 1, 2, 1), 1), ((6, 9, 9), 9, (1, 1, 1, 1), 0),
         ((7, 3, 2), 3, (1, 4, 3, 4), 0), ((26, 3, 3), 3, (1, 1, 1, 1), 0), ((27, 3, 2), 3, (1, 1, 1, 1), 0),
         ((53, 2, 3), 2, (1, 1, 1, 1), 0), ((55, 2, 2), 2, (1, 1, 1, 1), 0), ((54, 2, 2), 2, (2, 1, 1, 1), 1)]


@pytest.fixture(scope="module")
def st():
    import paper_1508_06103_amd as st_mod
    assert torch.cuda.is_available()
    return st_mod


@pytest.mark.parametrize("n,M,parts,delta", CASES)
def test_factors_of_line_lengths(st, n, M, parts, delta):
    prob = make_custom(n, M, 11, lattice=1)
    print(f"case {n} x {M} parts {parts} overlap {delta}", flush=True)
    sys.stdout.flush()
    op = st.KKTOperator(prob)
    pre = st.RAS(op, parts, delta)
    f32 = st.RAS(op, parts, delta, precision=st.F32)
    R = oras.RAS(prob, parts, delta, terms=kkt.kkt_terms(prob))
    for sid in sorted({0, len(R.subs) // 2, len(R.subs) - 1}):
        want = R.ilu[sid].padded()
        scale = np.abs(want).max(axis=(1, 2, 3), keepdims=True)
        # the same products in the same order: a few units of rounding per entry through the elimination
        assert (np.abs(pre.export_factors(sid) - want) / scale).max() <= 1e-11
        # FP32 factors are the FP64 ones rounded once
        assert (np.abs(f32.export_factors(sid) - want) / scale).max() <= 2.0 ** -23
    r = np.random.default_rng(5).standard_normal(prob.unknowns)
    z = pre.apply(torch.from_numpy(r).cuda()).cpu().numpy()
    ref = R.apply(r)
    assert np.linalg.norm(z - ref) <= 1e-11 * np.linalg.norm(ref)
