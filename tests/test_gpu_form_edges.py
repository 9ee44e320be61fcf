"""Kernels at the edges of their forms, against the oracle: tiles and z chunks
of the operator application, ring sweeps with one, two and four chunks a phase,
Gram-Schmidt passes over one and several ranges, coarse blocks around the
64-row panels with every kind of coarsened axis."""
import sys

import numpy as np
import pytest

from oracle import kkt, krylov, ras as oras, twolevel
from workloads.generate import make_custom, OTD

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def st():
    import paper_1508_06103_amd as st_mod
    assert torch.cuda.is_available()
    return st_mod


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# one tile of 1, 2, 3 and 4 wavefronts; tiles cut in x, in y and in both; one plane, a march of several
# planes in chunks of 3 with a remainder (many levels), chunks of one plane
MATVEC = [((2, 2, 2), 1, {}), ((9, 7, 2), 3, {}), ((10, 13, 2), 2, {}), ((13, 13, 3), 2, {}), ((90, 2, 2), 2, {}),
          ((2, 95, 3), 2, dict(variant=OTD)), ((20, 19, 2), 3, dict(faces=0b111111)), ((2, 2, 9), 300, {}),
          ((2, 3, 5), 500, dict(variant=OTD, faces=0)), ((3, 2, 1), 4, dict(faces=0b000001, sensors=np.array([5], dtype=np.int32)))]


@pytest.mark.parametrize("n,M,kw", MATVEC)
def test_matvec_tiles(st, n, M, kw):
    kw = dict(kw)
    if kw.get("faces") == 0b111111:
        nn = (n[0] + 1, n[1] + 1)
        kw["sensors"] = np.array([5 + nn[0] * (4 + nn[1]), 8 + nn[0] * (9 + nn[1])], dtype=np.int32)
    prob = make_custom(n, M, 21, lattice=1, **kw)
    _say(f"case {n} x {M}")
    op = st.KKTOperator(prob)
    F = kkt.assemble(prob)
    x = np.random.default_rng(2).standard_normal(F.shape[0])
    y = op.matvec(_dev(x)).cpu().numpy()
    ref = F @ x
    # a few hundred roundings per entry, of terms no larger than |F| |x|
    assert np.abs(y - ref).max() <= 1e-13 * (abs(F) @ np.abs(x)).max()


# boxes whose widest level has at most 32 rows, at most 64, and several chunks
BOXES = [((3, 2, 2), 2, (1, 1, 1, 1), 0), ((4, 5, 6), 5, (1, 2, 1, 2), 1), ((6, 6, 6), 6, (1, 1, 1, 1), 0),
         ((9, 9, 7), 8, (1, 1, 1, 1), 0), ((11, 11, 10), 12, (1, 1, 1, 1), 0), ((12, 4, 10), 20, (2, 1, 1, 1), 2)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,M,parts,delta", BOXES)
def test_ring_sweeps(st, n, M, parts, delta, prec):
    prob = make_custom(n, M, 22, lattice=1)
    _say(f"case {n} x {M} parts {parts} overlap {delta} {prec}")
    op = st.KKTOperator(prob)
    pre = st.RAS(op, parts, delta, precision=st.F64 if prec == "f64" else st.F32)
    R = oras.RAS(prob, parts, delta, terms=kkt.kkt_terms(prob))
    for seed in (3, 4):
        r = np.random.default_rng(seed).standard_normal(prob.unknowns)
        z = pre.apply(_dev(r)).cpu().numpy()
        ref = R.apply(r)
        # FP32: factors, values and sums rounded to 24 bits, carried through two triangular solves
        assert np.linalg.norm(z - ref) <= (1e-11 if prec == "f64" else 1e-4) * np.linalg.norm(ref)


# unknowns: one range with a remainder, three ranges; basis sizes up to the restart cross every group of vectors
@pytest.mark.parametrize("n,M,restart", [((3, 3, 3), 9, 12), ((7, 7, 7), 6, 12), ((5, 5, 5), 7, 70)])
def test_short_krylov_vectors(st, n, M, restart):
    prob = make_custom(n, M, 23, lattice=1)
    steps = 30 if restart < 30 else 20
    _say(f"case {n} x {M} restart {restart}, {steps} steps")
    op = st.KKTOperator(prob)
    parts = (1, 2, 2, 2)
    pre = st.RAS(op, parts, 1)
    R = oras.RAS(prob, parts, 1, terms=kkt.kkt_terms(prob))
    F = kkt.assemble(prob)
    b = kkt.rhs(prob)
    x, _ = st.solve(op, pre, restart=restart, rtol=1e-6, fixed_iters=steps)
    xo, _ = krylov.gmres(lambda v: F @ v, R.apply, b, restart=restart, rtol=1e-6, flexible=True, fixed_iters=steps)
    assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-7 * np.linalg.norm(xo)


# coarse blocks of 24, 63 + a remainder, 192 (three whole panels, two tiles) and 375 rows; axes with factor 1
COARSE = [((2, 2, 2), 2, (2, 2, 2, 2)), ((3, 4, 2), 6, (1, 2, 1, 3)), ((9, 6, 6), 4, (3, 2, 2, 4)),
          ((4, 8, 12), 6, (1, 2, 3, 1)), ((4, 4, 4), 3, (1, 1, 1, 3)), ((4, 4, 4), 3, (1, 1, 2, 1)),
          ((4, 4, 8), 4, (1, 1, 2, 2))]


@pytest.mark.parametrize("n,M,fac", COARSE)
def test_coarse_block_sizes(st, n, M, fac):
    nn = (n[0] + 1, n[1] + 1)
    mid = [fac[k] * max(1, (n[k] // fac[k]) // 2) for k in range(3)]
    if mid[0] == n[0]:
        mid[0] -= fac[0]   # off the Dirichlet face
    sens = np.array([mid[0] + nn[0] * (mid[1] + nn[1] * mid[2])], dtype=np.int32)
    prob = make_custom(n, M, 24, sensors=sens, faces=0 if mid[0] == 0 else 0b000011)
    _say(f"case {n} x {M} factor {fac}")
    op = st.KKTOperator(prob)
    tl = twolevel.TwoLevel(prob, None, None, fac, coarse="lu")
    X = np.random.default_rng(25).standard_normal((17, prob.unknowns))
    Xd = _dev(X)
    ref = np.stack([tl.coarse_correction(v) for v in X])
    size = np.linalg.norm(ref, axis=1)
    for prec, tol in ((st.F64, 1e-9), (st.F32, 1e-4)):
        C = st.Coarse(op, fac, method=st.COARSE_LU, precision=prec)
        assert np.linalg.norm(C.apply(Xd[0].contiguous()).cpu().numpy() - ref[0]) <= tol * size[0]
        for q in (2, 4, 5, 17):
            Y = C.apply_multi(Xd[:q].contiguous()).cpu().numpy()
            assert (np.linalg.norm(Y - ref[:q], axis=1) <= tol * size[:q]).all(), (prec, q)
