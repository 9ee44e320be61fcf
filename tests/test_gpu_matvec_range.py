"""kkt_matvec at the ends of the FP64 range, where its modes overflow or meet
infinities with both signs: the results are those of the sum over neighbours."""
import numpy as np
import pytest

from oracle import kkt
from workloads.generate import make_custom, DTO, OTD

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# one tile and one march; several tiles; one plane per march
MESHES = [((3, 2, 1), 3, DTO), ((20, 19, 5), 4, OTD), ((2, 2, 9), 300, DTO)]


@pytest.fixture(scope="module")
def st():
    import paper_1508_06103_amd as st_mod
    assert torch.cuda.is_available()
    return st_mod


def _setup(st, n, M, variant):
    prob = make_custom(n, M, 31, variant=variant, sensors=np.array([1 + (n[0] + 1)], dtype=np.int32))
    return st.KKTOperator(prob), kkt.assemble(prob).tocsr()


def _matvec(op, x):
    return op.matvec(torch.from_numpy(x).cuda()).cpu().numpy()


# (on the third mesh a row's diffusion entries alone, times 2^1023, are past the range: any order of the sum overflows)
@pytest.mark.parametrize("n,M,variant", MESHES[:2])
def test_large_entries(st, n, M, variant):
    print(f"case {n} x {M} variant {variant}", flush=True)
    op, F = _setup(st, n, M, variant)
    x = np.random.default_rng(1).uniform(2.5, 3.0, F.shape[0])
    x[2::3] *= 2.0 ** -40   # f enters divided by the time step
    y = _matvec(op, x * 2.0 ** 1020)   # two levels of c and a pair of neighbours are below 2^1024, eight values not
    assert np.isfinite(y).all()
    assert np.abs(y * 2.0 ** -1020 - F @ x).max() <= 1e-13 * (abs(F) @ x).max()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("n,M,variant", MESHES)
def test_one_non_finite_entry(st, n, M, variant, value):
    op, F = _setup(st, n, M, variant)
    nn = [k + 1 for k in n]
    N = nn[0] * nn[1] * nn[2]
    x = np.random.default_rng(2).standard_normal(F.shape[0])
    clean = _matvec(op, x)
    # a node inside x (the ends are Dirichlet) at the far corner of y and z
    node = n[0] - 1 + nn[0] * (n[1] + nn[1] * n[2])
    for slot in range(3):
        k = 3 * ((M // 2) * N + node) + slot
        print(f"case {n} x {M} variant {variant} entry {k} {value}", flush=True)
        bad = x.copy()
        bad[k] = value
        y = _matvec(op, bad)
        column = F[:, [k]].tocoo()
        hit = np.zeros(F.shape[0], dtype=bool)
        hit[column.row[column.data != 0]] = True
        assert not np.isfinite(y[hit]).any()
        # the entry's neighbours in space and time have no more rows than these
        near = np.zeros((M + 1, *nn[::-1], 3), dtype=bool)
        near[max(M // 2 - 1, 0):M // 2 + 2, n[2] - 1:, n[1] - 1:, n[0] - 2:] = True
        far = ~near.ravel()
        assert np.array_equal(y[far], clean[far])
        if slot == 2 and not np.isnan(value):
            # f enters the state rows through the mass matrix alone: one sign everywhere
            c = hit.copy()
            c.reshape(-1, 3)[:, 1:] = False
            assert c.any() and (y[c] == -value).all()


# thin meshes on both sides of the lines where the sum over neighbours serves the whole call: 4 columns and marches of 2
# and 3 planes, 16 columns and marches of 5 and 6
@pytest.mark.parametrize("n,M,variant", [((1, 1, 9), 204, DTO), ((1, 1, 10), 204, OTD), ((3, 3, 24), 204, OTD),
                                         ((3, 3, 29), 204, DTO)])
def test_thin_meshes(st, n, M, variant):
    print(f"case {n} x {M} variant {variant}", flush=True)
    prob = make_custom(n, M, 32, variant=variant, faces=0, sensors=np.array([5], dtype=np.int32))
    op, F = st.KKTOperator(prob), kkt.assemble(prob).tocsr()
    x = np.random.default_rng(3).standard_normal(F.shape[0])
    # a few hundred roundings per entry, of terms no larger than |F| |x|
    assert np.abs(_matvec(op, x) - F @ x).max() <= 1e-13 * (abs(F) @ np.abs(x)).max()
