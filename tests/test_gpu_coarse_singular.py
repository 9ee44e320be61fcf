"""A coarse level whose blocks overflow ends the elimination with EBREAKDOWN,
wherever the first non-finite pivot lies, and leaves the next setup alone."""
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


def _problem(n, layer):
    a = np.ones((n[2], n[1], n[0]))
    if layer is not None:
        a[layer] = 1.7e308   # element stiffness a h / 9 and more overflows at h = 100 / n
    node = np.array([1 + (n[0] + 1) * (1 + (n[1] + 1))], dtype=np.int32)
    return SimpleNamespace(n=n, M=2, a_elem=a.ravel(), v=(1.0, 0.5, 0.25), beta1=1e-4, beta2=1e-4, sensor_node=node,
                           data=np.zeros((3, 1)), length=(100.0, 100.0, 100.0), T=1.0, dirichlet_faces=0b000011,
                           variant=0, reg=0)


# one panel; six panels; 35 panels with tiles of the update beside them.  The first or the last element layer
@pytest.mark.parametrize("layer", [0, -1])
@pytest.mark.parametrize("n", [(2, 1, 2), (4, 4, 4), (8, 8, 8)])
def test_overflow_is_breakdown(st, n, layer):
    print(f"case {n} layer {layer}", flush=True)
    bad = st.KKTOperator(_problem(n, layer))
    with pytest.raises(st.StkktError) as e:
        st.Coarse(bad, (1, 1, 1, 2))
    assert e.value.code == st.EBREAKDOWN
    good = st.KKTOperator(_problem(n, None))
    x = torch.from_numpy(np.random.default_rng(1).standard_normal(good.n)).cuda()
    assert torch.isfinite(st.Coarse(good, (1, 1, 1, 2)).apply(x)).all()
