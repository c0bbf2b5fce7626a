"""State and forces in the caller's order at the sizes where the way of writing them changes."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1701_02059_amd import inputs as I
from tests.gpu_common import gpu_available, rel_err, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not gpu_available():
        pytest.skip("needs a GPU")
    from paper_1701_02059_amd import rbc
    rbc.lib()
    return rbc


@pytest.mark.parametrize("n", [1, 65_535, 65_536, 1_310_720, 1_310_721])
def test_outputs_in_caller_order(R, mp, n):
    import torch
    rng = np.random.default_rng(n)
    side = int(np.ceil(np.sqrt(n)))
    g = np.stack(np.meshgrid(np.arange(side), np.arange(side), [0.0], indexing="ij"), axis=-1).reshape(-1, 3)[:n] * 1.1
    x = (g + rng.normal(0, 0.03, g.shape))[rng.permutation(n)]
    nrm = rng.normal(0, 0.1, (n, 3)) + [0.0, 0.0, 1.0]
    nrm /= np.linalg.norm(nrm, axis=1)[:, None]
    s = I.System("sheet", x, nrm, np.zeros(n, np.int32), rng.normal(size=(n, 3)), rng.normal(size=(n, 3)),
                 np.zeros((0, 2), np.int32), np.zeros(0), np.zeros(3), np.zeros(3, np.int32))
    c = R.Context(mp, R.RBC_FP64)
    c.set_system(s)
    for got, want in zip(c.get_state(), (s.x, s.n, s.v, s.w)):
        assert np.array_equal(to_np(got), want)
    F, T = (to_np(t) for t in c.forces())
    idx = np.sort(rng.choice(n, min(n, 400), replace=False)).astype(np.int64)
    F0, T0 = O.forces_subset(O.params_for(s, mp), s, idx)[:2]
    assert rel_err(F[idx], F0) < 1e-10 and rel_err(T[idx], T0) < 1e-10     # as in the tests of whole systems
    # any output may be left out
    v = torch.full((n, 3), -7.0, dtype=torch.float64, device="cuda")
    t = torch.full_like(v, -7.0)
    assert R.lib().rbc_get_state(c._h, None, None, R._dev(v), None) == R.RBC_OK
    assert R.lib().rbc_forces(c._h, None, R._dev(t), None) == R.RBC_OK
    assert np.array_equal(to_np(v), s.v) and np.array_equal(to_np(t), T)
    c.close()
