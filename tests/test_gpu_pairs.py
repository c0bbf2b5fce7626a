"""The sorted pair export at the edges of its thread blocks, scan tiles and capacities."""
import ctypes as C

import numpy as np
import pytest

from oracle import oracle as O
from paper_1701_02059_amd import inputs as I
from gpu_common import gpu_available

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not gpu_available():
        pytest.skip("needs a GPU")
    from paper_1701_02059_amd import rbc
    rbc.lib()
    return rbc


def _cloud(n, seed=3):
    """n lipids at the density of a sheet, ids in random order."""
    rng = np.random.default_rng(seed)
    side = int(np.ceil(np.sqrt(n)))
    g = np.stack(np.meshgrid(np.arange(side), np.arange(side), indexing="ij"), axis=-1).reshape(-1, 2)[:n] * 1.1
    x = np.concatenate([g + rng.normal(0, 0.02, g.shape), rng.normal(0, 0.02, (n, 1))], axis=1)[rng.permutation(n)]
    nrm = np.tile([0.0, 0.0, 1.0], (n, 1))
    return I.System("sheet", x, nrm, np.zeros(n, np.int32), np.zeros((n, 3)), np.zeros((n, 3)),
                    np.zeros((0, 2), np.int32), np.zeros(0), np.zeros(3), np.zeros(3, np.int32))


@pytest.mark.parametrize("n", [1, 2, 127, 128, 129, 2047, 2048, 2049, 4097, 70_001])
def test_pairs_sorted_at_block_and_tile_edges(R, mp, n):
    s = _cloud(n)
    c = R.Context(mp, R.RBC_MIXED)
    c.set_system(s)
    ref = O.pairs(O.params_for(s, mp), s.x, s.type)
    assert np.array_equal(c.get_pairs(), ref)
    assert np.array_equal(c.get_pairs_noalloc(), ref)
    # a buffer smaller than the set receives the first pairs and the full count
    cap = len(ref) // 2
    out = np.full((cap + 1, 2), -7, dtype=np.int32)
    cnt = C.c_int64(0)
    L = R.lib()
    assert L.rbc_get_pairs(c._h, cap, out.ctypes.data_as(C.POINTER(C.c_int32)), C.byref(cnt)) == R.RBC_OK
    assert cnt.value == len(ref) and np.array_equal(out[:cap], ref[:cap]) and (out[cap] == -7).all()
    # the allocation-free export writes nothing then
    out[:] = -7
    assert L.rbc_get_pairs_noalloc(c._h, cap, out.ctypes.data_as(C.POINTER(C.c_int32)), C.byref(cnt)) == R.RBC_OK
    assert cnt.value == len(ref) and ((out == -7).all() or len(ref) == 0)
    c.step(3, 0.01)                                   # the sort scratch is free again for the updates
    c.update_cells(0)
    x = c.get_state()[0].cpu().numpy()
    assert np.array_equal(c.get_pairs(), O.pairs(O.params_for(s, mp), x, s.type))
    c.close()
