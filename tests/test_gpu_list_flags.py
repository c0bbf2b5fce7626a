"""Block-wide flags of the list build and the prune: the longest list over blocks without a
stage, and the prune that keeps every row where a block's offsets leave the FP32 range."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from paper_1701_02059_amd import inputs as I
from tests.gpu_common import gpu_available, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not gpu_available():
        pytest.skip("needs a GPU")
    from paper_1701_02059_amd import rbc
    rbc.lib()
    return rbc


def _lipids(x, v=None):
    nrm = np.tile([0.0, 0.0, 1.0], (len(x), 1))
    return I.System("flags", x, nrm, np.zeros(len(x), np.int32), np.zeros(x.shape) if v is None else v, np.zeros(x.shape),
                    np.zeros((0, 2), np.int32), np.zeros(0), np.zeros(3), np.zeros(3, np.int32))


def test_longest_list_of_blocks_without_a_union(R, mp):
    rng = np.random.default_rng(5)
    g = np.stack(np.meshgrid(np.arange(64), np.arange(64), [0.0], indexing="ij"), axis=-1).reshape(-1, 3) * 1.1
    x = (g + rng.normal(0, 0.03, g.shape))[rng.permutation(len(g))]
    d2 = ((x[:, None, :] - x[None, :, :]) ** 2).sum(-1)
    longest = int((d2 < (mp.r_c + 2 * mp.skin) ** 2).sum(1).max()) - 1
    c = R.Context(dataclasses.replace(mp, cell_target=1), R.RBC_FP64)
    c.set_system(_lipids(x))
    assert (c.debug_array(9) < 0).all()
    for _ in range(5):
        assert c.stats()["max_list_rows"] == longest
        c.update_cells(0)
    c.close()


def test_prune_keeps_every_row_beyond_the_fp32_offsets(R, mp):
    """One block of two sheets a little less than 4096 sigma apart, moving away from each other."""
    rng = np.random.default_rng(6)
    g = np.stack(np.meshgrid([0.0], np.arange(10), np.arange(10), indexing="ij"), axis=-1).reshape(-1, 3) * 1.15
    a, b = (g + rng.normal(0, 0.005, g.shape) for _ in range(2))
    x = np.r_[a, b + [4095.9, 0.0, 0.0]]
    v = np.r_[np.tile([-1.0, 0.0, 0.0], (len(a), 1)), np.tile([1.0, 0.0, 0.0], (len(b), 1))]
    q = dataclasses.replace(mp, eps=0.0, skin=0.65, inner_skin=0.15, update_every=1000)
    s = _lipids(x, v)
    c = R.Context(q, R.RBC_MIXED)
    c.set_system(s)
    rows, pruned = c.debug_array(8), c.debug_array(13)
    assert (c.debug_array(9) >= 0).all() and (pruned < rows).any()       # staged, and the build prunes
    st0 = c.stats()
    while c.stats()["prunes"] == st0["prunes"]:                          # away by 0.1 to 0.15 each
        assert c.stats()["steps"] < 40
        c.step(1, 0.01)
    assert c.stats()["rebuilds"] == st0["rebuilds"]
    x = to_np(c.get_state()[0])
    assert x[len(a):, 0].max() - x[:len(a), 0].min() > 4096.0
    assert np.array_equal(c.debug_array(13), c.debug_array(8)) and np.array_equal(c.debug_array(8), rows)
    assert np.array_equal(c.get_pairs(), O.pairs(O.params_for(s, q), x, s.type))
    c.close()
