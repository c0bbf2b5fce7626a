"""Cell updates where a block takes each cell: around the line between the lanes' and the
blocks' way, cells with a few members or none beside large ones, and several systems at once."""
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


def _sheet(n, seed, periodic=False, far=0):
    rng = np.random.default_rng(seed)
    side = int(np.ceil(np.sqrt(n)))
    g = np.stack(np.meshgrid(np.arange(side), np.arange(side), [0.0], indexing="ij"), axis=-1).reshape(-1, 3)[:n] * 1.1
    x = g + rng.normal(0, 0.03, g.shape)
    if far:                                          # members of distant cells that hold little else
        x[rng.permutation(n)[:far]] += [0.0, 0.0, 400.0]
    typ = np.where(rng.random(n) < 0.2, 1, 0).astype(np.int32)
    typ[0] = 0                                       # (the oracle seeds from lipids)
    nrm = np.tile([0.0, 0.0, 1.0], (n, 1))
    nrm[typ > 0] = 0.0
    box = np.array([1.1 * side, 1.1 * side, 30.0]) if periodic else np.zeros(3)
    perm = rng.permutation(n)
    return I.System("sheet", x[perm], nrm[perm], typ[perm], np.zeros((n, 3)), np.zeros((n, 3)), np.zeros((0, 2), np.int32),
                    np.zeros(0), box, (box > 0).astype(np.int32))


def _reference(s, q):
    p = O.params_for(s, q)
    seeds, own = O.voronoi_init(p, s, q.cell_target, q.lloyd_iters)
    keys = O.morton_sets(p, seeds, 1 << 30)
    perm = np.lexsort((np.arange(keys.size), keys))
    inv = np.empty_like(perm)
    inv[perm] = np.arange(perm.size)
    return seeds[perm], inv[own]


@pytest.mark.parametrize("target", [55, 56, 57, 257, 2049, 4000, 10_000])
@pytest.mark.parametrize("kind", [dict(n=9001), dict(n=9001, periodic=True), dict(n=9001, far=3), dict(n=40), dict(n=1)],
                         ids=["sheet", "periodic", "far", "few", "one"])
def test_large_cells_follow_the_oracle(R, mp, kind, target):
    s = _sheet(seed=target, **kind)
    q = dataclasses.replace(mp, cell_target=target, lloyd_iters=3)
    c = R.Context(q, R.RBC_FP64)
    c.set_system(s)
    own, seeds = c.cells()
    seeds0, own0 = _reference(s, q)
    assert np.array_equal(own, own0)
    assert np.abs(seeds - seeds0).max() < 1e-10
    rad = c.debug_array(7)[:, 3]
    d = s.x - seeds[own]
    for a in range(3):
        if s.periodic[a]:
            d[:, a] -= s.box[a] * np.rint(d[:, a] / s.box[a])
    ref = np.zeros(len(seeds))
    np.maximum.at(ref, own, np.linalg.norm(d, axis=1))
    assert np.abs(rad - ref).max() < 1e-10
    assert np.array_equal(to_np(c.get_state()[0]), s.x)
    assert np.array_equal(c.get_pairs(), O.pairs(O.params_for(s, q), s.x, s.type))
    c.close()


def test_large_cells_of_several_systems(R, mp):
    q = dataclasses.replace(mp, cell_target=300, lloyd_iters=3)
    systems = [_sheet(n, n) for n in (1, 299, 5000, 20_000)]
    e = R.Ensemble(q, R.RBC_FP64, max_slots=4)
    slots = [e.stage(s) for s in systems]
    assert e.commit() == []
    e.step(6, 0.005)
    for s, k in zip(systems, slots):
        c = R.Context(q, R.RBC_FP64)
        c.set_system(s)
        c.step(6, 0.005)
        for a, b in zip(e.get_state(k), c.get_state()):
            assert np.array_equal(to_np(a), to_np(b))
        c.close()
    e.close()
