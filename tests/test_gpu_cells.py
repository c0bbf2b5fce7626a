"""Cell builds and updates at the sizes where their kernels change: cells beyond the lanes',
the wavefront's and the block's share of members, one cell in all, the largest ranked and the
smallest radix-sorted number of cells.  Owners, centroids and the order inside a cell follow
the oracle."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from paper_1701_02059_amd import inputs as I
from tests.gpu_common import gpu_available

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not gpu_available():
        pytest.skip("needs a GPU")
    from paper_1701_02059_amd import rbc
    rbc.lib()
    return rbc


def _sheet(side, periodic=False, proteins=False):
    rng = np.random.default_rng(side)
    g = np.stack(np.meshgrid(np.arange(side), np.arange(side), [0.0], indexing="ij"), axis=-1).reshape(-1, 3) * 1.1
    x = g + rng.normal(0, 0.03, g.shape)
    typ = np.zeros(len(x), np.int32)
    if proteins:
        q = x[::5] + [0.3, 0.3, -2.0]
        x, typ = np.r_[x, q], np.r_[typ, np.where(np.arange(len(q)) % 9 == 0, 2, 1)].astype(np.int32)
    n = len(x)
    perm = rng.permutation(n)
    nrm = np.tile([0.0, 0.0, 1.0], (n, 1))
    nrm[typ > 0] = 0.0
    box = np.array([1.1 * side, 1.1 * side, 25.0]) if periodic else np.zeros(3)
    return I.System("sheet", x[perm], nrm[perm], typ[perm], np.zeros((n, 3)), np.zeros((n, 3)),
                    np.zeros((0, 2), np.int32), np.zeros(0), box, (box > 0).astype(np.int32))


def _renumbered(p, seeds, owner, kl):
    """Cells along the Morton curve of their centroids, the lipid cells first."""
    keys = O.morton_sets(p, seeds, kl)
    perm = np.lexsort((np.arange(keys.size), keys))
    inv = np.empty_like(perm)
    inv[perm] = np.arange(perm.size)
    return seeds[perm], inv[owner]


CASES = [(40, False, False, dict(cell_target=m)) for m in (1, 2, 16, 17, 63, 64, 65, 300, 5000)] + \
        [(40, True, False, dict(cell_target=m)) for m in (1, 16, 65)] + \
        [(40, False, True, dict(cell_target=m, protein_cells=1)) for m in (1, 16, 90, 3000)] + \
        [(70, False, True, dict(cell_target=2200)), (70, True, False, dict(cell_target=4000)),
         (181, False, False, dict(cell_target=1, lloyd_iters=1)), (182, False, False, dict(cell_target=1, lloyd_iters=1))]


@pytest.mark.parametrize("side,periodic,proteins,over", CASES,
                         ids=["-".join(map(str, (s, int(a), int(b), *o.values()))) for s, a, b, o in CASES])
def test_cells_at_the_edges_of_their_kernels(R, mp, side, periodic, proteins, over):
    s = _sheet(side, periodic, proteins)
    q = dataclasses.replace(mp, **over)
    p = O.params_for(s, q)
    c = R.Context(q, R.RBC_FP64)
    c.set_system(s)
    own, seeds = c.cells()
    if over.get("protein_cells"):
        seeds0, own0, kl = O.voronoi_init_sets(p, s, q.cell_target, q.lloyd_iters)
    else:
        (seeds0, own0), kl = O.voronoi_init(p, s, q.cell_target, q.lloyd_iters), 1 << 30
    seeds0, own0 = _renumbered(p, seeds0, own0, kl)
    assert np.array_equal(own, own0)
    assert np.abs(seeds - seeds0).max() < 1e-10
    # an update keeps the order of the members that a cell receives
    gid = c.debug_array(10).copy()
    c.update_cells(0)
    own2, seeds2 = c.cells()
    x, typ = s.x[gid], s.type[gid]
    if over.get("protein_cells"):
        ref, oref, order = O.voronoi_update_sets(p, x, typ, seeds, kl)
    else:
        ref, oref, order = O.voronoi_update(p, x, typ, seeds)
    assert np.array_equal(own2[gid], oref)
    assert np.abs(seeds2 - ref).max() < 1e-10
    assert np.array_equal(c.debug_array(10), gid[order])
    # the state moved with it
    out = c.get_state()
    assert np.array_equal(out[0].cpu().numpy(), s.x) and np.array_equal(out[1].cpu().numpy(), s.n)
    c.close()
