"""Neighbour lists where the block's stage, candidate lists and hit words run out or split.

Against the oracle's neighbour set and forces: at the build, and after steps that prune
and rebuild the lists.
"""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from paper_1701_02059_amd import inputs as I
from tests.gpu_common import PP_FP64_TOL, PP_MIXED_TOL, check_forces, gpu_available, to_np

pytestmark = pytest.mark.gpu

FP64_TOL = 1e-10          # as in the tests of whole systems
MIXED_TOL = 1e-5


@pytest.fixture(scope="module")
def R():
    if not gpu_available():
        pytest.skip("needs a GPU")
    from paper_1701_02059_amd import rbc
    rbc.lib()
    return rbc


def _system(x, typ, rng, box=(0.0, 0.0, 0.0)):
    n = len(x)
    perm = rng.permutation(n)
    nrm = rng.normal(0, 0.15, (n, 3)) + [0.0, 0.0, 1.0]
    nrm /= np.linalg.norm(nrm, axis=1)[:, None]
    typ = typ.astype(np.int32)
    nrm[typ > 0] = 0.0
    v = rng.normal(0, 0.4, (n, 3))
    box = np.asarray(box, float)
    return I.System("lists", x[perm], nrm[perm], typ[perm], v[perm], np.zeros((n, 3)), np.zeros((0, 2), np.int32),
                    np.zeros(0), box, (box > 0).astype(np.int32))


def _sheet(side, rng, z=0.0, a=1.1):
    g = np.stack(np.meshgrid(np.arange(side), np.arange(side), [0.0], indexing="ij"), axis=-1).reshape(-1, 3) * a
    return g + rng.normal(0, 0.02, g.shape) + [0.0, 0.0, z]


def _make(kind):
    rng = np.random.default_rng(11)
    if kind == "sheet":                     # with a layer of protein beads under it
        x, p = _sheet(40, rng), _sheet(18, rng, -1.6, 2.4)
        typ = np.r_[np.zeros(len(x)), np.where(np.arange(len(p)) % 7 == 0, 2, 1)]
        return _system(np.r_[x, p], typ, rng)
    if kind == "periodic":
        x = _sheet(40, rng)
        return _system(x, np.zeros(len(x)), rng, (44.0, 44.0, 30.0))
    if kind.startswith("gas"):              # single lipids far from the sheet make cells wide
        x = _sheet(40, rng)
        g = np.stack(np.meshgrid(*[np.arange(13)] * 3, indexing="ij"), axis=-1).reshape(-1, 3) * 4.0
        g = g[np.abs(g[:, 2] - 24.0) > 1.0] - [2.0, 2.0, 24.0]
        g = g[rng.permutation(len(g))[:int(kind[3:])]] + rng.normal(0, 0.1, (int(kind[3:]), 3))
        x = np.r_[x, g]
        return _system(x, np.zeros(len(x)), rng)
    if kind == "pillar":                    # one cell, with a far member on each side, pairs with every other
        x = _sheet(70, rng) * [1.0, 1.0, 0.0]
        x = np.r_[x, [[38.0, 38.0, 60.0], [38.0, 38.0, -60.0]]]
        s = _system(x, np.zeros(len(x)), rng)
        # neither of the two seeds a cell: their ids become the last ones
        far = np.flatnonzero(np.abs(s.x[:, 2]) > 50.0)
        order = np.r_[np.delete(np.arange(s.N), far), far]
        return dataclasses.replace(s, x=s.x[order], n=s.n[order], v=s.v[order])
    g = np.stack(np.meshgrid(*[np.arange(13)] * 3, indexing="ij"), axis=-1).reshape(-1, 3) * 1.2
    x = g + rng.normal(0, 0.01, g.shape)    # a solid: 80 partners per particle, 400 candidates per cell
    return _system(x, (rng.random(len(x)) < 0.2).astype(int), rng, (15.6, 15.6, 15.6) if kind == "solid-periodic" else (0, 0, 0))


CASES = [("sheet", dict()), ("sheet", dict(cell_target=9)), ("sheet", dict(cell_target=3)),
         ("sheet", dict(cell_target=1)), ("sheet", dict(cell_target=200)), ("sheet", dict(protein_cells=1, skin=0.65)),
         ("periodic", dict()), ("periodic", dict(cell_target=1)), ("gas7", dict()), ("gas40", dict()),
         ("gas700", dict()), ("gas40", dict(cell_target=60)), ("solid", dict()), ("solid", dict(cell_target=40)),
         ("solid-periodic", dict()), ("pillar", dict(cell_target=9)), ("pillar", dict(cell_target=12))]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("kind,over", CASES, ids=[k + "".join(f"-{a}{b}" for a, b in o.items()) for k, o in CASES])
def test_lists_at_the_limits_of_a_block(R, mp, kind, over, prec):
    s = _make(kind)
    q = dataclasses.replace(mp, **over)
    p = O.params_for(s, q)
    c = R.Context(q, R.RBC_FP64 if prec == "fp64" else R.RBC_MIXED)
    c.set_system(s)
    tol, pp = (FP64_TOL, PP_FP64_TOL) if prec == "fp64" else (MIXED_TOL, PP_MIXED_TOL)
    if over.get("cell_target") == 1:
        assert (c.debug_array(9) < 0).all()          # more own cells than a stage has bits for
    if kind == "pillar":
        assert c.stats()["max_cell_pairs"] > 256     # more than a row's scratch
    for steps in (0, 12):
        if steps:
            c.step(steps, 0.01)
        x, nrm = (to_np(a) for a in c.get_state()[:2])
        assert np.array_equal(c.get_pairs(), O.pairs(p, x, s.type))
        F, T = (to_np(a) for a in c.forces()[:2])
        F0, T0 = O.forces(p, s, x=x, nrm=nrm)[:2]
        check_forces(F, F0, tol, pp, f"{kind} F")
        check_forces(T, T0, tol, pp, f"{kind} tau")
    c.close()
