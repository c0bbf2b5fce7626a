"""List padding on fully periodic boxes: the padding entry's coordinates, wrapped, may be a
particle's own position, and its rows must still add nothing.

A particle at the origin of a cubic box whose length divides 1e8 meets it at separation zero.
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


def _system(L, kind):
    """A cloud with long lists, and the particle at the origin with three partners."""
    rng = np.random.default_rng(17)
    g = np.arange(7) * 1.4 + 0.5 * (L - 6 * 1.4)
    x = np.stack(np.meshgrid(g, g, g, indexing="ij"), axis=-1).reshape(-1, 3)
    x += rng.normal(0, 0.05, x.shape)
    near = np.array([[0.0, 0.0, 0.0], [1.2, 0.1, 0.0], [-0.1, 1.3, 0.2], [0.1, 0.0, 1.25]])
    x = np.mod(np.r_[near, x], L)
    typ = np.zeros(len(x), np.int32)
    typ[0] = kind
    nrm = rng.normal(size=x.shape)
    nrm /= np.linalg.norm(nrm, axis=1, keepdims=True)
    nrm[typ > 0] = 0.0
    assert (x[0] == 0.0).all() and 1e8 % L == 0.0
    z = np.zeros(x.shape)
    return I.System("cloud", x, nrm, typ, z, z.copy(), np.zeros((0, 2), np.int32), np.zeros(0), np.full(3, float(L)),
                    np.ones(3, np.int32))


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("theta", [0.0, 0.1], ids=["default-constants", "general-constants"])
@pytest.mark.parametrize("L,kind", [(20, 0), (50, 0), (20, 1)])
def test_padding_adds_nothing_at_the_origin(R, mp, L, kind, theta, prec):
    s = _system(L, kind)
    q = dataclasses.replace(mp, sin_theta0=theta)
    p = O.params_for(s, q)
    F0, T0, U0, W0 = O.forces(p, s)
    c = R.Context(q, R.RBC_FP64 if prec == "fp64" else R.RBC_MIXED)
    c.set_system(s)
    tol, pp = (FP64_TOL, PP_FP64_TOL) if prec == "fp64" else (MIXED_TOL, PP_MIXED_TOL)
    for energy in (False, True):
        F, T = (to_np(t) for t in c.forces(energy=energy)[:2])
        check_forces(F, F0, tol, pp, "F")
        check_forces(T, T0, tol, pp, "tau")
    E = to_np(c.forces(energy=True)[2])
    assert E[0] == pytest.approx(U0, rel=tol) and np.isfinite(E[1])
    c.step(2, 1e-3)
    assert all(np.isfinite(to_np(t)).all() for t in c.get_state())
    c.close()
