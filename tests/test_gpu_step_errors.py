"""Lists that overflow in the middle of a step call and fit again before it ends.

Where pairs are lost the call reports it: two clusters without forces (eps = 0) pass through
each other, each with 59 partners within the cutoff.  Where the nearest partners fit, none is.
"""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from paper_1701_02059_amd import inputs as I
from tests.gpu_common import gpu_available, to_np

pytestmark = pytest.mark.gpu

DT, V, X0 = 0.01, 3.0, 6.0            # the clusters meet after 200 steps


@pytest.fixture(scope="module")
def R():
    if not gpu_available():
        pytest.skip("needs a GPU")
    from paper_1701_02059_amd import rbc
    rbc.lib()
    return rbc


def _passing(filler=0):
    """Two clusters of 60 lipids on course for each other, and a resting sheet far below."""
    rng = np.random.default_rng(3)
    ball = rng.normal(size=(120, 3))
    ball *= 0.9 * rng.random((120, 1)) ** (1 / 3) / np.linalg.norm(ball, axis=1)[:, None]
    side = np.repeat([-1.0, 1.0], 60)
    x = ball + np.outer(side, [X0, 0.0, 0.0])
    v = np.outer(-V * side, [1.0, 0.0, 0.0])
    if filler:
        m = int(np.ceil(np.sqrt(filler)))
        g = np.stack(np.meshgrid(np.arange(m), np.arange(m), [0.0], indexing="ij"), axis=-1).reshape(-1, 3)
        x, v = np.r_[x, g * 1.1 - [0.0, 0.0, 50.0]], np.r_[v, np.zeros(g.shape)]
    nrm = np.tile([0.0, 0.0, 1.0], (len(x), 1))
    return I.System("passing", x, nrm, np.zeros(len(x), np.int32), v, np.zeros(x.shape), np.zeros((0, 2), np.int32),
                    np.zeros(0), np.zeros(3), np.zeros(3, np.int32))


@pytest.mark.parametrize("graphs", [False, True])
@pytest.mark.parametrize("filler", [0, 1 << 20], ids=["small", "waiting-statistics"])
def test_an_overflow_between_good_builds_is_reported(R, mp, filler, graphs):
    c = R.Context(dataclasses.replace(mp, eps=0.0), R.RBC_MIXED)
    c.set_graphs(graphs)
    s = _passing(filler)
    c.set_system(s)
    c.step(100, DT)                                  # before they meet
    with pytest.raises(R.RbcError) as ei:
        c.step(220, DT)                              # through each other
    assert ei.value.status == R.RBC_ERR_CAPACITY
    c.sync()                                         # the lists of the call's last build fit
    c.step(20, DT)                                   # and so do the next call's
    x = to_np(c.get_state()[0])
    assert np.abs(x - (s.x + 340 * DT * s.v)).max() < 1e-9
    c.close()


def test_a_slot_that_overflowed_between_good_builds_is_frozen(R, mp):
    q = dataclasses.replace(mp, eps=0.0)
    quiet = I.config("tiny")
    e = R.Ensemble(q, R.RBC_MIXED, max_slots=2)
    bad, good = e.admit(_passing()), e.admit(quiet)
    e.step(100, DT)
    with pytest.raises(R.RbcError) as ei:
        e.step(220, DT)
    assert ei.value.status == R.RBC_ERR_CAPACITY
    assert e.failed() == {bad: R.RBC_ERR_CAPACITY}
    got = [to_np(t) for t in e.get_state(good)]
    e.close()
    ref = R.Ensemble(q, R.RBC_MIXED, max_slots=1)
    k = ref.admit(quiet)
    ref.step(100, DT)
    ref.step(220, DT)
    for a, b in zip(got, ref.get_state(k)):
        assert np.array_equal(a, to_np(b))
    ref.close()


def _crossing(filler=0):
    """Two layers of lipids crossing a block of them in its lattice's gaps: up to 112 partners
    within rc + 2 skin while they overlap, 88 within rc + 1.2 skin."""
    rng = np.random.default_rng(4)
    a = 1.25
    g = np.stack(np.meshgrid(*[np.arange(5)] * 3, indexing="ij"), axis=-1).reshape(-1, 3) * a
    b = np.stack(np.meshgrid(np.arange(2), np.arange(4), np.arange(4), indexing="ij"), axis=-1).reshape(-1, 3) * a
    x = np.r_[g, b + [-4.5 - a, 0.5 * a, 0.5 * a]]
    x += rng.normal(0, 0.01, x.shape)
    v = np.r_[np.zeros(g.shape), np.tile([V, 0.0, 0.0], (len(b), 1))]
    if filler:
        m = int(np.ceil(np.sqrt(filler)))
        f = np.stack(np.meshgrid(np.arange(m), np.arange(m), [0.0], indexing="ij"), axis=-1).reshape(-1, 3)
        x, v = np.r_[x, f * 1.1 - [0.0, 0.0, 50.0]], np.r_[v, np.zeros(f.shape)]
    nrm = rng.normal(size=x.shape)
    nrm /= np.linalg.norm(nrm, axis=1)[:, None]
    return I.System("crossing", x, nrm, np.zeros(len(x), np.int32), v, np.zeros(x.shape), np.zeros((0, 2), np.int32),
                    np.zeros(0), np.zeros(3), np.zeros(3, np.int32))


@pytest.mark.parametrize("target", [16, 300], ids=["staged", "wide"])
@pytest.mark.parametrize("filler", [0, 1 << 20], ids=["small", "waiting-statistics"])
def test_lists_that_overflow_in_passing_lose_no_pair(R, mp, filler, target):
    """A build that a particle overflows keeps its nearest partners, and the next one comes before
    any other can be in range: the trajectory is the oracle's, and the call succeeds."""
    q = dataclasses.replace(mp, eps=0.01, cell_target=target)
    s = _crossing(filler)
    small = _crossing()
    n = small.N
    p = O.params_for(small, q)
    c = R.Context(q, R.RBC_FP64)
    c.set_system(s)
    worst = 0
    for steps in (120, 60, 60, 60, 60, 150):
        try:
            c.step(steps, DT)
        except R.RbcError as e:                      # the call's last lists do not fit: reported as ever
            assert e.status == R.RBC_ERR_CAPACITY
            worst += 1
    x, nrm, v, w = (to_np(t)[:n] for t in c.get_state())
    ref = O.vv_run(p, small, DT, 510)
    assert np.abs(x - ref[0]).max() < 1e-9 and np.abs(nrm - ref[2]).max() < 1e-9
    assert 0 < worst < 6
    c.close()
    c = R.Context(q, R.RBC_FP64)
    c.set_system(s)
    c.step(510, DT)                                  # in one call: the last builds fit
    assert np.abs(to_np(c.get_state()[0])[:n] - ref[0]).max() < 1e-9
    c.close()
