"""Instances of more than one tile (n > 12) run by size class, all of one size
in lockstep: chunks of a class, angles outside the reduced range, and runs whose
phases leave the fast range (those instances go to the persistent launch)."""
import numpy as np
import pytest

import oracle
import qaoa_inputs as qi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")


def _graphs(sizes, seed, scale=1.0):
    return [qi.erdos_renyi(n, 0.5, seed=[seed, k], weights="uniform", wlow=-scale, whigh=scale)
            for k, n in enumerate(sizes)]


def _run(graphs, p, g0, b0, **opt):
    from paper_2407_13012_amd import QaoaBatch
    with QaoaBatch(graphs, p, **opt) as b:
        return b.run(g0, b0), b.run(g0, b0)


def _check(graphs, g0, b0, res, steps, atol):
    gam, bet, e0, e1 = res
    for i, g in enumerate(graphs):
        w = float(np.abs(g.weight_array()).sum())
        og, ob, oe0, oe1 = oracle.adam_qaoa(g.n, oracle.cost_of(g), g0[i], b0[i], steps, scale=1.0 / w)
        assert abs(e0[i] - oe0) <= 1e-10 * max(1.0, w), (i, g.n)
        np.testing.assert_allclose(np.r_[gam[i], bet[i]], np.r_[og, ob], rtol=0, atol=atol)
        assert abs(e1[i] - oe1) <= atol * max(1.0, w), (i, g.n)


@pytest.mark.parametrize("p,steps", [(1, 2), (2, 0), (3, 3)])
def test_chunks_do_not_change_results(p, steps):
    """One workgroup's memory holds one instance of each size at a time, so every
    class runs in chunks; with memory for all of them each class is one chunk.
    n = 13 and 14 (one and two tiles), 17 (a spectator class), angles in [-4, 4]."""
    graphs = _graphs([13, 14, 13, 17, 9, 14, 13, 16], seed=5)
    rng = np.random.default_rng([5, p])
    g0, b0 = rng.uniform(-4, 4, (len(graphs), p)), rng.uniform(-4, 4, (len(graphs), p))
    one, again = _run(graphs, p, g0, b0, steps=steps, workgroups=1)
    many, _ = _run(graphs, p, g0, b0, steps=steps)
    for a, b, c in zip(one, again, many):
        np.testing.assert_array_equal(a, b)
        np.testing.assert_array_equal(a, c)
    # tolerances of the engine's other oracle comparisons
    _check(graphs, g0, b0, many, steps, 1e-8)


def test_far_phases_take_the_persistent_launch():
    """Weights near 1e6: |gamma C| may pass the fast reduction's bound, so the
    whole batch runs one workgroup per instance.  The start energy then carries
    the rounding of arguments near 1e8 (1e8 * 2^-53 per phase)."""
    graphs = _graphs([13, 15, 11], seed=6, scale=1e6)
    p = 2
    g0, b0 = np.tile(qi.linear_ramp(p)[0], (3, 1)), np.tile(qi.linear_ramp(p)[1], (3, 1))
    (gam, bet, e0, e1), _ = _run(graphs, p, g0, b0, steps=1)
    for i, g in enumerate(graphs):
        C = oracle.cost_of(g)
        E = oracle.expectation(g.n, C, oracle.state(g.n, C, g0[i], b0[i]))
        assert abs(e0[i] - E) <= 1e-7 * float(np.abs(g.weight_array()).sum())
    assert np.all(np.isfinite(gam)) and np.all(np.isfinite(e1))


def test_small_tiles_of_a_class():
    """A class on small tiles (three instances of n = 14) and, with a depth that
    their second pass exceeds or beside a class that fills the card, on the large
    ones: the same results to rounding, and the oracle's."""
    graphs = _graphs([14, 14, 18, 14], seed=7)
    p, steps = 3, 3
    g0, b0 = np.tile(qi.linear_ramp(p)[0], (4, 1)), np.tile(qi.linear_ramp(p)[1], (4, 1))
    small, _ = _run(graphs, p, g0, b0, steps=steps)
    large, _ = _run(graphs, p, g0, b0, steps=steps, group_by_n={14: 3, 18: 6})
    big = _graphs([20, 20, 20], seed=8)
    beside, _ = _run(graphs + big, p, np.tile(g0[0], (7, 1)), np.tile(b0[0], (7, 1)), steps=steps)
    for a, b, c in zip(small, large, beside):
        np.testing.assert_allclose(a, b, rtol=0, atol=1e-9)
        np.testing.assert_allclose(a, c[:4], rtol=0, atol=1e-9)
    _check(graphs, g0, b0, small, steps, 1e-8)
