"""Batches of which some sizes, by the phases that a run could reach, take the
persistent launch, whose workgroups run instances of several tiles in whole slots."""
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


def _graph(n, seed, scale=1.0):
    return qi.erdos_renyi(n, 0.5, seed=[seed, n], weights="uniform", wlow=-scale, whigh=scale)


def _run(graphs, p, g0, b0, **opt):
    from paper_2407_13012_amd import QaoaBatch
    with QaoaBatch(graphs, p, **opt) as b:
        return b.run(g0, b0), b.run(g0, b0)


def _check(g, i, res, g0, b0, steps, **adam):
    # the tolerances of the engine's other oracle comparisons
    gam, bet, e0, e1 = res
    w = float(np.abs(g.weight_array()).sum())
    og, ob, oe0, oe1 = oracle.adam_qaoa(g.n, oracle.cost_of(g), g0[i], b0[i], steps, scale=1.0 / w, **adam)
    assert abs(e0[i] - oe0) <= 1e-10 * max(1.0, w), (i, g.n)
    np.testing.assert_allclose(np.r_[gam[i], bet[i]], np.r_[og, ob], rtol=0, atol=1e-8, err_msg=f"n={g.n}")
    assert abs(e1[i] - oe1) <= 1e-8 * max(1.0, w), (i, g.n)


def test_far_sizes_beside_near_ones():
    """n = 15 has weights near 1e6, whose start energy carries the rounding of
    arguments near 1e8 (1e8 * 2^-53 per phase); the other sizes are unaffected."""
    p, steps = 2, 3
    graphs = [_graph(14, 1), _graph(15, 2, scale=1e6), _graph(16, 3), _graph(9, 4), _graph(15, 5), _graph(14, 6)]
    g0, b0 = (np.tile(a, (len(graphs), 1)) for a in qi.linear_ramp(p))
    res, again = _run(graphs, p, g0, b0, steps=steps, workgroups=2)
    for a, b in zip(res, again):
        np.testing.assert_array_equal(a, b)
    for i, g in enumerate(graphs):
        if i != 1:
            _check(g, i, res, g0, b0, steps)
    C = oracle.cost_of(graphs[1])
    E = oracle.expectation(15, C, oracle.state(15, C, g0[1], b0[1]))
    assert abs(res[2][1] - E) <= 1e-7 * float(np.abs(graphs[1].weight_array()).sum())
    assert all(np.all(np.isfinite(x)) for x in res)
