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


@pytest.mark.parametrize("waves", [1, 2])
@pytest.mark.parametrize("depth", [10, 3])
def test_persistent_launch_of_several_tiles(waves, depth):
    """beta2 <= beta1^2 bounds no step of Adam, so every instance takes the persistent
    launch: gradients, Adam and final energies against the oracle (n = 13 two groups of
    qubits at any depth, 17 three at depth 3), more instances than workgroups, with
    one-tile ones in the same queue and in the LDS-resident launch."""
    p, steps, adam = 3, 4, dict(beta1=0.6, beta2=0.3)
    graphs = [_graph(n, 20 + k) for k, n in enumerate([17, 13, 12, 16, 13, 7])]
    g0, b0 = (np.tile(a, (len(graphs), 1)) for a in qi.linear_ramp(p))
    opt = dict(steps=steps, workgroups=3, waves_per_simd=waves, max_group=depth, **adam)
    res, again = _run(graphs, p, g0, b0, **opt)
    mixed, _ = _run(graphs, p, g0, b0, resident_max_n=9, **opt)
    for a, b, c in zip(res, again, mixed):
        np.testing.assert_array_equal(a, b)
        np.testing.assert_allclose(a, c, rtol=0, atol=1e-12)
    for i, g in enumerate(graphs):
        _check(g, i, res, g0, b0, steps, **adam)


@pytest.mark.parametrize("resident", [0, 8])
def test_captured_queue_replays(resident):
    """One-tile instances: the captured graph (queue reset, persistent launch and, with
    resident_max_n, the LDS-resident one) replayed with other work and other start
    angles in between, against eager launches and the oracle."""
    import torch
    from paper_2407_13012_amd import QaoaBatch
    p, steps = 2, 3
    graphs = [_graph(n, 40 + k) for k, n in enumerate([12, 5, 9, 12, 2, 11, 8])]
    g0, b0 = (np.tile(a, (len(graphs), 1)) for a in qi.linear_ramp(p))
    opt = dict(steps=steps, workgroups=3, resident_max_n=resident)
    with QaoaBatch(graphs, p, use_graph=False, **opt) as b:
        eager, eager2 = b.run(g0, b0), b.run(g0 + 0.1, b0)
    with QaoaBatch(graphs, p, use_graph=True, **opt) as b:
        for _ in range(3):
            for start, want in ((g0, eager), (g0 + 0.1, eager2)):
                got = b.run(start, b0)
                torch.ones(1 << 20, device="cuda").sum().item()
                for x, y in zip(got, want):
                    np.testing.assert_array_equal(x, y)
    for i, g in enumerate(graphs):
        _check(g, i, eager, g0, b0, steps)
