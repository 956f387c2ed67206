"""The one-launch gradient of small states (at most 4096 stored amplitudes)
against the oracle: every size class of its kernel (one wave with idle
positions, one wave, 2 to 16 waves), folded (MaxCut, n >= 9) and whole states,
rotations in both ranges of beta (the flipped one exchanges z and ~z), one to 32
layers, and phases beyond the fast reduction's range."""
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


def _check(inst, prec, gamma, beta, wsum, arg_err=0.0):
    from paper_2407_13012_amd import QaoaHandle
    C = oracle.cost_of(inst)
    E0, dg0, db0 = oracle.gradient(inst.n, C, gamma, beta)
    with QaoaHandle.from_instance(inst, prec) as q:
        E, dg, db = q.gradient(gamma, beta)
        assert q.gradient_noalloc(gamma, beta)[0] == E
    # rounding: p layers of n rotations and a phase, each a few ulps of a unit
    # vector, on sums bounded by sum |w| (E, dgamma: its square at worst)
    p, n = len(gamma), inst.n
    eps = 2.0 ** -53 if prec == "c128" else 2.0 ** -24
    tol = (8 * p * (n + 4) * eps + p * arg_err) * max(1.0, wsum)
    assert abs(E - E0) <= tol, (E, E0, tol)
    assert np.abs(db - db0).max() <= 2 * n * tol
    assert np.abs(dg - dg0).max() <= 2 * max(1.0, wsum) * tol


def _inst(family, n, seed, scale=1.0):
    if family == "maxcut":
        g = qi.complete_graph(n, seed=seed, weights="uniform", wlow=-scale, whigh=scale)
        return g, float(np.abs(g.weight_array()).sum())
    q = qi.qubo_erdos_renyi(n, 0.5, seed=seed)
    q.J *= scale
    q.h *= scale
    return q, float(np.abs(q.J).sum() + np.abs(q.h).sum())


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("family,n", [("qubo", n) for n in (1, 2, 5, 6, 7, 8, 9, 10, 11, 12)] +
                         [("maxcut", n) for n in (2, 8, 9, 10, 11, 12, 13)])
@pytest.mark.parametrize("p", [1, 2, 3])
def test_small_gradient_matches_oracle(prec, family, n, p):
    inst, wsum = _inst(family, n, [9, n, p])
    rng = np.random.default_rng([9, n, p, 1])
    _check(inst, prec, rng.uniform(-1, 1, p), rng.uniform(-4, 4, p), wsum)


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_small_gradient_beta_at_quarter_turns(prec):
    """|cos| = |sin|, a pure flip, and no rotation at all."""
    for family, n in (("qubo", 11), ("maxcut", 12)):
        inst, wsum = _inst(family, n, [10, n])
        _check(inst, prec, np.array([0.3, 0.2, -0.4, 0.1]), np.pi / 4 * np.array([1.0, 2.0, 0.0, -3.0]), wsum)


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("p", [32, 33])
def test_small_gradient_layer_limit(prec, p):
    """32 layers in one launch; 33 take the sweeps."""
    from paper_2407_13012_amd import QaoaHandle
    inst, wsum = _inst("maxcut", 10, [11, p])
    gamma, beta = qi.ramp_with_noise(p, seed=[11, p])
    C = oracle.cost_of(inst)
    E0, dg0, db0 = oracle.gradient(inst.n, C, gamma, beta)
    eps = 2.0 ** -53 if prec == "c128" else 2.0 ** -24
    tol = 8 * p * (inst.n + 4) * eps * wsum
    with QaoaHandle.from_instance(inst, prec) as q:
        E, dg, db = q.gradient(gamma, beta)
    assert abs(E - E0) <= tol
    assert max(np.abs(dg - dg0).max(), np.abs(db - db0).max()) <= 2 * wsum * tol


def test_small_gradient_far_phases():
    """|gamma C| near 1e7: the oracle's arguments are rounded by 1e7 * 2^-53 each."""
    inst, wsum = _inst("qubo", 10, [12], scale=1e6)
    _check(inst, "c128", np.array([0.7, -1.1]), np.array([0.4, 1.9]), wsum, arg_err=4 * wsum * 2.0 ** -53)
