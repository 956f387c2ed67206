"""The large-tile sweeps (n = 23 and 24, complex64 24 and 25: two sweeps per
layer) against the oracle: folded and whole states, both forms of the rotation on
either side of a layer boundary, one layer, and the reverse sweep from a stored
state; and the same size through the other tiles, which a cost of |gamma C|
beyond the fast range takes."""
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


@pytest.mark.parametrize("prec,n,family,beta", [
    ("c128", 23, "qubo", [1.2, 0.4]), ("c128", 23, "maxcut", [0.4, -1.2]), ("c128", 24, "maxcut", [0.4, 0.7]),
    ("c128", 24, "qubo", [1.3, -1.2]), ("c128", 23, "qubo", [0.6]),
    ("c64", 24, "qubo", [1.2, 0.4]), ("c64", 25, "maxcut", [0.4, -1.2]), ("c64", 25, "qubo", [0.4, 0.7]),
    ("c64", 24, "maxcut", [1.3, -1.2]), ("c64", 24, "qubo", [0.6])])
def test_large_tiles_match_oracle(prec, n, family, beta):
    from paper_2407_13012_amd import QaoaHandle
    beta = np.array(beta)
    p = beta.size
    eps = 2.0 ** -53 if prec == "c128" else 2.0 ** -24
    if family == "maxcut":
        inst = qi.erdos_renyi(n, 0.3, seed=[15, n], weights="uniform", wlow=-1.0, whigh=1.0)
        wsum = float(np.abs(inst.weight_array()).sum())
    else:
        inst = qi.qubo_erdos_renyi(n, 0.2, seed=[15, n])
        wsum = float(np.abs(inst.J).sum() + np.abs(inst.h).sum())
    gamma = np.linspace(0.2, 0.9, p)
    C = oracle.cost_of(inst)
    E0, dg0, db0 = oracle.gradient(n, C, gamma, beta)
    psi = oracle.state(n, C, gamma, beta)
    # rounding as for the smaller sizes: p layers of n rotations and a phase,
    # each a few ulps of a unit vector, on sums bounded by sum |w|
    tol = 8 * p * (n + 4) * eps * wsum
    with QaoaHandle.from_instance(inst, prec) as q:
        E, dg, db = q.gradient(gamma, beta)
        assert abs(E - E0) <= tol
        assert np.abs(dg - dg0).max() <= 2 * wsum * tol and np.abs(db - db0).max() <= 2 * n * tol
        assert abs(q.evaluate(gamma, beta) - E0) <= tol
        dg2, db2 = q.gradient_from_state(gamma, beta)
        assert np.abs(dg2 - dg0).max() <= 2 * wsum * tol and np.abs(db2 - db0).max() <= 2 * n * tol
        s = q.statevector(gamma, beta)
        assert np.abs(s - psi).max() <= 8 * p * (n + 4) * eps * np.abs(psi).max() * (1 + wsum)


def test_far_phases_take_the_other_tiles():
    """A layer with |gamma| sum |w| beyond 5e5 sends the call to the other tiles;
    the next call, without it, is back on the large ones."""
    from paper_2407_13012_amd import QaoaHandle
    n = 23
    inst = qi.qubo_erdos_renyi(n, 0.2, seed=[16, n])
    C = oracle.cost_of(inst)
    wsum = float(np.abs(inst.J).sum() + np.abs(inst.h).sum())
    gamma, beta = np.array([0.4, 2.0e5]), np.array([0.3, 1.2])
    E0, dg0, db0 = oracle.gradient(n, C, gamma, beta)
    # phase arguments up to 2e5 * wsum are rounded once on either side
    tol = (8 * 2 * (n + 4) + 4 * 2.0e5 * wsum) * 2.0 ** -53 * wsum
    with QaoaHandle.from_instance(inst) as q:
        E, dg, db = q.gradient(gamma, beta)
        assert abs(E - E0) <= tol and np.abs(db - db0).max() <= 2 * n * tol
        E1 = q.gradient(gamma[:1], beta[:1])[0]  # back on the large tiles
        assert abs(E1 - oracle.gradient(n, C, gamma[:1], beta[:1])[0]) <= tol
