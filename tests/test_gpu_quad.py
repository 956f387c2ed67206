"""The small-tile sweeps (states above 4096 amplitudes up to 16 MiB) against the
oracle: each tile size (10, 11, 12 bits) at its smallest and largest n, folded
and whole, both forms of every rotation on either side of a layer boundary, and
the reverse sweep from a stored state; and the same state through the large
tiles, which a cost of |gamma C| beyond the fast range takes."""
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


# beta in the tan range (a), the cot range (b): every pair at a layer boundary
BETAS = {"tan": [0.3, -0.5, 0.7], "mixed": [1.2, 0.4, -1.1, 1.9], "cot": [1.3, -1.2, 2.0], "one": [0.6]}


@pytest.mark.parametrize("prec,sizes", [("c128", (13, 14, 18, 19, 20, 21)), ("c64", (13, 14, 17, 18, 19, 21))])
@pytest.mark.parametrize("family", ["qubo", "maxcut"])
@pytest.mark.parametrize("form", list(BETAS))
def test_small_tiles_match_oracle(prec, sizes, family, form):
    from paper_2407_13012_amd import QaoaHandle
    beta = np.array(BETAS[form])
    p = beta.size
    eps = 2.0 ** -53 if prec == "c128" else 2.0 ** -24
    for n in sizes:
        if form != "mixed" and n > 19:
            continue  # one oracle run per large size
        if family == "maxcut":
            inst = qi.erdos_renyi(n, 0.3, seed=[13, n], weights="uniform", wlow=-1.0, whigh=1.0)
            wsum = float(np.abs(inst.weight_array()).sum())
        else:
            inst = qi.qubo_erdos_renyi(n, 0.2, seed=[13, n])
            wsum = float(np.abs(inst.J).sum() + np.abs(inst.h).sum())
        gamma = np.linspace(0.2, 0.9, p)
        C = oracle.cost_of(inst)
        E0, dg0, db0 = oracle.gradient(n, C, gamma, beta)
        psi = oracle.state(n, C, gamma, beta)
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


def test_far_phases_take_the_large_tiles():
    """A layer with |gamma| sum |w| beyond 5e5 sends the call to the large tiles;
    the next call, without it, is back on the small ones."""
    from paper_2407_13012_amd import QaoaHandle
    n = 15
    inst = qi.qubo_erdos_renyi(n, 0.3, seed=[14, n])
    C = oracle.cost_of(inst)
    wsum = float(np.abs(inst.J).sum() + np.abs(inst.h).sum())
    gamma, beta = np.array([0.4, 2.0e5]), np.array([0.3, 1.2])
    E0, dg0, db0 = oracle.gradient(n, C, gamma, beta)
    # phase arguments up to 2e5 * wsum are rounded once on either side
    tol = (8 * 2 * (n + 4) + 4 * 2.0e5 * wsum) * 2.0 ** -53 * wsum
    with QaoaHandle.from_instance(inst) as q:
        E, dg, db = q.gradient(gamma, beta)
        assert abs(E - E0) <= tol and np.abs(db - db0).max() <= 2 * n * tol
        E1 = q.gradient(gamma[:1], beta[:1])[0]  # back on the small tiles
        assert abs(E1 - oracle.gradient(n, C, gamma[:1], beta[:1])[0]) <= tol
