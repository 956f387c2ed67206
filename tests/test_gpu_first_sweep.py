"""The last backward sweep, which makes layer 1's phi from the cost entries, and
the sweep before it, which leaves phi unwritten: two and three sweeps per layer,
one to three layers, folded and whole states, both forms of the rotation, phases
beyond the fast range, gradients from scratch and from a stored state."""
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


@pytest.mark.parametrize("prec,n,family", [("c128", 22, "maxcut"), ("c128", 21, "qubo"), ("c128", 25, "maxcut"),
                                           ("c64", 23, "maxcut"), ("c64", 22, "qubo"), ("c64", 26, "maxcut")])
@pytest.mark.parametrize("gamma,beta", [([0.4], [0.6]), ([0.4, 0.9], [1.2, 0.4]), ([0.3, 0.5, 0.8], [0.4, 1.3, -0.7]),
                                        ([2.0e5, 0.4], [0.3, 1.2])])
def test_gradient_through_the_first_layer(prec, n, family, gamma, beta):
    from paper_2407_13012_amd import QaoaHandle
    far = gamma[0] > 1e5
    if n > 24 and len(gamma) == 3 or far and (n > 22 or prec == "c64"):
        pytest.skip("covered at the smaller sizes")
    gamma, beta = np.array(gamma), np.array(beta)
    p = beta.size
    eps = 2.0 ** -53 if prec == "c128" else 2.0 ** -24
    if family == "maxcut":
        inst = qi.erdos_renyi(n, 0.3, seed=[17, n], weights="uniform", wlow=-1.0, whigh=1.0)
        wsum = float(np.abs(inst.weight_array()).sum())
    else:
        inst = qi.qubo_erdos_renyi(n, 0.2, seed=[17, n])
        wsum = float(np.abs(inst.J).sum() + np.abs(inst.h).sum())
    C = oracle.cost_of(inst)
    E0, dg0, db0 = oracle.gradient(n, C, gamma, beta)
    # rounding of p layers of n rotations and a phase, each a few ulps of a unit
    # vector, on sums bounded by sum |w|; far phase arguments are rounded once on
    # either side
    tol = (8 * p * (n + 4) + (4 * gamma[0] * wsum if far else 0)) * eps * wsum
    with QaoaHandle.from_instance(inst, prec) as q:
        for E, dg, db in (q.gradient(gamma, beta), (q.evaluate(gamma, beta), *q.gradient_from_state(gamma, beta)),
                          q.gradient(gamma, beta)):
            assert abs(E - E0) <= tol
            assert np.abs(dg - dg0).max() <= 2 * wsum * tol and np.abs(db - db0).max() <= 2 * n * tol
