"""Sampling kernels (8 or 32 shots per wave, sub-block masses of a folded state
taken in pairs): identical shots and objective values to the oracle's, at the
shot counts around a wave's share and the change of variant, and at states
smaller than a sub-block, of one, and of many."""
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


@pytest.mark.parametrize("n,family", [(2, "qubo"), (5, "qubo"), (8, "er"), (9, "qubo"), (13, "er"), (18, "er")])
@pytest.mark.parametrize("shots", [1, 7, 9, 33, 65536, 65537])
def test_shots_identical_to_oracle(n, family, shots):
    from paper_2407_13012_amd import QaoaHandle
    inst = (qi.qubo_erdos_renyi(n, 0.5, seed=[8, n]) if family == "qubo"
            else qi.erdos_renyi(n, 0.5, seed=[8, n], weights="uniform", wlow=-1.0, whigh=1.0))
    gamma, beta = qi.uniform_angles(2, seed=[8, n, 1])
    C = oracle.cost_of(inst)
    z_ref, c_ref = oracle.sample(n, oracle.state(n, C, gamma, beta), C, shots, seed=77)
    with QaoaHandle.from_instance(inst) as q:
        q.statevector(gamma, beta, copy=False)
        z, c = q.sample(shots, 77)
    assert np.array_equal(z, z_ref) and np.array_equal(c, c_ref)


def test_shots_of_a_single_basis_state():
    """All mass on one state, in the middle of a sub-block with zeros around it:
    gamma = pi/2 on sum x_i, beta = pi/4 gives |1...1> up to phases; rounding
    leaves the others below 1e-30."""
    from paper_2407_13012_amd import QaoaHandle
    n = 10
    with QaoaHandle.qubo(n, np.zeros((0, 2), np.int32), [], h=np.ones(n)) as q:
        q.statevector([np.pi / 2], [np.pi / 4], copy=False)
        for shots in (100, 70000):
            z, _ = q.sample(shots, 3)
            assert z.min() == z.max() and z[0] in (0, (1 << n) - 1)
