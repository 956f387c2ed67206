"""Exports of folded MaxCut states and their cost diagonals to pageable and pinned
host memory (the latter written by a kernel, also from the middle of an
allocation): the entries of the export to device memory."""
import numpy as np
import pytest

import qaoa_inputs as qi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n", [13, 14, 17, 20])  # 13: folded in complex128 only
def test_host_exports_equal_device_exports(n, prec):
    import torch
    from paper_2407_13012_amd import QaoaHandle
    N, kind = 1 << n, torch.complex128 if prec == "c128" else torch.complex64
    gamma, beta = qi.uniform_angles(2, seed=[21, n])
    with QaoaHandle.from_instance(qi.erdos_renyi(n, 0.3, seed=[21, n], weights="uniform", wlow=-1.0, whigh=1.0), prec) as q:
        dev = q.statevector(gamma, beta, out=torch.zeros(N, dtype=kind, device="cuda")).cpu().numpy()
        cost = q.cost_diagonal(torch.zeros(N, dtype=torch.float64, device="cuda")).cpu().numpy()
        assert np.abs(dev).max() > 0 and np.ptp(cost) > 0
        pinned = torch.zeros(N + 3, dtype=kind, pin_memory=True).numpy()
        pinned_cost = torch.zeros(N + 1, dtype=torch.float64, pin_memory=True).numpy()
        assert np.array_equal(q.statevector(gamma, beta), dev)
        assert np.array_equal(q.cost_diagonal(), cost)
        for at in (0, 3):
            assert np.array_equal(q.statevector(gamma, beta, out=pinned[at:at + N]), dev)
        for at in (0, 1):
            assert np.array_equal(q.cost_diagonal(pinned_cost[at:at + N]), cost)
