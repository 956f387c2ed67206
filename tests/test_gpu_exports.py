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
        dev, cost = torch.zeros(N, dtype=kind, device="cuda"), torch.zeros(N, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()  # the handle has a stream of its own
        q.statevector(gamma, beta, out=dev)
        q.cost_diagonal(cost)
        torch.cuda.synchronize()
        dev, cost = dev.cpu().numpy(), cost.cpu().numpy()
        assert np.abs(dev).max() > 0 and np.ptp(cost) > 0
        pinned = torch.zeros(N + 3, dtype=kind, pin_memory=True).numpy()
        pinned_cost = torch.zeros(N + 1, dtype=torch.float64, pin_memory=True).numpy()
        assert np.array_equal(q.statevector(gamma, beta), dev)
        assert np.array_equal(q.cost_diagonal(), cost)
        for at in (0, 3):
            assert np.array_equal(q.statevector(gamma, beta, out=pinned[at:at + N]), dev)
        for at in (0, 1):
            assert np.array_equal(q.cost_diagonal(pinned_cost[at:at + N]), cost)


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_device_export_to_memory_that_kernels_do_not_write(prec):
    """Managed memory takes the route of another device's: copies, with the half
    turned round in place between them and back after (the state stays usable)."""
    import ctypes
    import torch
    from paper_2407_13012_amd import QaoaHandle, load_library
    lib, n = load_library(), 15
    N, kind = 1 << n, torch.complex128 if prec == "c128" else torch.complex64
    gamma, beta = qi.uniform_angles(2, seed=[22, n])
    ptr = ctypes.c_void_p()
    assert lib.hipMallocManaged(ctypes.byref(ptr), ctypes.c_size_t(16 * N), ctypes.c_uint(1)) == 0
    try:
        with QaoaHandle.from_instance(qi.erdos_renyi(n, 0.3, seed=[22, n]), prec) as q:
            dev = q.statevector(gamma, beta)
            E = q.expectation()
            a = [np.ascontiguousarray(x, dtype=np.float64) for x in (gamma, beta)]
            assert lib.qaoa_statevector(q.raw, 2, *(ctypes.c_void_p(x.ctypes.data) for x in a), ptr, 1) == 0
            torch.cuda.synchronize()
            got = np.frombuffer((ctypes.c_char * (N * dev.itemsize)).from_address(ptr.value), dtype=dev.dtype)
            assert np.array_equal(got, dev)
            assert q.expectation() == E
    finally:
        torch.cuda.synchronize()
        assert lib.hipFree(ptr) == 0


def test_device_export_in_a_captured_graph():
    import torch
    from paper_2407_13012_amd import QaoaHandle
    n = 14
    gamma, beta = qi.uniform_angles(2, seed=[23, n])
    s = torch.cuda.Stream()
    with QaoaHandle.maxcut(n, qi.erdos_renyi(n, 0.3, seed=[23, n]).edges, stream=s) as q:
        out = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
        torch.cuda.synchronize()
        want = q.statevector(gamma, beta)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            q.statevector(gamma, beta, out=out)
        for _ in range(3):
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want)
            out.zero_()
            torch.cuda.synchronize()
            q.gradient(gamma, beta)
