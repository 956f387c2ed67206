"""Shots found through the masses of runs of 16 amplitudes are those of the scan
of the whole sub-block: the same shots from calls on either side of the count
from which the run masses are kept, and the oracle's from the same state where
some targets fall within the rounding of a boundary (2^24 masses, 10^6 shots)."""
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


def _instance(n, family):
    return (qi.qubo_erdos_renyi(n, 0.2, seed=[18, n]) if family == "qubo"
            else qi.erdos_renyi(n, 0.2, seed=[18, n], weights="uniform", wlow=-1.0, whigh=1.0))


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n,family", [(26, "qubo"), (27, "er"), (28, "er"), (29, "er")])
def test_same_shots_with_and_without_run_masses(prec, n, family):
    from paper_2407_13012_amd import QaoaHandle
    gamma, beta = qi.uniform_angles(2, seed=[18, n, 1])
    least = (1 << (n - (family == "er"))) >> 10  # shots from which the masses are kept (n <= 28)
    with QaoaHandle.from_instance(_instance(n, family), prec) as q:
        q.statevector(gamma, beta, copy=False)
        z0, c0 = q.sample(least - 1, 5)
        z1, c1 = q.sample(least, 5)
        z2, c2 = q.sample(1000, 5)
    assert np.array_equal(z0, z1[:-1]) and np.array_equal(c0, c1[:-1])
    assert np.array_equal(z2, z1[:1000]) and np.array_equal(c2, c1[:1000])


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n,family", [(8, "qubo"), (13, "er"), (20, "qubo"), (23, "er")])
def test_same_shots_from_either_share_of_a_wave(prec, n, family):
    from paper_2407_13012_amd import QaoaHandle
    gamma, beta = qi.uniform_angles(2, seed=[18, n, 1])
    C = oracle.cost_of(_instance(n, family))
    with QaoaHandle.from_instance(_instance(n, family), prec) as q:
        psi = q.statevector(gamma, beta).astype(np.complex128)
        for shots in (1, 9, 1 << 14, (1 << 14) + 1):
            z, c = q.sample(shots, 5)
            z_ref, _ = oracle.sample(n, psi, C, shots, seed=5)
            assert np.array_equal(z, z_ref)
            assert np.array_equal(c, C[z] if prec == "c128" else C.astype(np.float32)[z].astype(np.float64))


def test_shots_at_the_rounding_of_a_boundary():
    from paper_2407_13012_amd import QaoaHandle
    n, shots = 24, 1_000_000
    inst = qi.erdos_renyi(n, 0.3, seed=[19, n], weights="uniform", wlow=-1.0, whigh=1.0)
    gamma, beta = qi.uniform_angles(1, seed=[19, n, 1])
    C = oracle.cost_of(inst)
    with QaoaHandle.from_instance(inst) as q:
        psi = q.statevector(gamma, beta)
        z, c = q.sample(shots, 11)
    z_ref, c_ref = oracle.sample(n, psi, C, shots, seed=11)
    assert np.array_equal(z, z_ref) and np.array_equal(c, c_ref)


def test_shots_without_room_for_the_run_masses():
    import torch
    from paper_2407_13012_amd import QaoaHandle, _binding
    n, limit, refused = 20, [None], []

    def alloc(nbytes, stream, _user):
        if limit[0] is not None and nbytes > limit[0]:
            refused.append(int(nbytes))
            return None
        return torch.cuda.caching_allocator_alloc(int(nbytes), torch.cuda.current_device(), int(stream or 0))

    def free(ptr, _nbytes, _stream, _user):
        torch.cuda.caching_allocator_delete(int(ptr))

    own = _binding.Allocator(_binding.ALLOC_FN(alloc), _binding.FREE_FN(free), None)
    gamma, beta = qi.uniform_angles(2, seed=[20, n, 1])
    inst = _instance(n, "qubo")
    with QaoaHandle.from_instance(inst) as q:
        q.statevector(gamma, beta, copy=False)
        z_ref, c_ref = q.sample(100, 5)
    _binding.qaoa_set_allocator(own)
    try:
        q = QaoaHandle.from_instance(inst)
    finally:
        _binding.qaoa_set_allocator(None)
    with q:
        q.statevector(gamma, beta, copy=False)
        limit[0] = 400 << 10  # the run masses take 512 KiB, everything else 70
        z, c = q.sample(100, 5)
        E = q.evaluate(gamma, beta)
    assert len(refused) == 1 and np.isfinite(E)
    assert np.array_equal(z, z_ref) and np.array_equal(c, c_ref)
