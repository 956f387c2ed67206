"""The byte counts and loads that bench.py reports for folded states and for
batches whose larger instances run by size."""
import numpy as np

import bench


def test_stored_amplitudes():
    # more than one tile (2^12 complex128, 2^13 complex64 amplitudes): half
    assert [bench.stored_amplitudes(n) for n in (12, 13, 26)] == [2.0 ** 12, 2.0 ** 12, 2.0 ** 25]
    assert [bench.stored_amplitudes(n, 8) for n in (13, 14)] == [2.0 ** 13, 2.0 ** 13]


def test_batch_step_bytes():
    # one tile: as the byte model; LDS-resident: 2p - 1 reads of the cost entries
    assert bench.batch_step_bytes(12, 4) == bench.batch_bytes_per_amp(12, 4) * 4096
    assert bench.batch_step_bytes(12, 4, resident_max_n=12) == 8 * 7 * 4096
    # folded, two groups, p = 4: forward 24 + 3 x 40, the turn 40, backward 2 x 72 + 56
    # (phi not stored) + 24 (lam and C read)
    assert bench.batch_step_bytes(20, 4) == (24 + 3 * 40 + 40 + 2 * 72 + 56 + 24) * 2 ** 19
    # p = 1: first sweep 24, the turn 40, the last sweep 24
    assert bench.batch_step_bytes(13, 1) == (24 + 40 + 24) * 2 ** 12
    # three groups, p = 1: 24 + 32, the turn 40, 48 without phi's store, 24
    assert bench.batch_step_bytes(20, 1, 4) == (24 + 32 + 40 + 48 + 24) * 2 ** 19


def test_launch_loads():
    """Two workgroups that take three one-tile instances, all busy to the end, beside
    three instances of one size that start and end together."""
    ns = np.array([14, 14, 14, 10, 9, 8, 5])
    which = np.array([0, 0, 0, 0, 0, 0, 1])
    t0 = np.array([0.0, 0.0, 0.0, 0.0, 0.0, 1.0, 2.0])
    t1 = np.array([3.0, 3.0, 3.0, 1.0, 2.0, 2.0, 4.0])
    out = bench.launch_loads(ns, which, t0, t1, 2, 256)
    assert out["size_classes"] == {"instances": 3, "span_s": 3.0, "first_start_s": 0.0}
    assert out["streamed"]["busy_fraction"] == 1.0 and out["streamed"]["workgroups"] == 2
    assert out["resident"]["busy_fraction"] == 1.0 and out["resident"]["workgroups"] == 1
    assert out["largest_n"] == {"n": 14, "mean_s": 3.0, "last_end_s": 3.0}
