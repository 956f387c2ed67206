"""The cost diagonal at the edges of its kernel's term chunks (64 terms to a
wavefront's test, 256 to a read) and of its 4096-entry tiles: every entry is
the ordered sum of its active terms, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")


@pytest.mark.parametrize("n", [1, 5, 10, 13, 15])
@pytest.mark.parametrize("terms", [0, 1, 63, 64, 65, 128, 255, 256, 257, 600])
def test_terms_are_summed_in_order(n, terms):
    from paper_2407_13012_amd import QaoaHandle
    rng = np.random.default_rng([n, terms])
    masks = (rng.integers(0, 1 << n, terms) & rng.integers(0, 1 << n, terms)).astype(np.uint64)
    w = rng.standard_normal(terms) * 10.0 ** rng.integers(-8, 8, terms)
    offset = 0.25
    z = np.arange(1 << n, dtype=np.uint64)
    ref = np.full(1 << n, offset)
    for m, x in zip(masks, w):
        ref[(z & m) == m] += x
    with QaoaHandle.poly(n, masks, w, offset) as q:
        assert np.array_equal(q.cost_diagonal(), ref)


@pytest.mark.parametrize("n", [5, 14])
@pytest.mark.parametrize("m", [32, 33, 128, 129, 300])
def test_edges_are_summed_in_order(n, m):
    from paper_2407_13012_amd import QaoaHandle
    rng = np.random.default_rng([n, m, 7])
    i = rng.integers(0, n, m)
    e = np.stack([i, (i + rng.integers(1, n, m)) % n], axis=1).astype(np.int32)
    w = rng.standard_normal(m) * 10.0 ** rng.integers(-8, 8, m)
    z = np.arange(1 << n)
    ref = np.zeros(1 << n)
    for (a, b), x in zip(e, w):
        ref[((z >> a) ^ (z >> b)) & 1 == 1] += x
    with QaoaHandle.maxcut(n, e, w) as q:
        assert np.array_equal(q.cost_diagonal(), ref)
