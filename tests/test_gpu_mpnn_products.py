"""Edges of the warm-start network's products: output widths that are not whole
groups of 8 (p = 1, 3) and the widest (p = 16), batches whose node and graph
counts leave remainders in the row and K tiles (one node, one graph, 65 nodes, a
split's last slice).  test_gpu_mpnn.py pins the values against the oracle; here
a batch is compared with what its tiling must not change:

* a graph's prediction does not depend on the batch around it (rows of a product
  are independent and its K order is fixed): bitwise;
* the loss is the mean squared distance of the predictions from the targets, and
  the last bias gradient the sum of the errors: rounding of those sums;
* listing every graph twice halves every error (exactly, a power of two) and
  doubles the rows that are summed: the gradient changes only by the rounding of
  fp32 sums of at most 1040 terms, 1040 * 2^-24 = 6e-5 of the sum of their
  magnitudes; 1e-3 of a block's largest entry allows for cancellation among them.
"""
import numpy as np
import pytest

import qaoa_inputs as qi
from oracle import mpnn as om
from test_gpu_mpnn import block_check, model, targets

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")


@pytest.mark.parametrize("p,sizes", [(1, [2]), (3, [7]), (16, [64]), (3, [33, 32]), (8, [9] * 7 + [10]),
                                     (1, [13] * 40), (16, [20] * 25), (4, [257, 3, 260])])
def test_tile_edges(p, sizes):
    graphs = [qi.erdos_renyi(n, 0.5, seed=[21, p, k], weights="uniform", wlow=-1, whigh=1)
              for k, n in enumerate(sizes)]
    G = len(graphs)
    gt, bt = targets(graphs, p, seed=p)
    rng = np.random.default_rng(p)
    t32 = (qi.mpnn_init_params(p, 4) + rng.normal(0, 0.02, om.num_params(p))).astype(np.float32)
    m, _ = model(p, theta=t32)
    with m:
        g, b = m.predict(graphs)
        for i in {0, G // 2, G - 1}:
            gi, bi = m.predict([graphs[i]])
            assert np.array_equal(gi[0], g[i]) and np.array_equal(bi[0], b[i])
        L, grad = m.loss_grad(graphs, gt, bt)
        L1, _ = m.loss_grad(graphs, gt, bt, want_grad=False)
        L2, twice = m.loss_grad(graphs * 2, np.tile(gt, (2, 1)), np.tile(bt, (2, 1)))
    D = np.concatenate([g - gt, b - bt], axis=1)
    assert L == L1 and abs(L - np.mean(D * D)) <= 1e-12 * L and abs(L2 - L) <= 1e-12 * L
    dY = 2.0 * D / D.size
    assert np.all(np.abs(grad[-2 * p:] - dY.sum(0)) <= (G + 2) * 2.0 ** -24 * np.abs(dY).sum(0))
    block_check(twice.astype(np.float64), grad.astype(np.float64), p)
