"""Merging of a leaf's candidates into the neighbour lists (random projection
trees), bit for bit against the oracle (needs an MI355X): list lengths at both
ends, leaves that end inside a batch of 64 candidates, and points on a coarse
grid, where most distances tie and the order is that of the ids."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,kappa,leaf,rounds,grid", [
    (1500, 4, 64, 200, 3, 0), (1300, 4, 1, 65, 3, 0), (1024, 3, 63, 128, 2, 0), (900, 2, 64, 300, 3, 8), (700, 3, 17, 64, 4, 3)])
def test_lists_bit_exact(N, d, kappa, leaf, rounds, grid):
    import torch
    from paper_1410_0260_amd import askit as A
    print(f"\n[rpknn lists] N={N} d={d} kappa={kappa} leaf={leaf} rounds={rounds} grid={grid}", flush=True)
    g = np.random.default_rng(N)
    X = (g.integers(0, grid, (N, d)) if grid else g.standard_normal((N, d))).astype(np.float32)
    oi, od = O.rpknn(X, kappa, leaf, rounds, 5)
    gi, gd = A.knn_rptree(torch.from_numpy(X).cuda(), kappa, leaf, rounds, 5)
    assert np.array_equal(gd.cpu().numpy(), od)
    assert np.array_equal(gi.cpu().numpy(), oi)
