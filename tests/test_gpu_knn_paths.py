"""Neighbour lists bit for bit against the FP64 oracle (needs an MI355X) on the
search's routes by size and list length: small point sets swept whole (with
rows that overflow their slots), list lengths that leave the candidates no room
(direct re-ranking, small, in column segments and through the triangular
sweep), and thousands of coincident points (rows that overflow every filter and
are scanned exactly)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1410_0260_amd import synth

pytestmark = pytest.mark.gpu

CASES = [  # N, d, kappa, leaf, coincident points
    (65, 3, 64, 32, 0), (1500, 4, 64, 256, 0), (3000, 40, 49, 200, 0), (16384, 6, 64, 256, 0), (16385, 6, 50, 256, 0), (32769, 5, 64, 256, 0),
    (20011, 12, 64, 300, 0), (33000, 8, 16, 256, 0), (8000, 20, 16, 256, 0), (15000, 64, 32, 512, 0), (300, 5, 48, 40, 0),
    (32833, 70, 16, 300, 0), (33000, 96, 16, 300, 0), (33001, 100, 24, 300, 0), (33000, 128, 16, 300, 0),
    (40001, 30, 16, 256, 6000), (6000, 4, 64, 128, 2500), (6000, 4, 8, 128, 2500), (33001, 3, 64, 128, 1500),
]


@pytest.mark.parametrize("N,d,kappa,m,dup", CASES)
def test_lists_bit_exact(N, d, kappa, m, dup):
    import torch
    from paper_1410_0260_amd import askit as A
    print(f"\n[knn paths] N={N} d={d} kappa={kappa} m={m} coincident={dup}", flush=True)
    X = synth.mixture_points(N, d, min(d, 4), 4, 1e-3, N + kappa)
    if dup:
        X[np.random.default_rng(N).choice(N, dup, replace=False)] = X[0]
    h = A.setup(torch.from_numpy(X).cuda(), A.default_params(leaf_size=m, kappa=kappa, max_skeleton=16,
                                                             sample_rows=36, bandwidth=1.0, seed=1))
    gi = h.export(A.X_KNN_IDX, np.int32).reshape(N, kappa)
    gd = h.export(A.X_KNN_DIST, np.float64).reshape(N, kappa)
    inf = h.info()
    h.close()
    print(f"[knn paths] retried {inf['knn_retry_rows']}, uncertified {inf['knn_uncertified_rows']}", flush=True)
    rows = np.arange(N) if N <= 8000 else np.sort(np.random.default_rng(7).choice(N, 1500, replace=False))
    # all rows against all points, without the row itself
    oi, od = O.knn(X[rows], X, kappa + 1, exclude_self=False)
    for a, r in enumerate(rows):
        keep = oi[a] != r
        if keep.all():                       # coincident points with smaller ids pushed the row out of its list
            keep[-1] = False
        assert np.array_equal(gi[r], oi[a][keep]), f"row {r}"
        assert np.array_equal(gd[r], od[a][keep]), f"row {r}"


WIDE = [  # N, d, kappa, leaf, coincident points
    (200, 129, 16, 64, 0), (129, 300, 64, 64, 0), (4097, 144, 32, 256, 0), (5000, 150, 8, 128, 1500), (3000, 1000, 49, 512, 0),
    (33001, 200, 16, 512, 0), (34000, 136, 32, 512, 2000),
]


@pytest.mark.parametrize("N,d,kappa,m,dup", WIDE)
def test_wide_lists_bit_exact(N, d, kappa, m, dup):
    """More than 128 dimensions: column segments, windows and the triangular
    sweep, partial blocks of rows, columns and dimensions, rows without a
    certificate."""
    test_lists_bit_exact(N, d, kappa, m, dup)
