"""The evaluation kernel against FP64 direct sums (needs an MI355X): one leaf
holds every point, so u is the direct sum and every difference is the
kernel's rounding.  Dimensions at the edges of the coordinate forms (FP32 up
to 6, bf16 up to 12, FP16 from 13 on, padded to 16, 32, 48 or 64), target
counts at the edges of the target blocks (32, 64, 128, 256), source counts that
leave partial tiles, column counts of every contraction, both bandwidth rules,
and points too far apart for the FP16 form.

Tolerance per target, relative to S = sum |K||w|: an exponent is off by at
most 16 x 2^-24 of E = the largest g (|x|^2 + |y|^2) (three dropped terms of
2^-24 |x||y| per split product, at most 10 truncated sums at full size, and
the norms' own rounding), the sums by 128 x 2^-24 (64 sources per step, up to
32 steps, and exp2)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [  # N, d, h (0: variable), columns, offset of the points (300: deviation 0.1, beyond the FP16 range)
    (33, 2, 0.5, 1, 0), (64, 4, 0.7, 1, 0), (65, 6, 0.6, 5, 0), (129, 5, 0.0, 4, 0), (256, 7, 0.9, 1, 0),
    (257, 12, 1.1, 33, 0), (300, 13, 1.0, 2, 0), (511, 16, 1.0, 64, 0), (513, 17, 2.0, 1, 0), (1000, 33, 0.0, 3, 0),
    (1000, 48, 2.0, 32, 0), (2047, 64, 3.0, 1, 0), (2048, 64, 0.0, 37, 0), (700, 40, 0.1, 1, 300), (70, 20, 0.0, 1, 0),
]


@pytest.mark.parametrize("N,d,h,R,off", CASES)
def test_direct_sums(N, d, h, R, off):
    import torch
    from paper_1410_0260_amd import askit as A
    print(f"\n[eval tile] N={N} d={d} h={h} R={R} offset={off}", flush=True)
    g = np.random.default_rng(N + d)
    X = (g.standard_normal((N, d)) * (0.1 if off else 1.0) + off).astype(np.float32)
    W = g.standard_normal((N, R)).astype(np.float32)
    hd = A.setup(torch.from_numpy(X).cuda(), A.default_params(
        leaf_size=2048, kappa=16, max_skeleton=32, sample_rows=52, bandwidth=h or 1.0, bw_neighbor=0 if h else 8, seed=3))
    hd.update_weights(torch.from_numpy(W).cuda())
    U = hd.evaluate().cpu().numpy().astype(np.float64)
    hs = hd.export(A.X_BANDWIDTH, np.float64)
    hd.close()
    X = X.astype(np.float64)
    gj = 1.0 / (2 * hs * hs)
    D = ((X[:, None, :] - X[None]) ** 2).sum(2) if N * N * d < 3e7 else \
        np.stack([((x - X) ** 2).sum(1) for x in X])
    K = np.exp(-D * gj[None, :])
    E = 2 * 1.4427 * gj.max() * ((X - X.mean(0)) ** 2).sum(1).max() * 2
    tol = 2.0 ** -24 * (16 * E + 128)
    err = np.abs(U - K @ W) / (K @ np.abs(W))
    print(f"[eval tile] largest error {err.max():.2e}, tolerance {tol:.2e}", flush=True)
    assert err.max() < tol
