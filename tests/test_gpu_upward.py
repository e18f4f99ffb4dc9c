"""The upward pass and the slot sums at every column form (needs an MI355X).

Upward: skeleton weights from the exported blocks in FP64, for blocks below and
above the 256 columns staged at a time and skeletons that leave partial row
groups; every column has the bits it has alone.  Tolerance per entry: an fma
chain of nr / 64 terms per lane, six adds over the wave and the last one, each
within 2^-24 of sum |P||w| + |w0|.

Sums: u and its near part of 1, 3 and 4 columns (the staged, the one-column and
the four-column form) and of 5, 32 and 64 agree bit for bit, column by column."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [  # N, d, leaf, smax, tau
    (4096, 8, 128, 64, 1e-6), (6000, 3, 64, 33, 0.0), (9001, 16, 512, 256, 1e-3), (5000, 24, 400, 300, 0.0),
]


@pytest.mark.parametrize("N,d,leaf,smax,tau", CASES)
def test_skeleton_weights_and_sums(N, d, leaf, smax, tau):
    import torch
    from paper_1410_0260_amd import askit as A
    print(f"\n[upward] N={N} d={d} leaf={leaf} smax={smax} tau={tau}", flush=True)
    g = np.random.default_rng(N + smax)
    X = g.standard_normal((N, d)).astype(np.float32)
    W = g.standard_normal((N, 64)).astype(np.float32)
    h = A.setup(torch.from_numpy(X).cuda(), A.default_params(
        leaf_size=leaf, kappa=16, max_skeleton=smax, sample_rows=smax + 20, id_tol=tau, bandwidth=float(d) ** 0.5,
        seed=3))
    wide = {}
    for R in (64, 1, 2, 3, 4, 5, 7, 8, 15, 17, 32):
        h.update_weights(torch.from_numpy(W[:, :R].copy()).cuda())
        u, un = (t.cpu().numpy() for t in h.evaluate_parts())
        e = h.structures()
        k = e["k"]
        if R == 64:
            ref = e
        for a in range(1, len(k)):
            assert np.array_equal(e["Wsk"][a, :k[a]], ref["Wsk"][a, :k[a], :R]), (R, a)
        wide.setdefault(R > 4, (u, un))
        for x, y in zip(wide[R > 4], (u, un)):
            n = min(x.shape[1], R)
            assert np.array_equal(x[:, :n], y[:, :n]), R
    h.close()
    Wt = W[ref["perm"]].astype(np.float64)
    nodes, k, off, worst = ref["nodes"], ref["k"], 0, 0.0
    for a in range(1, len(k)):
        lo, hi, left, right = (int(nodes[a][f]) for f in ("lo", "hi", "left", "right"))
        n = int(ref["ncols"][a])
        ncap = hi - lo if left < 0 else 2 * smax
        B = Wt[lo:hi] if left < 0 else np.concatenate([ref["Wsk"][c, :k[c]] for c in (left, right)]).astype(np.float64)
        assert len(B) == n
        pv, ka = ref["colperm"][a], int(k[a])
        P = ref["P"][off:off + ka * (n - ka)].reshape(ka, n - ka).astype(np.float64)
        off += min(smax, int(ref["T_cnt"][a]), ncap) * ncap
        w0, w1 = B[pv[:ka]], B[pv[ka:n]]
        err = np.abs(ref["Wsk"][a, :ka] - (w0 + P @ w1))
        S = np.abs(P) @ np.abs(w1) + np.abs(w0)
        worst = max(worst, float((err / ((n / 64 + 8) * 2.0 ** -24 * S)).max()) if ka else 0.0)
    print(f"[upward] largest error over its bound {worst:.3f}", flush=True)
    assert worst < 1.0
