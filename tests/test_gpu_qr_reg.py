"""The register form of the pivoted QR against the FP64 oracle (needs an
MI355X) at the edges of its three shapes (64, 128 and 256 columns; 64, 96 and
160 sampled rows), one row beyond each (the next shape, or the streaming
form), more sampled rows than points outside a node, and a loose tolerance
(ranks far below the bound).  Skeletons index for index, P within FP32
storage."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1410_0260_amd import synth
from tests.gpu_common import run_both
from tests.test_gpu_parity import gparams

pytestmark = pytest.mark.gpu

CASES = [  # N, d, m, s, l, tau
    (900, 6, 64, 32, 64, 1e-6), (900, 6, 64, 32, 65, 1e-6), (1100, 8, 128, 64, 96, 1e-6), (1100, 8, 128, 64, 97, 1e-6),
    (1500, 10, 256, 128, 160, 1e-6), (1500, 10, 256, 128, 161, 1e-6), (300, 4, 33, 17, 64, 1e-6), (170, 5, 120, 40, 80, 1e-6),
    (1200, 5, 200, 90, 130, 1e-2), (40, 3, 20, 16, 30, 0.0),
]


@pytest.mark.parametrize("N,d,m,s,ell,tau", CASES)
def test_skeletons_and_projections(N, d, m, s, ell, tau):
    print(f"\n[qr reg] N={N} d={d} m={m} s={s} l={ell} tau={tau}", flush=True)
    p = O.Params(m=m, kappa=8, smax=s, ell=ell, tau=tau, h=1.0, seed=3)
    X = synth.mixture_points(N, d, min(d, 4), 3, 1e-3, N + ell)
    st, g = run_both(X, synth.weights(N, 1, N), p, gparams(p))
    sk, nodes, off = st["sk"], st["nodes"], 0
    for a in range(1, len(nodes)):
        k, n = sk.k[a], sk.ncols[a]
        assert g["k"][a] == k and np.array_equal(g["S"][a, :k], sk.S[a, :k]), f"node {a}"
        n_a = nodes[a]["hi"] - nodes[a]["lo"]
        ncap = n_a if nodes[a]["left"] < 0 else 2 * s
        if k and n > k:
            Pg, Po = g["P"][off:off + k * (n - k)].reshape(k, n - k), sk.proj(a)
            assert np.linalg.norm(Pg - Po) <= 1e-5 * max(1.0, np.linalg.norm(Po)), f"node {a}"
        off += min(s, min(ell, N - n_a), ncap) * ncap


@pytest.mark.parametrize("N,d,leaf,s,ell", [(1000, 3, 63, 30, 60), (2000, 4, 125, 60, 90), (3600, 4, 225, 120, 148),
                                            (1999, 12, 250, 63, 96)])
def test_forms_agree_bit_for_bit(N, d, leaf, s, ell, monkeypatch):
    """The register form and the gang (forced), and for more than 256 columns
    allowed (a larger bound of the same tree's leaves) the streaming form, with
    tau = 0 and a wide kernel: the last pivots are rounding, so one bit in any
    step shows."""
    import torch
    from paper_1410_0260_amd import askit as A
    print(f"\n[qr forms] N={N} d={d} leaf={leaf} s={s} l={ell}", flush=True)
    X = torch.from_numpy(np.random.default_rng(N).standard_normal((N, d)).astype(np.float32)).cuda()
    runs = []
    for m, gang in ((leaf, ""), (leaf, "1"), (2 * leaf - 2, "0")):
        if gang:
            monkeypatch.setenv("ASKIT_QR_GANG", gang)
        h = A.setup(X, A.default_params(leaf_size=m, kappa=8, max_skeleton=s, sample_rows=ell, id_tol=0.0,
                                        bandwidth=2.0 * d ** 0.5, seed=3))
        runs.append(h.structures())
        h.close()
    for g in runs[1:]:
        assert np.array_equal(g["nodes"], runs[0]["nodes"])
        for f in ("k", "S"):
            assert np.array_equal(g[f], runs[0][f]), f
        for a in range(1, len(g["k"])):
            n = g["ncols"][a]
            assert np.array_equal(g["colperm"][a, :n], runs[0]["colperm"][a, :n]), a
        assert np.array_equal(g["P"], runs[0]["P"])
