"""Interaction lists and the query sort at the edges of their forms (needs an
MI355X): trees of one node, with a partly filled last level, of 8,191 nodes
(the largest whose row masks are used) and above, level-restricted or not,
against lists built here from the exported neighbours; query counts around the
4,096 keys that are sorted in LDS."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TREES = [  # N, leaf, kappa, levels that may be pruned (0: all)
    (100, 128, 8, 0), (129, 128, 8, 0), (1000, 63, 5, 0), (3001, 47, 33, 0), (3001, 47, 33, 2), (2050, 2, 4, 0),
    (8192, 2, 16, 0), (9000, 2, 3, 0),
]


def _lists(e, N, minlev):
    nodes = e["nodes"]
    pos = np.empty(N, np.int64)
    pos[e["perm"]] = np.arange(N)
    lo, hi, left, right, lev = (nodes[f].astype(np.int64) for f in ("lo", "hi", "left", "right", "level"))
    near, far = {}, {}
    for r in range(N):
        q = pos[e["knn_idx"][e["perm"][r]]]
        q = np.sort(np.append(q[e["knn_idx"][e["perm"][r]] >= 0], r))
        has = np.searchsorted(q, hi) > np.searchsorted(q, lo)
        near[r], far[r] = [], []
        stack = [0]
        while stack:
            a = stack.pop()
            if not has[a] and lev[a] >= minlev:
                far[r].append(a)
            elif left[a] < 0:
                near[r].append(a)
            else:
                stack += [right[a], left[a]]
    return near, far


@pytest.mark.parametrize("N,leaf,kappa,prune", TREES)
def test_lists_match_brute_force(N, leaf, kappa, prune):
    import torch
    from paper_1410_0260_amd import askit as A
    print(f"\n[lists] N={N} leaf={leaf} kappa={kappa} prune={prune}", flush=True)
    X = np.random.default_rng(N + leaf).standard_normal((N, 3)).astype(np.float32)
    h = A.setup(torch.from_numpy(X).cuda(), A.default_params(
        leaf_size=leaf, kappa=kappa, max_skeleton=8, sample_rows=16, bandwidth=1.0, seed=2, prune_levels=prune))
    e = h.structures()
    h.close()
    depth = int(e["nodes"]["level"].max())
    near, far = _lists(e, N, max(1, depth - prune + 1) if prune else 0)
    ptr, node, mask = e["slab_ptr"], e["slab_node"], e["slab_mask"]
    row0 = e["slab_row0"]
    ns = len(row0)
    for part, want in ((0, near), (1, far)):
        got = {r: [] for r in range(N)}
        for s in range(ns):
            p0, p1 = ptr[part * (ns + 1) + s], ptr[part * (ns + 1) + s + 1]
            if not prune:
                assert np.all(np.diff(node[p0:p1]) > 0)
            for i in range(p0, p1):
                m = int(mask[i])
                while m:
                    b = (m & -m).bit_length() - 1
                    got[int(row0[s]) + b].append(int(node[i]))
                    m &= m - 1
        for r in range(N):
            assert sorted(got[r]) == sorted(want[r]), (part, r)


@pytest.mark.parametrize("M", [1, 2, 3, 1025, 4096, 4097, 8200, 20000])
def test_query_sort(M):
    """Every query is evaluated once and lands in its row: u of M new points
    against the FP64 direct sum, tau = 0 and a tree of one level of leaves."""
    import torch
    from paper_1410_0260_amd import askit as A
    print(f"\n[lists] M={M}", flush=True)
    g = np.random.default_rng(M)
    X, W = g.standard_normal((1500, 3)).astype(np.float32), g.standard_normal((1500, 1)).astype(np.float32)
    Y = g.standard_normal((M, 3)).astype(np.float32)
    h = A.setup(torch.from_numpy(X).cuda(), A.default_params(
        leaf_size=400, kappa=8, max_skeleton=256, sample_rows=300, id_tol=0.0, bandwidth=3.0, seed=2))
    h.update_weights(torch.from_numpy(W).cuda())
    u = h.query(torch.from_numpy(Y).cuda()).cpu().numpy().astype(np.float64)
    h.close()
    D = ((Y.astype(np.float64)[:, None] - X.astype(np.float64)[None]) ** 2).sum(2)
    K = np.exp(-D / 18.0)
    # a smooth kernel of rank well below 256: the skeletons are exact to FP32,
    # 1,500 terms and two levels of projections of moderate norm
    err = np.abs(u - K @ W) / (K @ np.abs(W))
    print(f"[lists] largest error {err.max():.2e}", flush=True)
    assert err.max() < 1e-4


@pytest.mark.parametrize("N,leaf", [(300, 256), (4000, 64), (20000, 8), (40000, 2)])
def test_pairs_cover_every_source_once(N, leaf):
    """Sources sorted by key in one to three passes: with a kernel that is 1
    everywhere (rank 1, so one skeleton point is exact) every target's u is the
    sum of the weights; FP32 sums of N positive terms, 2^-20 relative."""
    import torch
    from paper_1410_0260_amd import askit as A
    print(f"\n[lists] N={N} leaf={leaf}", flush=True)
    g = np.random.default_rng(N)
    X, W = g.standard_normal((N, 3)).astype(np.float32), g.random((N, 1)).astype(np.float32)
    h = A.setup(torch.from_numpy(X).cuda(), A.default_params(
        leaf_size=leaf, kappa=4, max_skeleton=8, sample_rows=16, id_tol=1e-3, bandwidth=1e6, seed=2))
    h.update_weights(torch.from_numpy(W).cuda())
    u = h.evaluate().cpu().numpy().astype(np.float64)
    h.close()
    err = np.abs(u / W.astype(np.float64).sum() - 1).max()
    print(f"[lists] largest error {err:.2e}", flush=True)
    assert err < 2.0 ** -20 * max(1.0, N / 4096)
