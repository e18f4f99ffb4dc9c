"""The calls that programs make of the gfx950 ASKIT library, at the sizes they are made.

Kinds of case (key "kind"):

  solve   a point set seen for the first time: setup + update_weights + evaluate
  rp      the same on approximate neighbours: knn_rptree + setup_with_knn + update + evaluate
  apply   one more weight block on a resident setup: update_weights + evaluate
  query   new target points against a resident setup: query or query_neighbors
  batch   one more weight block on many small resident problems: Batch.run
  serve   a burst of weight and query requests to a resident server

Points are Gaussian mixtures on a random q-dimensional subspace of R^d plus a
little ambient noise (q = d: a plain normal cloud), weights are N(0, 1).
"""
import math
import random

import torch

from paper_1410_0260_amd import askit as A

# leaf size, neighbours, skeleton size, sampled rows, ID tolerance
PARAMS = {
    "small": dict(m=128, kappa=16, s=64, ell=84, tau=1e-6),     # CPU-checkable workload
    "batch": dict(m=256, kappa=16, s=128, ell=148, tau=1e-5),   # the batched workload's instances
    "trend": dict(m=256, kappa=64, s=128, ell=148, tau=0.0),    # fixed rank, 4-D normal points
    "paper": dict(m=512, kappa=32, s=256, ell=276, tau=1e-5),   # 2^20 points, serving, 1000-D
}


def listed():
    return [
        # The smallest problem of the repository: launches, host waits and latency.
        dict(name="solve_4k", kind="solve", N=4096, d=8, q=3, comps=4, noise=1e-3, h=8.0, p="small", R=1, prec=0),
        # The fixed-rank runs on 4-D normal points with many neighbours per point.
        dict(name="solve_100k_4d", kind="solve", N=100000, d=4, q=4, comps=1, noise=0.0, h=3.54, p="trend", R=1,
             prec=0),
        # The benchmark's step: 2^20 points in 64-D with a wide kernel.
        dict(name="solve_1m_64d", kind="solve", N=1 << 20, d=64, q=8, comps=16, noise=1e-3, h=16.0, p="paper", R=1,
             prec=0),
        # Wide rows, 16 right-hand sides, the bf16x3 precision form, a size that is no multiple of anything.
        dict(name="solve_50k_1000d", kind="solve", N=50001, d=1000, q=6, comps=8, noise=1e-4, h=16.0, p="paper",
             R=16, prec=1),
        # Approximate neighbours from random projection trees.
        dict(name="solve_rp_131k_4d", kind="rp", N=131071, d=4, q=4, comps=1, noise=0.0, h=3.54, p="trend", R=1,
             prec=0, rounds=4),
        # An iteration of a solver on a small resident problem: the smallest call.
        dict(name="apply_4k", kind="apply", N=4096, d=8, q=3, comps=4, noise=1e-3, h=8.0, p="small", R=1, prec=0),
        # An iteration of a solver at the benchmark's size.
        dict(name="apply_1m_64d", kind="apply", N=1 << 20, d=64, q=8, comps=16, noise=1e-3, h=16.0, p="paper", R=1,
             prec=0),
        # A full block of weight columns (block solvers, several outputs) on a ragged size.
        dict(name="apply_200k_64rhs", kind="apply", N=200003, d=32, q=8, comps=16, noise=1e-3, h=16.0, p="paper",
             R=64, prec=0),
        # Prediction at a handful of new points: latency of the neighbour search.
        dict(name="query_17", kind="query", N=1 << 18, d=64, q=8, comps=16, noise=1e-3, h=16.0, p="paper", R=1,
             prec=0, M=17, op="query"),
        # Prediction at a large set of new points.
        dict(name="query_20k", kind="query", N=1 << 20, d=64, q=8, comps=16, noise=1e-3, h=16.0, p="paper", R=1,
             prec=0, M=20011, op="query"),
        # Many uneven resident problems with the variable bandwidth, one more weight vector for all.
        dict(name="batch_64", kind="batch", count=64, Nmin=2048, Nmax=65536, p="batch", R=1, mix=1),
        # A burst of mixed requests to a resident server.
        dict(name="serve_12", kind="serve", N=1 << 18, d=64, q=8, comps=32, noise=1e-3, h=16.0, p="paper", R=1,
             prec=0, requests=12, max_rhs=64, max_queries=4096, passes=4, mix=1),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _points_drawn(rng, most):
    """A point set of at most `most` coordinates in all (most / 16 points), and 2^20 points (2^16 above 128 dimensions)."""
    p = rng.choice(list(PARAMS))
    d = 4 if p == "trend" else _log_int(rng, 5, 1000 if p == "paper" else 64)
    N = _log_int(rng, 1500, min(1 << 16 if d > 128 else 1 << 18 if p == "trend" else 1 << 20, most // max(d, 16)))
    q = d if p == "trend" else rng.randint(3, min(8, d))
    return dict(N=N, d=d, q=q, comps=1 if p == "trend" else rng.choice([4, 8, 16]),
                noise=0.0 if p == "trend" else 1e-3, h=3.54 if p == "trend" else 16.0, p=p)


def draw(rng):
    kind = rng.choice(["solve"] * 4 + ["apply"] * 3 + ["query"] * 2 + ["rp", "batch", "serve"])
    if kind == "batch":
        return dict(kind=kind, count=_log_int(rng, 4, 64), Nmin=2048, Nmax=_log_int(rng, 4096, 65536), p="batch",
                    R=rng.choice([1, 1, 2, 3, 8]), mix=rng.randrange(1 << 20))
    if kind == "rp":
        return dict(kind=kind, N=_log_int(rng, 3000, 131071), d=4, q=4, comps=1, noise=0.0, h=3.54, p="trend", R=1,
                    prec=0, rounds=rng.randint(1, 4))
    c = _points_drawn(rng, 1 << 22 if kind == "serve" else 1 << 26)
    if kind == "solve":
        return dict(kind=kind, **c, R=_log_int(rng, 1, 16), prec=rng.choice([0, 0, 0, 1]))
    if kind == "apply":
        return dict(kind=kind, **c, R=_log_int(rng, 1, 64) if c["N"] <= 300000 else 1, prec=rng.choice([0, 0, 0, 1]))
    if kind == "query":
        return dict(kind=kind, **c, R=rng.choice([1, 1, 4, 16]), prec=0, M=_log_int(rng, 1, 20000),
                    op=rng.choice(["query", "query", "neighbors"]))
    return dict(kind=kind, **c, R=1, prec=0, requests=rng.randint(4, 12), max_rhs=64, max_queries=4096,
                passes=rng.choice([0, 1, 4]), mix=rng.randrange(1 << 20))


# ------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _cloud(case, seed, rows):
    """rows(): point sets of the given sizes from one mixture (same subspace and component means)."""
    d, q = case["d"], case["q"]
    cpu = torch.Generator().manual_seed(seed)
    basis = torch.linalg.qr(torch.randn(d, q, generator=cpu, dtype=torch.float64))[0].float().cuda()
    if q == d:
        basis = torch.eye(d, device="cuda")
    means = 3.0 * torch.randn(case["comps"], q, generator=cpu).cuda() if case["comps"] > 1 else None
    out = []
    for k, n in enumerate(rows):
        g = _gen(seed * 64 + k + 1)
        z = torch.randn(n, q, generator=g, device="cuda")
        if means is not None:
            z += means[torch.randint(case["comps"], (n,), generator=g, device="cuda")]
        x = z @ basis.T
        if case["noise"] > 0:
            x += math.sqrt(case["noise"]) * torch.randn(n, d, generator=g, device="cuda")
        out.append(x.contiguous())
    return out


def _weights(n, R, seed):
    return torch.randn(n, R, generator=_gen(seed * 64 + 63), device="cuda")


def _requests(case):
    """Sizes of a burst's requests: half weight blocks, half query sets; the same for every seed."""
    r = random.Random(case["mix"])
    out = []
    for k in range(case["requests"]):
        if k % 2 == 0:
            out.append(("weights", r.randint(1, case["max_rhs"])))
        else:
            out.append(("query", _log_int(r, 1, case["max_queries"])))
    return out


def _instances(case):
    """(N, d) of a batch's problems: N log-uniform, d in {16, 32, 64}; the same for every seed."""
    r = random.Random(case["mix"])
    return [(_log_int(r, case["Nmin"], case["Nmax"]), r.choice([16, 32, 64])) for _ in range(case["count"])]


def _params(case):
    p = PARAMS[case["p"]]
    var = case["kind"] == "batch"
    return A.default_params(leaf_size=p["m"], kappa=p["kappa"], max_skeleton=p["s"], sample_rows=p["ell"],
                            id_tol=p["tau"], bandwidth=1.0 if var else case["h"], bw_neighbor=16 if var else 0,
                            precision=case.get("prec", 0), seed=2)


def _inputs(case, seed):
    """Every tensor that goes into the calls of a case."""
    kind = case["kind"]
    if kind == "batch":
        Xs = [_cloud(dict(d=d, q=4, comps=1, noise=1e-3), seed * 256 + i, [n])[0]
              for i, (n, d) in enumerate(_instances(case))]
        return dict(Xs=Xs, W=_weights(sum(len(x) for x in Xs), case["R"], seed))
    if kind == "query":
        X, Y = _cloud(case, seed, [case["N"], case["M"]])
        return dict(X=X, Y=Y, W=_weights(case["N"], case["R"], seed))
    if kind == "serve":
        req = _requests(case)
        X, *Ys = _cloud(case, seed, [case["N"]] + [n if what == "query" else 1 for what, n in req])
        given = [Ys[k] if what == "query" else _weights(case["N"], n, seed * 64 + k) for k, (what, n) in enumerate(req)]
        return dict(X=X, W=_weights(case["N"], case["R"], seed), req=[what for what, _ in req], given=given)
    X, = _cloud(case, seed, [case["N"]])
    return dict(X=X, W=_weights(case["N"], case["R"], seed))


# --------------------------------------------------------------------- runs
def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case, params=_params(case))
    kind = case["kind"]
    if kind in ("apply", "query", "serve"):
        s["handle"] = A.setup(s["X"], s["params"])
    if kind == "query":
        s["handle"].update_weights(s["W"])
    if kind == "serve":
        s["server"] = A.Server(s["handle"], s["W"], A.server_config(weight_passes=case["passes"]))
    if kind == "batch":
        s["batch"] = A.Batch(s.pop("Xs"), s["params"])
        s["U"] = torch.empty_like(s["W"])
    return s


def _solve(s, handle):
    handle.update_weights(s["W"])
    U = handle.evaluate()
    handle.close()
    return U


def run(state):
    s, case = state, state["case"]
    kind = case["kind"]
    if kind == "solve":
        return _solve(s, A.setup(s["X"], s["params"]))
    if kind == "rp":
        knn, _ = A.knn_rptree(s["X"], PARAMS[case["p"]]["kappa"], 256, case["rounds"], 2)
        return _solve(s, A.setup_with_knn(s["X"], knn, s["params"]))
    if kind == "apply":
        s["handle"].update_weights(s["W"])
        return s["handle"].evaluate()
    if kind == "query":
        return s["handle"].query(s["Y"]) if case["op"] == "query" else s["handle"].query_neighbors(s["Y"])
    if kind == "batch":
        return s["batch"].run(s["W"], s["U"])
    sv = s["server"]
    tickets = [sv.submit_weights(x) if what == "weights" else sv.submit_query(x)
               for what, x in zip(s["req"], s["given"])]
    return [sv.wait(t) for t in tickets]


# --------------------------------------------------------------------- work
def _eval_work(n, d, R, p, N):
    """flops of n targets' sums: at the least the own leaf directly and one skeleton a level."""
    levels = max(0.0, math.log2(max(1.0, N / p["m"])))
    return n * min(N, p["m"] + p["s"] * levels) * (2 * d + 3 + 2 * R)


def _setup_work(N, d, p):
    """flops of a setup: G and a pivoted QR of rank s at every node, kappa^2 candidate distances a point."""
    nodes = max(0, 2 * N / p["m"] - 1)
    n = min(p["m"], 2 * p["s"])
    return nodes * p["ell"] * n * (3 * d + 4 * p["s"]) + 3.0 * N * p["kappa"] ** 2 * d


def work(case):
    p, R = PARAMS[case["p"]], case["R"]
    if case["kind"] == "batch":
        inst = _instances(case)
        return dict(bytes=sum(4 * n * (d + 2 * R) for n, d in inst),
                    flops=sum(_eval_work(n, d, R, p, n) for n, d in inst))
    N, d = case["N"], case["d"]
    if case["kind"] == "query":
        M = case["M"]
        look = 2.0 * M * d * p["kappa"] ** 2
        if case["op"] == "neighbors":
            return dict(bytes=4 * d * (N + M) + 12 * M * p["kappa"], flops=look)
        return dict(bytes=4 * d * (N + M) + 4 * R * M, flops=look + _eval_work(M, d, R, p, N))
    if case["kind"] == "serve":
        req = _requests(case)
        return dict(bytes=sum(4 * N * (d + 2 * n) if what == "weights" else 4 * d * (N + n) for what, n in req),
                    flops=sum(_eval_work(N, d, n, p, N) if what == "weights" else
                              _eval_work(n, d, R, p, N) + 2.0 * n * d * p["kappa"] ** 2 for what, n in req))
    flops = _eval_work(N, d, R, p, N)
    if case["kind"] != "apply":
        flops += _setup_work(N, d, p)
    return dict(bytes=4 * N * (d + 2 * R), flops=flops)


# -------------------------------------------------------------------- exact
def _sums(T, X, W, h):
    """The kernel sums of sources X with weights W at targets T in 64 bits."""
    c = X.double().mean(0)
    X, T, W = X.double() - c, T.double() - c, W.double()
    a = 1.0 / (2 * h * h)
    right = torch.cat([2 * a * X, -a * X.square().sum(1, keepdim=True), torch.ones(len(X), 1, device=X.device,
                                                                                  dtype=X.dtype)], 1).T.contiguous()
    U = torch.empty(len(T), W.shape[1], device=X.device, dtype=X.dtype)
    rows = max(1, (1 << 28) // len(X))
    for i in range(0, len(T), rows):
        t = T[i:i + rows]
        left = torch.cat([t, torch.ones_like(t[:, :1]), -a * t.square().sum(1, keepdim=True)], 1)
        U[i:i + rows] = (left @ right).exp_() @ W
    return U


def _nearest(T, X, kappa):
    """Squared distances of the kappa nearest sources of each target in 64 bits (the ids have no such value)."""
    X = X.double()
    out = []
    for i in range(0, len(T), 256):
        t = T[i:i + 256].double()
        r2 = (t.square().sum(1, keepdim=True) + X.square().sum(1)[None, :]).addmm_(t, X.T, alpha=-2)
        near = r2.topk(min(2 * kappa, len(X)), largest=False)[1]
        d2 = (X[near] - t[:, None, :]).square().sum(2)
        out.append(d2.sort(1)[0][:, :kappa])
    return torch.cat(out)


def exact(case, seed):
    if case["kind"] == "batch":   # narrow variable bandwidths: the method's own error is far above rounding
        return None
    s = _inputs(case, seed)
    if case["kind"] == "query":
        if case["op"] == "neighbors":
            return None, _nearest(s["Y"], s["X"], PARAMS[case["p"]]["kappa"])
        return _sums(s["Y"], s["X"], s["W"], case["h"])
    if case["kind"] == "serve":
        return [_sums(x, s["X"], s["W"], case["h"]) if what == "query" else _sums(s["X"], s["X"], x, case["h"])
                for what, x in zip(s["req"], s["given"])]
    return _sums(s["X"], s["X"], s["W"], case["h"])
