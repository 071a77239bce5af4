"""The work that users of this library have it do, as timed cases: whole fits from the smallest workload of the
benchmark to the largest that a pass of two seconds allows, fits with the options used in earnest (early termination by
recall, the angular metric, points kept in host memory), single assignment steps of a serving or refreshing program,
the exact assignment, the centroid update and the ground truth of a recall measurement.

Inputs are rows of the seeded mixtures of ``paper_2603_20009_amd.datagen`` (unit norm, skewed variance per dimension),
made on the GPU.  Row lengths, cluster counts and row counts of the listed cases are those of the workloads C1 to C5 and
of the parity tests; ``draw`` spreads over the ranges between them, odd sizes and ragged row lengths among them.

The hierarchical fit has no case: one near-tie in its first phase changes the size of a cluster and with it every later
draw of initial rows, so the outputs of two correct builds cannot be compared value by value.
"""
from __future__ import annotations

import functools
import math

import torch

from paper_2603_20009_amd import datagen, skm


def listed():
    return [
        # A serving program labels a few rows against a small codebook: launches and host work are all there is.
        dict(name="assign few rows", kind="assign", n=64, d=128, k=100, prev=False, kept_rotation=False),
        # A batch of new rows into a trained index (C2's row length and cluster count); the program keeps the rotation.
        dict(name="assign batch", kind="assign", n=20_000, d=1536, k=1024, prev=False, kept_rotation=True),
        # Labels of a large collection refreshed after its centroids moved a little (C5's shape, a quarter of its rows).
        dict(name="assign refresh", kind="assign", n=2_500_000, d=384, k=32_768, prev=True, kept_rotation=False),
        # Exact nearest centroids of rows whose length is no multiple of 16.
        dict(name="exact ragged rows", kind="exact", n=100_003, d=100, k=1000),
        # One centroid update of a user's own loop (C3's shape).
        dict(name="update", kind="update", n=1_000_000, d=768, k=4096),
        # Exact neighbours of a held-out query set (C3's recall measurement).
        dict(name="ground truth", kind="truth", n=1_000_000, d=768, queries=1000, topk=10),
        # C1: a small fit, bound by latency.
        dict(name="fit small", kind="fit", n=20_000, d=128, k=100, iters=10, components=100, recipe="linear", option=""),
        # An odd-sized fit under the angular metric.
        dict(name="fit angular odd", kind="fit", n=120_001, d=200, k=777, iters=6, components=1500, recipe="embed",
             option="angular"),
        # Rows that stay in page-locked host memory and pass through the device in batches.
        dict(name="fit host rows", kind="host", n=200_000, d=768, k=1024, iters=3, components=2048),
        # C3: fit with early termination by recall (four iterations: where the stop comes on this workload).
        dict(name="fit with recall", kind="fit", n=1_000_000, d=768, k=4096, iters=4, components=8192, recipe="embed",
             option="etr"),
        # C2: the workload that the benchmark reports.
        dict(name="fit headline", kind="fit", n=1_000_000, d=1536, k=1024, iters=10, components=4096, recipe="embed",
             option=""),
        # C4's points with C3's cluster count: many clusters, ten iterations.  (A fit into C4's 16 384 clusters leaves sixty
        # rows to a cluster; some run empty, and the draws that re-seed them turn one near-tie into another fit.  Steps
        # against that many centroids are timed above.)
        dict(name="fit many clusters", kind="fit", n=1_000_000, d=1536, k=4096, iters=10, components=16_384,
             recipe="embed", option=""),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _row_length(rng, lo=64, hi=1536):
    """Embedding lengths are multiples of 64 as a rule; a third of the draws are not."""
    d = _log(rng, lo, hi)
    return d if rng.random() < 1 / 3 else min(hi, max(lo, (d + 32) // 64 * 64))


def draw(rng):
    kind = rng.choice(["assign", "assign", "exact", "update", "truth", "fit", "fit", "fit", "host"])
    d = _row_length(rng)
    most = 1_500_000_000 // d           # rows: at most the bytes of the listed cases
    if kind == "assign":
        prev = rng.random() < 0.5
        n, k = _log(rng, 64, min(most, 2_500_000)), _log(rng, 100, 32_768)
        return dict(kind=kind, n=n, d=d, k=min(k, 25_000_000_000_000 // (n * d)), prev=prev, kept_rotation=rng.random() < 0.5)
    if kind == "exact":
        n, k = _log(rng, 1000, min(most, 1_000_000)), _log(rng, 64, 16_384)
        return dict(kind=kind, n=n, d=d, k=min(k, 6_000_000_000_000 // (n * d)))
    if kind == "update":
        n = _log(rng, 5000, min(most, 1_000_000))
        return dict(kind=kind, n=n, d=d, k=_log(rng, 32, min(16_384, n // 16)))
    if kind == "truth":
        return dict(kind=kind, n=_log(rng, 20_000, min(most, 1_000_000)), d=d, queries=_log(rng, 64, 1000),
                    topk=rng.choice([1, 10, 100]))
    if kind == "host":
        n = _log(rng, 20_000, 150_000_000 // d)
        k = _log(rng, 64, min(4096, n // 100))
        return dict(kind=kind, n=n, d=d, k=k, iters=3, components=2 * k)
    n = _log(rng, 5000, min(most, 1_000_000))
    k = _log(rng, 32, min(4096, n // 150))
    option = rng.choice(["", "", "", "angular", "etr"])
    iters = 4 if option == "etr" else rng.choice([4, 6, 10])
    return dict(kind=kind, n=n, d=d, k=k, iters=iters, components=k * rng.choice([2, 4]),
                recipe="linear" if n < 50_000 and rng.random() < 0.5 else "embed", option=option)


@functools.lru_cache(maxsize=8)
def _rotation(d):
    """The orthogonal matrix that a serving program made when it trained its index (on the host, like a stored file)."""
    g = torch.Generator().manual_seed(d)
    q, r = torch.linalg.qr(torch.randn(d, d, generator=g, dtype=torch.float64))
    return (q * torch.sign(torch.diagonal(r))).float().contiguous()


def _member_means(rows, comp, pick, count):
    """For every picked row the mean of itself, twice, and the next `count` rows of its component (fixed order: the same
    bits every time)."""
    order = torch.argsort(comp, stable=True)
    sizes = torch.bincount(comp, minlength=int(comp.max()) + 1)
    start = torch.cumsum(sizes, 0) - sizes
    c = comp[pick]
    at = torch.empty_like(order)
    at[order] = torch.arange(order.numel(), device=order.device)
    out = 2.0 * rows[pick]
    for r in range(1, count + 1):
        out += rows[order[start[c] + (at[pick] - start[c] + r) % sizes[c]]]
    return out / (count + 2)


def _nearest(X, Y):
    """Labels of the rows of X against Y, in plain matrix products."""
    y2 = (Y * Y).sum(1)
    step = max(1, (1 << 29) // Y.shape[0])
    out = [torch.addmm(y2, X[s:s + step], Y.T, alpha=-2.0).argmin(1) for s in range(0, X.shape[0], step)]
    return torch.cat(out).int()


def prepare(case, seed):
    kind, n, d = case["kind"], case["n"], case["d"]
    if kind in ("fit", "host"):
        X = datagen.mixture(n, d, case["components"], seed, case.get("recipe", "embed"), "cuda")
        if kind == "host":
            host = torch.empty(n, d, pin_memory=True)
            host.copy_(X)
            return dict(case=case, X=host, seed=seed)
        opts = skm.FitOptions(angular=case["option"] == "angular")
        if case["option"] == "etr":
            q = datagen.mixture(1000, d, case["components"], seed, case["recipe"], "cuda", sample_seed=seed + 7)
            opts = skm.FitOptions(etr=True, queries=q)
        return dict(case=case, X=X, seed=seed, opts=opts)
    if kind == "truth":
        X = datagen.mixture(n, d, 8192, seed, "embed", "cuda")
        return dict(case=case, X=X, Q=datagen.mixture(case["queries"], d, 8192, seed, "embed", "cuda", sample_seed=seed + 7))
    # Steps against trained centroids: each is the mean of a few rows of a component of another sample of the same
    # mixture; components are picked at random, so that, as in a trained index, most hold a few centroids and some none.
    k = case["k"]
    X = datagen.mixture(n, d, max(1, k // 3), seed, "embed", "cuda")
    T, comp = datagen.mixture(8 * k, d, max(1, k // 3), seed, "embed", "cuda", sample_seed=seed + 7, return_labels=True)
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 13)
    pick = torch.randperm(T.shape[0], generator=g, device="cuda")[:k]
    Y = _member_means(T, comp, pick, 6)
    if kind == "update":
        return dict(case=case, X=X, labels=_nearest(X, Y), Y=Y)
    if kind == "exact":
        return dict(case=case, X=X, Y=Y)
    prev = _nearest(X, _member_means(T, comp, pick, 5)) if case["prev"] else None   # labels from before the last update
    R = _rotation(d).cuda() if case["kept_rotation"] else None
    return dict(case=case, X=X, Y=Y, prev=prev, opts=skm.FitOptions(R=R))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "fit":
        r = skm.fit(state["X"], case["k"], case["iters"], state["seed"], state["opts"])
        return dict(centroids=r.centroids, labels=r.assign, dist=r.dist)
    if kind == "host":
        r = skm.fit_host(state["X"], case["k"], case["iters"], state["seed"])
        return dict(centroids=r.centroids, labels=r.assign, dist=r.dist)
    if kind == "assign":
        a, dist, _ = skm.assign(state["X"], state["Y"], state["prev"], opts=state["opts"])
        return dict(labels=a, dist=dist)
    if kind == "exact":
        a, dist = skm.assign_exact(state["X"], state["Y"])
        return dict(labels=a, dist=dist)
    if kind == "update":
        counts = skm.update(state["X"], state["labels"], state["Y"])
        return dict(centroids=state["Y"], counts=counts)
    return dict(neighbours=skm.etr_ground_truth(state["X"], state["Q"], case["topk"]))


def work(case):
    kind, n, d = case["kind"], case["n"], case["d"]
    if kind == "truth":
        nq = case["queries"]
        return dict(bytes=4 * (n + nq) * d + 8 * nq * case["topk"], flops=2 * n * nq * d)
    k = case["k"]
    if kind == "exact":
        return dict(bytes=4 * (n + k) * d + 8 * n, flops=2 * n * k * d)
    if kind == "update":
        return dict(bytes=4 * (n + 2 * k) * d + 4 * (n + k), flops=n * d)
    first = skm.dprime_init(d)          # dimensions of the first test: what a pruned step multiplies for every pair
    if kind == "assign":
        return dict(bytes=4 * (n + k) * d + 8 * n + (4 * n if case["prev"] else 0),
                    flops=2 * (n + k) * d * d + 2 * n * k * first)
    # rotation, one exact assignment, then pruned steps; every step reads every row once
    steps = case["iters"] + 1
    return dict(bytes=steps * 4 * n * d + 4 * k * d + 8 * n,
                flops=2 * n * d * d + 2 * n * k * d + (steps - 1) * 2 * n * k * first)


def tolerance(case):
    kind = case["kind"]
    if kind == "update":                # fp64 sums, fp32 means; the sizes are counts
        return dict(rel=1e-6, max=1e-5, differ=0.0)
    if kind == "truth":                 # two neighbours at the same distance to 32 bits may change places
        return dict(rel=0.0, differ=2e-3)
    if kind == "exact":                 # near-ties to 32 bits
        return dict(rel=1e-5, max=1e-3, differ=1e-3)
    if kind == "assign":                # and pairs that a test drops or keeps within the same rounding
        return dict(rel=1e-4, max=0.3, differ=1e-3)
    # a near-tie that falls the other way in one iteration moves a point, and with it two centroids, in all later ones
    return dict(rel=3e-3, max=0.9, differ=2e-3)
