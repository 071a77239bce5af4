"""The forms that a kernel takes by size, type or alignment, at the sizes where one hands over to another: each against the
CPU oracle (fp64) or against the form next to it."""
import ctypes
import os
import subprocess
import sys
import threading
import zlib

import numpy as np
import pytest
import torch

from parity import EPS0, check_assignment
from test_gpu_parity import check_ground_truth, cuda, dg, say, skm  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


# The exact assignment reads rows whose length is a multiple of four as they are from 32 dimensions on, unless the padded
# length is a multiple of 32; other rows, and rows that are not 16-byte aligned, go through a padded copy.
@pytest.mark.parametrize("n,d,k", [(1000, 36, 70), (257, 44, 129), (700, 100, 130), (300, 124, 40), (200, 20, 30),
                                   (150, 1004, 60), (129, 52, 1), (128, 34, 128)])
def test_exact_assignment_of_rows_that_are_no_multiple_of_16(skm, orc, dg, n, d, k):  # noqa: F811
    say("exact rows", n, d, k)
    rng = np.random.default_rng(n + d + k)
    X = dg.mixture(n, d, 20, 2, "linear").numpy()
    Y = X[rng.choice(n, k, replace=k > n)] + (0.01 * rng.standard_normal((k, d))).astype(np.float32)
    ao, do = orc.assign_full(X.astype(np.float64), Y.astype(np.float64))
    a, dist = skm.assign_exact(cuda(X), cuda(Y))
    check_assignment(a.cpu().numpy(), ao, X, Y, min_agree=0.999)
    same = a.cpu().numpy() == ao
    assert np.abs(dist.cpu().numpy()[same] - do[same]).max() < 1e-6 * max(1.0, do.max())
    # the same rows behind a start that is not 16-byte aligned: the padded copy, the same sums with zeros behind them
    shifted = torch.empty(n * d + 1, device="cuda")
    shifted[1:] = cuda(X).reshape(-1)
    b, dist_b = skm.assign_exact(shifted[1:].view(n, d), cuda(Y))
    assert torch.equal(a, b) and torch.equal(dist, dist_b)


# Labels and direct distances from the keys of the argmin, without tables: a form for every 256 dimensions up to 2048, one for rows
# beyond.  A lane adds d / 64 squares, its sum and the lanes' six more steps of rounding to a sum of positive terms.
@pytest.mark.parametrize("d", [240, 256, 272, 512, 528, 768, 1024, 1040, 1536, 1552, 2048, 2064])
def test_exact_distances_on_both_sides_of_every_form(skm, d):  # noqa: F811
    say("exact distances", d)
    g = torch.Generator().manual_seed(d)
    X, Y = torch.randn(67, d, generator=g), torch.randn(5, d, generator=g)
    D = torch.cdist(X.double(), Y.double(), compute_mode="donot_use_mm_for_euclid_dist") ** 2
    a, dist = skm.assign_exact(X.cuda(), Y.cuda())
    want, at = D.min(1)
    assert torch.equal(a.cpu().long(), at)
    assert float(((dist.cpu().double() - want).abs() / want).max()) <= (d / 64 + 12) * 2.0 ** -23


# Behind the first test of a listed tile: one product and widened tests (no counts per block asked for, three blocks or more,
# pairs handed over), or three products throughout.  Poor incumbents leave tiles that are done again in three products,
# good ones tiles that hand over at the first test.
@pytest.mark.parametrize("poor", [0, 4, 1])          # no incumbent, every fourth, or all of them drawn at random
@pytest.mark.parametrize("n,d,k,dp", [(1500, 304, 257, 48), (700, 208, 256, 16), (513, 1536, 600, 192),
                                      (129, 272, 513, 80), (2000, 240, 64, 48)])
def test_listed_tiles_in_one_product(skm, orc, dg, n, d, k, dp, poor):  # noqa: F811
    say("listed", n, d, k, dp, poor)
    rng = np.random.default_rng(7 * n + k)
    X = dg.mixture(n, d, 30, n + k, "linear" if d < 512 else "embed").numpy()
    R = orc.random_rotation(d, 5)
    Y = X[rng.integers(0, n, k)] + (0.01 * rng.standard_normal((k, d))).astype(np.float32)   # (more than points, some)
    Xr, Yr = orc.rotate(X, R), orc.rotate(Y, R)
    prev = orc.assign_full(Xr, Yr)[0].astype(np.int32)
    if poor:
        prev[::poor] = rng.integers(0, k, len(prev[::poor]))
    ref = orc.assign_pruned(Xr, Yr, prev, dp, EPS0, 0)
    a, dist, row = skm.assign(cuda(X), cuda(Y), cuda(prev), dp, skm.FitOptions(R=cuda(R), screen=1))
    assert row["screen_dims"] > 0
    check_assignment(a.cpu().numpy(), ref.assign, Xr, Yr)
    same = a.cpu().numpy() == ref.assign
    assert np.abs(dist.cpu().numpy()[same] - ref.dist[same]).max() < 2e-5 * max(1.0, ref.dist.max())
    surv_ref = n * (k - 1) - ref.pruned_first
    assert abs(row["survivors"] - surv_ref) <= max(2, 1e-3 * surv_ref)
    assert abs(row["completed"] - ref.enter[-1]) <= max(2, 1e-3 * ref.enter[-1])
    assert row["changed"] == int((a.cpu().numpy() != prev).sum())


# Grouping by label: a stable counting order for k <= 8192 and n >= 8 k, a scatter with ordered segments otherwise (segments
# up to 2048 by rank, longer ones sorted).  The means are fp64 sums rounded to fp32: any order gives them to 1 ulp.
@pytest.mark.parametrize("n,d,k,skew", [(800, 16, 100, 0), (799, 16, 100, 0), (65_536, 16, 8192, 0), (65_535, 16, 8192, 0),
                                        (66_000, 20, 8193, 0), (30_000, 64, 9000, 25_000), (20_001, 48, 3000, 2049),
                                        (4096, 32, 1, 0), (33, 100, 33, 0)])
def test_update_at_the_borders_of_its_orders(skm, orc, dg, n, d, k, skew):  # noqa: F811
    say("update", n, d, k, skew)
    rng = np.random.default_rng(n + k)
    X = dg.mixture(n, d, 30, 4, "linear").numpy()
    a = rng.integers(0, k, n).astype(np.int32)
    a[:skew] = k // 2
    Y0 = rng.standard_normal((k, d)).astype(np.float32)
    Yo, co = orc.update(X.astype(np.float64), a, Y0.astype(np.float64))
    out = []
    for _ in range(2):
        Yg = cuda(Y0)
        assert (skm.update(cuda(X), cuda(a), Yg).cpu().numpy() == co).all()
        out.append(Yg.cpu().numpy())
    assert np.abs(out[0] - Yo).max() < 1e-6
    assert np.array_equal(out[0][co == 0], Y0[co == 0])
    if n >= 8 * k and k <= 8192:
        assert np.array_equal(out[0], out[1])        # the stable order: the same bits every time


# Panels of 64 rows, the last square or narrower, factored twice where it is: d at the panels' edges.
@pytest.mark.parametrize("d", [17, 63, 64, 65, 127, 128, 129, 191, 200])
def test_rotation_at_the_edges_of_its_panels(skm, d):  # noqa: F811
    R = skm.make_rotation(d, 11).cpu().numpy().astype(np.float64)
    # d entries, each off by half an ulp of fp32 at most, meet in an element of R R^T: 2^-24 sqrt(d) at most by Cauchy-Schwarz
    assert np.abs(R @ R.T - np.eye(d)).max() < 2 * 2.0 ** -24 * np.sqrt(d)


# Up to 128 rows one workgroup makes the matrix, beyond that a chain of kernels whose last 128 rows go round twice: the matrix
# is the orthonormal factor of the normals that (d, seed) stand for, computed here by numpy's QR.  An element is off by half
# an ulp of fp32 plus what fp64 rounding leaves of either factor, 64 eps times the condition of the matrix of normals.
def normals_of(d, seed):
    def mix(z):
        z = z + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))

    with np.errstate(over="ignore"):
        t = np.arange((d * d + 1) // 2, dtype=np.uint64) * np.uint64(2) + np.uint64((seed + 3 * 0xD1342543DE82EF95) % 2**64)
        u1, u2 = ((mix(z) >> np.uint64(11)).astype(np.float64) / 2.0**53 for z in (t, t + np.uint64(1)))
    m = np.sqrt(-2.0 * np.log(u1))
    return np.stack([m * np.cos(2 * np.pi * u2), m * np.sin(2 * np.pi * u2)], 1).reshape(-1)[:d * d].reshape(d, d)


def check_rotation_of_normals(skm, d, seed):  # noqa: F811
    G = normals_of(d, seed)
    q, r = np.linalg.qr(G.T)
    want = (q * np.sign(np.diag(r))).T
    got = skm.make_rotation(d, seed).cpu().numpy().astype(np.float64)
    assert (np.abs(got - want) <= 2.0**-24 * np.abs(want) + 64 * 2.0**-52 * np.linalg.cond(G)).all()
    assert np.abs(got @ got.T - np.eye(d)).max() < 2 * 2.0 ** -24 * np.sqrt(d)      # as below


@pytest.mark.parametrize("d", [1, 2, 15, 16, 17, 64, 65, 100, 128, 129, 192, 193, 260])
def test_rotation_is_the_orthonormal_factor_of_its_normals(skm, d):  # noqa: F811
    say("rotation", d)
    check_rotation_of_normals(skm, d, 5)


# The second factor of a panel is taken without eliminations where its Gram matrix is within 2^-33 of the unit matrix, as it is for the
# seeds of the other tests.  For these it is off by 16 times that and more, in fp64 steps of the same kind, so that what rounding
# does in another order does not bring it back: both generators take the eliminations in their last panel of 64, 36 or 8 rows.
@pytest.mark.parametrize("d,seed", [(64, 346), (64, 366), (100, 340), (100, 8), (128, 392), (128, 54), (192, 41), (192, 16), (200, 32)])
def test_rotation_whose_second_factor_takes_the_eliminations(skm, d, seed):  # noqa: F811
    say("rotation", d, seed)
    W, off = normals_of(d, seed), 0.0
    for p0 in range(0, d, 64):
        P, Q = W[p0:p0 + 64], W[:p0]
        for again in range(2 if d - p0 <= 128 else 1):
            P = P - (P @ Q.T) @ Q
            gram = P @ P.T
            if again:
                off = np.abs(gram - np.eye(len(P))).max()
            P = np.linalg.solve(np.linalg.cholesky(gram), P)
        W[p0:p0 + 64] = P
    assert off > 16 * 2.0**-33
    check_rotation_of_normals(skm, d, seed)


# The ground truth goes through the points in chunks of whole rounds of tiles (256 points x 256 queries): one tile row and
# several, a ragged last chunk, and too few points for the one-product form.
@pytest.mark.parametrize("n,d,nq,K", [(40_000, 1536, 300, 10), (70_001, 1000, 257, 1), (20_000, 96, 64, 10),
                                      (140_000, 64, 5, 100)])
def test_ground_truth_in_chunks(skm, orc, dg, n, d, nq, K):  # noqa: F811
    say("ground truth", n, d, nq, K)
    X = dg.mixture(n, d, 200, 3, "embed").numpy()
    Q = dg.mixture(nq, d, 200, 3, "embed", sample_seed=99).numpy()
    gt = skm.etr_ground_truth(cuda(X), cuda(Q), K).cpu().numpy()
    check_ground_truth(gt, orc.ground_truth(X, Q, K), X, Q)


def test_calls_of_several_threads_share_the_kept_blocks(skm, dg):  # noqa: F811
    """Calls without a lent workspace keep their device blocks for the next such call: calls of several threads on streams of
    their own, between calls that give everything back, return what a call alone returns."""
    n, d, k = 6000, 96, 130
    X = dg.mixture(n, d, 40, 5, "linear").cuda()
    Y = X[:k].contiguous() + 0.01
    want = skm.assign(X, Y, None)[0]
    wrong, errors = [], []

    def work(i):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for r in range(6):
                    if r % 3 == i % 3:
                        skm.release_memory()
                    got = skm.assign(X, Y, None)[0]
                    s.synchronize()
                    if not torch.equal(got, want):
                        wrong.append((i, r))
        except Exception as e:   # noqa: BLE001
            errors.append(repr(e))

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors and not wrong
    skm.release_memory()
    assert torch.equal(skm.assign(X, Y, None)[0], want)


# The probes of a query are drawn from keys in registers (1, 4 or 16 a thread of 256) or, beyond 4096 centroids, read again.
@pytest.mark.parametrize("k", [256, 1025, 4096, 4097])
def test_recall_at_the_borders_of_its_forms(skm, orc, dg, k):  # noqa: F811
    say("recall", k)
    n, d, nq, K = 2 * k + 11, 32, 30, 10
    X = dg.mixture(n, d, 30, 3, "linear").numpy()
    Q = dg.mixture(nq, d, 30, 4, "linear").numpy()
    R = orc.random_rotation(d, 6)
    kw = dict(etr=True, topk=K, probe_frac=0.01, adjust_dprime=False, etr_tol=-1.0)
    ref = orc.fit(X, k, 2, 2, orc.FitParams(eps0=EPS0, **kw), R=R, init_idx=orc.sample_rows(2, n, k), queries=Q)
    got = skm.fit(cuda(X), k, 2, 2, skm.FitOptions(R=cuda(R), queries=cuda(Q), **kw))
    for g, r in zip(got.trace[:2], ref.trace):
        assert g["recall"] == pytest.approx(r["recall"], abs=2.0 / (nq * K))   # (a near-tie may move one neighbour or one probe)


# A split leaves two centroids at y (1 +- 1/1024); the points between them are decided by the last bits of their distances,
# and one that falls the other way moves every later centroid of the two.  The order in which products and norms are added
# therefore stays what it is: the labels of these fits (all split an empty cluster) are pinned bit by bit.
def test_labels_of_fits_that_split_a_cluster_are_pinned(skm):  # noqa: F811
    n, d, k = 20_000, 128, 100
    scale = (1.0 - 0.9 * np.arange(d) / (d - 1)).astype(np.float32)
    with open(os.path.join(os.path.dirname(__file__), "golden", "split_fit_labels.txt")) as f:
        pins = [line.split() for line in f if not line.startswith("#")]
    other = []
    for seed, crc in pins:
        say("pinned fit", seed)
        rng = np.random.default_rng(int(seed))
        means = rng.standard_normal((k, d), dtype=np.float32)
        X = rng.standard_normal((n, d), dtype=np.float32) * scale + means[rng.integers(0, k, n)]
        r = skm.fit(cuda(X), k, 10, int(seed))
        assert sum(t["nempty"] for t in r.trace) > 0
        if zlib.crc32(r.assign.cpu().numpy().tobytes()) != int(crc, 16):
            other.append(seed)
    assert not other


# The last 256 rows are projected and factorised twice: the matrix before rounding is orthogonal to some 1e-14, and with one
# pass less an entry of each of these rounds to the other side.
def test_rotation_matrices_are_pinned(skm):  # noqa: F811
    with open(os.path.join(os.path.dirname(__file__), "golden", "rotations.txt")) as f:
        pins = [line.split() for line in f if not line.startswith("#")]
    other = []
    for d, seed, crc in pins:
        say("pinned rotation", d, seed)
        if zlib.crc32(skm.make_rotation(int(d), int(seed)).cpu().numpy().tobytes()) != int(crc, 16):
            other.append((d, seed))
    assert not other


# A call that ends with an error leaves no kernel behind that could still write into its page-locked blocks (the next call of
# the thread, on whatever stream, takes them): initial rows out of range are refused before anything is enqueued, and what
# is only seen later is returned once the stream has been waited for.
def test_calls_that_end_with_an_error_leave_nothing_running(skm, dg):  # noqa: F811
    n, d, k = 60_000, 512, 16
    X = dg.mixture(n, d, 40, 3, "linear", "cuda")
    ws = torch.full((skm.workspace_bytes(n, d, k),), 0xA5, dtype=torch.uint8, device="cuda")
    rows = list(range(k - 1))
    torch.cuda.synchronize()
    for bad in (n, -1):
        with pytest.raises(skm.SkmError, match="init_idx"):
            skm.fit(X, k, 3, 1, skm.FitOptions(init_idx=rows + [bad], workspace=ws))
        assert torch.cuda.current_stream().query()
        assert bool((ws == 0xA5).all())
        with pytest.raises(skm.SkmError, match="init_idx"):
            skm.fit_host(X[:1000].cpu(), k, 2, 1, opts=skm.FitOptions(init_idx=rows + [bad]))
    with pytest.raises(skm.SkmError, match="nq > n"):
        skm.fit(X, k, 3, 1, skm.FitOptions(etr=True, nq=n + 1))
    assert torch.cuda.current_stream().query()
    # the thread's next calls, on another stream
    labels = torch.arange(n, device="cuda", dtype=torch.int32) % k
    Y = torch.zeros(k, d, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        counts = skm.update(X, labels, Y)
        a, _, row = skm.assign(X, Y, labels)
    torch.cuda.synchronize()
    assert torch.equal(counts.cpu(), torch.bincount(labels.cpu(), minlength=k).int())
    assert row["ms_step"] > 0 and int(a.min()) >= 0 and int(a.max()) < k


# An assignment with a label outside [0, k) is refused and leaves the outputs as they are, also where they are the labels
# that came in: in a step that writes the caller's arrays itself, and in one that groups the points first (k >= 4096).
@pytest.mark.parametrize("n,d,k", [(500, 64, 10), (3000, 100, 37), (40_000, 32, 4100)])
def test_refused_labels_leave_the_outputs_as_they_are(skm, dg, n, d, k):  # noqa: F811
    import ctypes as C
    say("refused labels", n, d, k)
    L = skm.lib()
    vp = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
    X = dg.mixture(n, d, 20, 5, "linear", "cuda")
    Y = X[:k].contiguous()
    for bad in (k, -1):
        prev = torch.zeros(n, dtype=torch.int32, device="cuda")
        prev[n // 2] = bad
        kept = prev.clone()
        a = torch.full((n,), -9, dtype=torch.int32, device="cuda")
        dist = torch.full((n,), -3.0, device="cuda")
        torch.cuda.synchronize()
        assert L.skm_assign_ex(vp(X), n, d, vp(Y), k, vp(prev), 0, None, vp(a), vp(dist)) == -1
        assert L.skm_assign_ex(vp(X), n, d, vp(Y), k, vp(prev), 0, None, vp(prev), vp(dist)) == -1
        torch.cuda.synchronize()
        assert bool((a == -9).all()) and bool((dist == -3.0).all()) and torch.equal(prev, kept)
    # in place, with labels that are good
    prev = torch.zeros(n, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    assert L.skm_assign_ex(vp(X), n, d, vp(Y), k, vp(prev), 0, None, vp(prev), vp(dist)) == 0
    b, dist_b, _ = skm.assign(X, Y, torch.zeros(n, dtype=torch.int32, device="cuda"), opts=skm.FitOptions(R=skm.make_rotation(d, 0)))
    torch.cuda.synchronize()
    assert torch.equal(prev, b) and torch.equal(dist, dist_b)


# Several tiles to a workgroup, some of them done again in three products (poor incumbents in every third row tile): the tile
# after such a one starts in one product behind the first test like any other.  d' = 16: its second unit is already the
# first of one product.
@pytest.mark.parametrize("n,d,k,dp", [(30_000, 153, 1100, 16), (30_000, 208, 1100, 16), (30_000, 200, 1100, 32)])
def test_listed_tiles_behind_one_that_was_done_again(skm, orc, dg, n, d, k, dp):  # noqa: F811
    say("listed, done again", n, d, k, dp)
    rng = np.random.default_rng(n + d)
    X = dg.mixture(n, d, k // 3, 17, "embed").numpy()
    R = orc.random_rotation(d, 6)
    Y = X[rng.choice(n, k, replace=False)] + (0.01 * rng.standard_normal((k, d))).astype(np.float32)
    Xr, Yr = orc.rotate(X, R), orc.rotate(Y, R)
    prev = orc.assign_full(Xr, Yr)[0].astype(np.int32)
    poor = (np.arange(n) // 128) % 3 == 0
    prev[poor] = rng.integers(0, k, int(poor.sum()))
    near = rng.random(n) < 0.5                     # and half of the others an incumbent that is beaten
    prev[near & ~poor] = orc.assign_full(Xr[near & ~poor], Yr[: k // 2])[0]
    ref = orc.assign_pruned(Xr, Yr, prev, dp, EPS0, 0)
    for screen in (1, -1):
        a, dist, row = skm.assign(cuda(X), cuda(Y), cuda(prev), dp, skm.FitOptions(R=cuda(R), screen=screen))
        check_assignment(a.cpu().numpy(), ref.assign, Xr, Yr)
        same = a.cpu().numpy() == ref.assign
        assert np.abs(dist.cpu().numpy()[same] - ref.dist[same]).max() < 2e-5 * max(1.0, ref.dist.max())
        assert abs(row["completed"] - ref.enter[-1]) <= max(2, 1e-3 * ref.enter[-1])


# ... and through points of any length and alignment: four values a load, the last one to three of a row one by one.
@pytest.mark.parametrize("n,d,shift", [(30_001, 97, 0), (30_000, 98, 0), (20_000, 259, 0), (30_000, 100, 1), (9000, 2050, 0)])
def test_ground_truth_of_rows_of_any_length(skm, orc, dg, n, d, shift):  # noqa: F811
    say("ground truth, rows of any length", n, d, shift)
    X = dg.mixture(n, d, 300, 8, "embed").numpy()
    Q = dg.mixture(40, d, 300, 8, "embed", sample_seed=9).numpy()
    buf = torch.full((n * d + 4,), 3e4, device="cuda")   # (what lies beside the rows is not theirs)
    rows = buf[shift:shift + n * d].view(n, d)
    rows.copy_(cuda(X))
    check_ground_truth(skm.etr_ground_truth(rows, cuda(Q), 10).cpu().numpy(), orc.ground_truth(X, Q, 10), X, Q)


# Rows of any length and alignment: fp32 products, four values a load from any 4-byte boundary, the last ones of a row one by one
# where the length is no multiple of four.  n, d around the tiles of 128 and the slabs of 16.
@pytest.mark.parametrize("n,d", [(127, 61), (129, 63), (1, 65), (128, 66), (300, 67), (257, 95), (130, 97), (65, 127), (200, 129), (140, 495)])
def test_products_of_rows_of_any_length(skm, dg, n, d):  # noqa: F811
    say("rows of any length", n, d)
    X = dg.mixture(n, d, 5, 2, "embed").cuda()
    R = skm.make_rotation(d, 3)
    shifted = torch.empty(n * d + 3, device="cuda")
    shifted[3:] = X.reshape(-1)
    rows = shifted[3:].view(n, d)                      # (not 16-byte aligned)
    # the bound of the split form of aligned rows, to which these are held as well: halves of 22 bits a value and fp32 sums, 2^-21 of
    # every product and 2^-24 of the partial sums at each of d / 16 steps of 16, all bounded by the norms (Cauchy-Schwarz; rows
    # and columns have norm 1)
    bound = 2.0 ** -21 + (d / 16 + 16) * 2.0 ** -24
    for x in (X, rows):
        for transpose in (False, True):
            ref = X.double() @ (R.double().T.contiguous() if transpose else R.double())
            assert (skm.rotate(x, R, transpose).double() - ref).abs().max().item() < bound
    if n > 1:                                          # a row that is not a number stays by itself
        X[n // 2] = float("nan")
        out = skm.rotate(X, R)
        bad = torch.isnan(out).any(1)
        assert bool(bad[n // 2]) and int(bad.sum()) == 1


# ... and their products know nothing of the other rows: beside one row that is larger by 2^20, 2^40 or 2^60, smaller by 2^20, or
# not finite, every other row has the bits that it has without it.
@pytest.mark.parametrize("d,shift", [(495, 0), (495, 1), (129, 0), (97, 3), (256, 1)])
def test_products_beside_a_row_of_another_size(skm, dg, d, shift):  # noqa: F811
    n = 300
    R = skm.make_rotation(d, 3)
    buf = torch.empty(n * d + 4, device="cuda")
    X = buf[shift:shift + n * d].view(n, d)
    X.copy_(dg.mixture(n, d, 5, 2, "embed"))
    ref = [skm.rotate(X, R, transpose) for transpose in (False, True)]
    row = X[200].clone()
    others = torch.arange(n, device="cuda") != 200
    for factor in (2.0 ** 20, 2.0 ** 40, 2.0 ** 60, 2.0 ** -20, float("inf"), float("nan")):
        say("rows of another size", d, shift, factor)
        X[200] = row * factor
        for transpose in (False, True):
            out = skm.rotate(X, R, transpose)
            assert torch.equal(out[others], ref[transpose][others])
            if 2.0 ** -20 <= factor < float("inf"):
                assert torch.equal(out[200], ref[transpose][200] * factor)      # (scaling by a power of two is exact)
            else:
                assert not torch.isfinite(out[200]).any()


def test_ground_truth_beside_a_point_of_another_size(skm, orc, dg):  # noqa: F811
    n, d = 700, 495                                                 # (few points: the scores of all of them)
    X = dg.mixture(n, d, 5, 2, "embed").numpy()
    Q = dg.mixture(9, d, 5, 2, "embed", sample_seed=4).numpy()
    for factor in (2.0 ** 20, 2.0 ** 40):
        say("ground truth beside a large point", factor)
        far = X.copy()
        far[300] *= np.float32(factor)
        ref = ((Q[:, None].astype(np.float64) - far[None]) ** 2).sum(2).argsort(1, kind="stable")[:, :10]
        check_ground_truth(skm.etr_ground_truth(cuda(far), cuda(Q), 10).cpu().numpy(), ref, far, Q)


# Few clusters, thousands of rows that change between them: the lists of a cluster's rows are worked off several times in an
# update (768 to 1024 rows of each wavefront), chunks of labels with many matches and with none.
@pytest.mark.parametrize("n,d,k", [(60_000, 24, 2), (150_000, 64, 3), (40_000, 300, 5)])
def test_incremental_update_with_many_changes_in_few_clusters(skm, dg, n, d, k):  # noqa: F811
    say("many changes", n, d, k)
    X = dg.mixture(n, d, 40, 6, "linear").cuda()
    R = skm.make_rotation(d, 1)
    inc = skm.fit(X, k, 12, 4, skm.FitOptions(R=R, eps0=float("inf")))
    full = skm.fit(X, k, 12, 4, skm.FitOptions(R=R, eps0=float("inf"), full_update=True))
    few = [row["changed"] for row in inc.trace[1:] if 16 * row["changed"] <= n]
    assert inc.timing["inc_updates"] > 0 and (k > 2 or max(few) > 1600)
    # fp64 sums in another order, rounded to fp32: a near-tie may move a point, and with it two means by 1 / their size
    moved = int((inc.assign != full.assign).sum())
    assert moved <= 4
    assert (inc.centroids - full.centroids).abs().max().item() < 1e-6 + 8.0 * (moved + 1) * k / n * float(moved > 0)


# Sums of short lists of rows (fewer than 32 on average: four rows in flight, numbers in registers) and of long ones: the same order of
# sums, so the same bits.  Lists around the four wavefronts, their rows in flight, 64 numbers and a segment of 512 rows.
@pytest.mark.parametrize("d,shift", [(16, 0), (100, 1), (258, 0), (771, 0), (1024, 0)])
def test_update_with_short_lists(skm, dg, d, shift):  # noqa: F811
    say("short lists", d, shift)
    sizes = [0, 1, 3, 4, 5, 15, 16, 17, 31, 33, 63, 64, 65, 81, 127, 130, 511, 512, 513, 1040]
    n, k = sum(sizes), len(sizes)
    g = torch.Generator().manual_seed(d)
    buf = torch.empty(n * d + 4, device="cuda")
    X = buf[shift:shift + n * d].view(n, d)
    X.copy_(torch.randn(n, d, generator=g))
    labels = torch.repeat_interleave(torch.arange(k), torch.tensor(sizes))[torch.randperm(n, generator=g)].int().cuda()
    means = []
    for lists in (k, n // 32 + 1):                       # (the others are empty: fewer than 32 rows a list)
        Y = torch.zeros(lists, d, device="cuda")
        assert skm.update(X, labels, Y)[:k].tolist() == sizes
        means.append(Y[:k])
    assert n >= 32 * k and torch.equal(means[0], means[1])
    want = torch.zeros(k, d, dtype=torch.float64, device="cuda").index_add_(0, labels.long(), X.double())
    want /= torch.tensor(sizes, device="cuda").clamp_min(1)[:, None]
    assert float((means[1].double() - want).abs().max()) <= 2.0 ** -24 * float(want.abs().max()) + 1e-12   # (fp64 sums, rounded once)


# ... and of the rows that joined and left: few changes a cluster, and many clusters (below, one by one).
def test_incremental_update_with_few_changes_in_many_clusters(skm, dg):  # noqa: F811
    n, d, k = 120_000, 40, 6000
    say("few changes", n, d, k)
    X = dg.mixture(n, d, 3 * k, 6, "linear", "cuda")
    R = skm.make_rotation(d, 1)
    inc, full = (skm.fit(X, k, 6, 4, skm.FitOptions(R=R, eps0=float("inf"), full_update=f)) for f in (False, True))
    few = [row["changed"] for row in inc.trace[1:] if 8 * row["changed"] <= n]
    assert inc.timing["inc_updates"] > 0 and max(few) * 2 * k > 1 << 25       # (not the form for a handful of changes)
    # fp64 sums in another order, rounded to fp32: no near-tie of these rows hangs on that, so every list is the same
    assert torch.equal(inc.assign, full.assign)
    assert float((inc.centroids - full.centroids).abs().max()) < 1e-6 and float((inc.dist - full.dist).abs().max()) < 1e-5


# Rows of a host-resident fit that stay on the device between its passes: all of them with their tables, or as many whole
# batches as half of the free memory holds; the results are those of a fit that sends every row in every pass, bit by bit.
@pytest.mark.parametrize("n,d,k,room", [(140_000, 100, 40, "all"), (300_000, 64, 300, "all"), (280_000, 256, 30, "some")])
def test_host_resident_fit_keeps_what_fits(skm, dg, n, d, k, room):  # noqa: F811
    say("kept rows", n, d, k, room)
    X = dg.mixture(n, d, 60, 3, "embed")
    skm.release_memory()
    before = torch.cuda.mem_get_info()[0]
    sent = skm.fit_host(X, k, 3, 5, batch_rows=131_072)
    used = before - torch.cuda.mem_get_info()[0]       # the workspace, which the library keeps for the next call
    filler = None
    if room == "some":
        # free, without the kept workspace: one and a half batches of rotated rows, twice (half of it is taken)
        torch.cuda.empty_cache()
        leave = used + 3 * 131_072 * d * 4
        skm.release_memory()
        filler = torch.empty(torch.cuda.mem_get_info()[0] - leave, dtype=torch.uint8, device="cuda")
    kept = skm.fit_host(X, k, 3, 5)
    del filler
    torch.cuda.empty_cache()
    assert torch.equal(sent.assign, kept.assign) and torch.equal(sent.dist, kept.dist)
    assert torch.equal(sent.centroids, kept.centroids)
    assert [r["survivors"] for r in sent.trace] == [r["survivors"] for r in kept.trace]


# Tables stay with the rows only in a block that the library keeps between calls; here rows alone are such a block.
def test_host_resident_fit_keeps_rows_without_tables(skm, dg):  # noqa: F811
    n, d, k = 1_700_000, 256, 300
    say("kept rows without tables", n, d, k)
    Xh = dg.mixture(n, d, 60, 3, "embed", "cuda").cpu()
    assert n * 10 * d > 1 << 32 > n * 6 * d              # (with tables 10 bytes a value and more)
    R = skm.make_rotation(d, 2)
    used, fits = [], []
    for batch_rows in (131_072, 0):
        skm.release_memory()
        torch.cuda.empty_cache()
        before = torch.cuda.mem_get_info()[0]
        fits.append(skm.fit_host(Xh, k, 2, 5, batch_rows=batch_rows, opts=skm.FitOptions(R=R)))
        used.append(before - torch.cuda.mem_get_info()[0])
    assert abs(used[1] - used[0] - n * d * 4) < 1 << 26     # (a process keeps some more of its first calls)
    sent, kept = fits
    assert torch.equal(sent.assign, kept.assign) and torch.equal(sent.dist, kept.dist) and torch.equal(sent.centroids, kept.centroids)


# The room that is planned counts the blocks that the library keeps idle: where none of them is large enough and the device is full
# otherwise, they go back for it.
def test_host_resident_fit_takes_the_idle_blocks(skm, dg):  # noqa: F811
    n, d, k = 600_000, 256, 30
    say("kept rows from idle blocks", n, d, k)
    X = dg.mixture(n, d, 60, 3, "embed", "cuda")
    R = skm.make_rotation(d, 2)
    Xh = X.cpu()
    sent = skm.fit_host(Xh, k, 3, 5, batch_rows=131_072, opts=skm.FitOptions(R=R))
    torch.cuda.synchronize()
    skm.release_memory()
    blocks, labels = [], torch.arange(n, device="cuda", dtype=torch.int32)
    for many in (560_000, 580_000, 600_000):             # (updates of so many means: each a little too large for the block before)
        Y = X[:many].clone()
        torch.cuda.empty_cache()
        before = torch.cuda.mem_get_info()[0]
        skm.update(X, labels % many, Y)
        torch.cuda.empty_cache()
        blocks.append(before - torch.cuda.mem_get_info()[0])
    del X, Y, labels
    tables = n * 9 * d                                   # rows, split copies, prefix norms: 8.25 bytes a value and 128 a row
    assert min(blocks) > 1 << 30 and max(blocks) < tables and sum(blocks) < 4 << 30
    held = fill_device(tables // 2)
    before = torch.cuda.mem_get_info()[0]
    kept = skm.fit_host(Xh, k, 3, 5, opts=skm.FitOptions(R=R))
    after = torch.cuda.mem_get_info()[0]
    del held
    torch.cuda.empty_cache()
    assert after - before > 1 << 28                      # (idle blocks have gone, for less than they held)
    assert torch.equal(sent.assign, kept.assign) and torch.equal(sent.dist, kept.dist) and torch.equal(sent.centroids, kept.centroids)


# Iteration 1 goes through the one-product filter from 2048 clusters on, through the product of all pairs otherwise: the labels of
# a fit of one iteration on both sides of the line.
@pytest.mark.parametrize("n,k", [(16_383, 512), (16_384, 511), (16_384, 512), (16_500, 513), (4096, 2047), (4096, 2048)])
def test_iteration_one_on_both_sides_of_the_filter(skm, orc, dg, n, k):  # noqa: F811
    say("iteration 1", n, k)
    d = 48
    X = dg.mixture(n, d, 300, 8, "embed").numpy()
    R = orc.random_rotation(d, 2)
    fit = skm.fit(cuda(X), k, 1, 6, skm.FitOptions(R=cuda(R), final_assign=False))
    assert (fit.trace[0]["screen_dims"] > 0) == (k >= 2048)
    Xr = orc.rotate(X, R)
    Y0 = Xr[orc.sample_rows(6, n, k)]
    ref, _ = orc.assign_full(Xr, Y0)
    check_assignment(fit.assign.cpu().numpy(), ref, Xr, Y0, min_agree=0.999)


# Below that line the ties that rounding decides fall as they do without the filter: rows half way between two of the initial
# centroids, most of them the nearest two or three to within 1e-7.  One more such point on the other side is another fit.
@pytest.mark.parametrize("n,d,k", [(16_384, 96, 512), (20_001, 64, 777), (30_000, 256, 1024), (17_000, 100, 2047)])
def test_near_ties_of_iteration_one(skm, n, d, k):  # noqa: F811
    say("near-ties of iteration 1", n, d, k)
    g = torch.Generator().manual_seed(n + k)
    C = torch.nn.functional.normalize(torch.randn(k, d, generator=g), dim=1)
    near = torch.cdist(C, C).fill_diagonal_(9.0).argmin(1)          # every centroid's nearest one
    a = torch.randint(0, k, (n - k,), generator=g)
    X = torch.cat([C, 0.5 * (C[a] + C[near[a]])]).cuda()
    R = skm.make_rotation(d, 3)
    opts = dict(R=R, init_idx=range(k), final_assign=False)
    with_filter, without, forced = (skm.fit(X, k, 1, 1, skm.FitOptions(screen=s, **opts)) for s in (0, -1, 1))
    assert torch.equal(with_filter.assign, without.assign) and torch.equal(with_filter.centroids, without.centroids)
    assert not torch.equal(forced.assign, without.assign)           # (the rows do tell the two forms apart)


# A row that is no number gets a label like any other, on either side of the lines at which iteration 1 might change its form.
@pytest.mark.parametrize("n,k", [(16_400, 511), (16_400, 512), (20_000, 2047)])
def test_iteration_one_with_a_row_that_is_no_number(skm, dg, n, k):  # noqa: F811
    say("iteration 1, nan", n, k)
    d = 96
    X = dg.mixture(n, d, 300, 8, "embed", "cuda")
    opts = skm.FitOptions(R=skm.make_rotation(d, 3), init_idx=range(k), final_assign=False)
    want = skm.fit(X, k, 1, 1, opts)
    X[n - 7] = float("nan")
    got = skm.fit(X, k, 1, 1, opts)
    keep = torch.arange(n, device="cuda") != n - 7
    assert torch.equal(got.assign[keep], want.assign[keep]) and 0 <= int(got.assign[n - 7]) < k


def fill_device(leave):
    """Tensors that take the device's memory but for `leave` bytes (and what torch keeps)."""
    torch.cuda.empty_cache()
    held, piece = [], None
    while (room := torch.cuda.mem_get_info()[0] - leave) > 1 << 22:
        piece = room if piece is None else min(piece, room)
        try:
            held.append(torch.empty(piece, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            piece //= 2
    return held


# The block that an exact assignment plans holds all of its buffers, the split copy of the centroids in whole units of 32
# dimensions among them: a call like the one before finds all of its memory in the block that the library has kept.
@pytest.mark.parametrize("d", [40, 48])
def test_exact_assignment_in_the_block_of_the_call_before(skm, dg, d):  # noqa: F811
    say("exact assignment in a kept block", d)
    n, k = 1000, 200_000
    Y = dg.mixture(k, d, 50, 3, "linear", "cuda")
    X = (Y[:n] + 0.001).contiguous()
    skm.release_memory()
    a, dist = skm.assign_exact(X, Y)
    b, dist_b = skm.assign_exact(X, Y)
    held = fill_device(40 << 20)                        # (less than the split copy of the centroids)
    b, dist_b = skm.assign_exact(X, Y)
    del held
    torch.cuda.empty_cache()
    assert torch.equal(a, b) and torch.equal(dist, dist_b)


# Nearest centroids with the rows in registers (aligned rows of 32 to 128 dimensions, more than 192 columns or 448 beyond 64
# dimensions, four tiles of 256 x 64 to a CU): every number of 16-dimension steps, rows and columns that end inside a tile,
# ranges that begin and end inside a row tile; against the oracle and, where the old form stands beside it, bit by bit.
@pytest.mark.parametrize("n,d,k", [(66_000, 32, 257), (40_001, 48, 449), (33_000, 64, 513), (25_700, 80, 700), (36_000, 96, 511),
                                   (20_003, 112, 900), (18_000, 128, 1000), (16_384, 100, 1024), (90_000, 36, 193)])
def test_exact_assignment_with_rows_in_registers(skm, orc, dg, n, d, k):  # noqa: F811
    say("rows in registers", n, d, k)
    X = dg.mixture(n, d, 300, 5, "embed")
    Y = dg.mixture(k, d, 300, 5, "embed", sample_seed=3)
    a, dist = skm.assign_exact(X.cuda(), Y.cuda())
    few = torch.randperm(n, generator=torch.Generator().manual_seed(1))[:3000].sort().values
    few[-1] = n - 1
    ao, do = orc.assign_full(X[few].numpy().astype(np.float64), Y.numpy().astype(np.float64))
    check_assignment(a[few.cuda()].cpu().numpy(), ao, X[few].numpy(), Y.numpy(), min_agree=0.999)
    # a call with few rows takes the tiles of 128 x 128, which add the products in the same order
    part = slice(n // 3, n // 3 + 1500)
    scale = X.abs().max()
    rows = torch.cat([X[part], torch.full((1, d), float(scale))])    # (the same magnitude bound: the same halves)
    b, dist_b = skm.assign_exact(rows.cuda(), Y.cuda())
    assert torch.equal(a[part], b[:-1]) and torch.equal(dist[part], dist_b[:-1])


# ... and in the order of the 256 x 256 tiles where the product would take those (whole slabs of 32 dimensions, 512 tiles).
@pytest.mark.parametrize("n,d,k", [(140_000, 64, 450), (70_000, 96, 768), (80_001, 128, 500)])
def test_rows_in_registers_in_the_order_of_wide_tiles(skm, dg, n, d, k):  # noqa: F811
    say("rows in registers, wide tiles", n, d, k)
    X, Y = dg.mixture(n, d, 300, 5, "embed", "cuda"), dg.mixture(k, d, 300, 5, "embed", "cuda", sample_seed=3)
    X[: k] = 0.5 * (Y + Y.roll(1, 0))                                 # (rows for which the order decides)
    a, dist = skm.assign_exact(X, Y)
    few = torch.cat([X[:3000], torch.full((1, d), float(X.abs().max()), device="cuda")])     # (the same bound: the same halves)
    skm.debug_gemm_config(tile256=1)
    try:
        b, dist_b = skm.assign_exact(few, Y)
    finally:
        skm.debug_gemm_config()
    assert torch.equal(a[:3000], b[:-1]) and torch.equal(dist[:3000], dist_b[:-1])


def test_rows_in_registers_that_are_no_numbers(skm, dg):  # noqa: F811
    say("rows in registers, nan and inf")
    n, d, k = 70_000, 64, 300
    X, Y = dg.mixture(n, d, 100, 5, "embed").cuda(), dg.mixture(k, d, 100, 5, "embed", sample_seed=3).cuda()
    want = skm.assign_exact(X, Y)[0]
    X[5000] = float("nan")
    got = skm.assign_exact(X, Y)[0]
    keep = torch.arange(n, device="cuda") != 5000
    assert torch.equal(got[keep], want[keep]) and int(got[5000]) == 0


# Thresholds kept from the step before: of all points once no label changes any more, of those in untouched clusters while few
# do (rows of some length, at most a quarter as many changes as clusters).  Every row length that the pass is made for.
@pytest.mark.parametrize("n,d,k", [(66_000, 256, 300), (33_500, 500, 400), (24_000, 700, 500), (17_000, 1000, 400), (12_000, 1500, 300),
                                   (9000, 2000, 220), (20_000, 64, 100)])
def test_thresholds_kept_from_the_step_before(skm, dg, n, d, k):  # noqa: F811
    say("kept thresholds", n, d, k)
    X = dg.mixture(n, d, 2 * k, 4, "embed").cuda()
    R = skm.make_rotation(d, 2)
    fit = skm.fit(X, k, 14, 3, skm.FitOptions(R=R))
    changed = [row["changed"] for row in fit.trace[:-1]]
    assert 0 in changed and (n * d < 1 << 24 or any(0 < c <= k // 4 for c in changed))
    full = skm.fit(X, k, 14, 3, skm.FitOptions(R=R, full_update=True))        # (takes every threshold again)
    assert torch.equal(fit.assign, full.assign) and [r["survivors"] for r in fit.trace] == [r["survivors"] for r in full.trace]
    # fp32 sums of d squares in either form: d 2^-24 of the sum at most
    assert ((fit.dist - full.dist).abs() <= 2 * d * 2.0 ** -24 * full.dist + 1e-12).all()
    direct = ((X.double() - fit.centroids.double()[fit.assign.long()]) ** 2).sum(1)
    # ... and the rotated copies of rows and centroids are rounded to fp32: 2^-23 (||x|| + ||y||) per row (norms of 1 at most)
    assert ((fit.dist.double() - direct).abs() <= (2 * d * 2.0 ** -24) * direct + 8 * 2.0 ** -21 * direct.sqrt() + 1e-9).all()


# The pass that closes a step: 1024 points a workgroup, 8192 from 2^18 on; more workgroups than its 1024 threads from 8 388 609
# points on; sizes read ahead up to 1024 clusters (4096 from 2^18 points), the rest in a loop.
@pytest.mark.parametrize("n,d,k", [(1, 16, 1), (255, 20, 3), (1023, 16, 7), (1025, 16, 1024), (4097, 32, 1025), (20_000, 64, 2500),
                                   (262_143, 16, 10), (262_145, 16, 5000), (8_388_609, 16, 5)])
def test_what_the_closing_pass_reports(skm, n, d, k):  # noqa: F811
    say("closing pass", n, d, k)
    g = torch.Generator("cuda").manual_seed(n + k)
    X = torch.randn(n, d, generator=g, device="cuda")
    Y = X[torch.randperm(n, generator=g, device="cuda")[:k]].clone()
    prev = torch.randint(0, k, (n,), generator=g, device="cuda", dtype=torch.int32)
    a, dist, row = skm.assign(X, Y, prev, 16, skm.FitOptions(R=torch.eye(d, device="cuda")))
    assert row["changed"] == int((a != prev).sum()) and int(a.min()) >= 0 and int(a.max()) < k
    assert row["nempty"] == int((torch.bincount(a.long(), minlength=k) == 0).sum())
    # fp64 sums of the same fp32 values in another order: n 2^-53 of the sum at most
    assert row["objective"] == pytest.approx(float(dist.double().sum()), rel=n * 2.0 ** -53, abs=1e-300)


# The split copies and the planes of hi halves lie in pairs of rows, the plane in units of 32 dimensions: odd numbers of points
# and centroids, rows whose last unit is half full, first tests at odd and even multiples of 16 and behind the whole row, and
# tables written 16 and 64 points at a time.  What the filter and the one-product tiles leave out must not show.
@pytest.mark.parametrize("n,d,k,dp", [(1, 48, 1, 16), (127, 64, 255, 32), (1025, 80, 301, 48), (1026, 176, 257, 80), (2047, 336, 513, 96),
                                      (3001, 400, 259, 400), (513, 1040, 300, 112), (90_001, 64, 300, 16), (83_003, 112, 261, 32)])
def test_operands_in_pairs_of_rows(skm, orc, dg, n, d, k, dp):  # noqa: F811
    say("pairs of rows", n, d, k, dp)
    rng = np.random.default_rng(n + 3 * k)
    X = dg.mixture(n, d, 40, n + d, "linear" if d < 512 else "embed").numpy()
    R = orc.random_rotation(d, 7)
    Y = X[rng.integers(0, n, k)] + (0.01 * rng.standard_normal((k, d))).astype(np.float32)
    Xr, Yr = orc.rotate(X, R), orc.rotate(Y, R)
    prev = rng.integers(0, k, n).astype(np.int32)
    prev[::2] = orc.assign_full(Xr[::2], Yr)[0]
    runs = {}
    for screen in (-1, 1):
        a, dist, row = skm.assign(cuda(X), cuda(Y), cuda(prev), dp, skm.FitOptions(R=cuda(R), screen=screen))
        check = orc.assign_pruned(Xr, Yr, prev, dp, EPS0, 0) if n < 4000 else None
        if check is not None:
            check_assignment(a.cpu().numpy(), check.assign, Xr, Yr)
            assert abs(row["survivors"] - (n * (k - 1) - check.pruned_first)) <= max(2, 1e-3 * n * k)
        runs[screen] = (a, dist, row["survivors"], row["completed"])
    (a0, d0, s0, c0), (a1, d1, s1, c1) = runs[-1], runs[1]
    assert s0 == s1 and c0 == c1
    differ = a0 != a1   # (a pair finishes in a tile of split products or, handed over, in fp32: near-ties may fall either way)
    assert int(differ.sum()) <= 1e-3 * n
    assert ((d0 - d1).abs()[~differ] <= 2e-5 * max(1.0, float(d0.max()))).all()


# Candidates of iteration 1 dealt out to their points: from 2^26 elements on, rows of 128 dimensions or more, four slots a point
# up to 768 clusters and eight above, what does not fit left to the list (points of few components, and of one, have dozens of
# candidates), one launch of all blocks and several.
@pytest.mark.parametrize("n,d,k,components", [(66_001, 1024, 600, 1500), (66_000, 1024, 600, 20), (90_001, 752, 300, 4), (141_001, 480, 2100, 3000),
                                              (141_000, 480, 2100, 60), (524_289, 128, 513, 900), (33_003, 2050, 9000, 9000)])
def test_candidates_dealt_out_to_their_points(skm, dg, n, d, k, components):  # noqa: F811
    say("dealt out", n, d, k, components)
    X = dg.mixture(n, d, components, 3, "embed").cuda()
    idx = np.random.default_rng(n).choice(n, k, replace=False)
    R = torch.eye(d, device="cuda")
    runs = [skm.fit(X, k, 1, 1, skm.FitOptions(R=R, init_idx=idx, final_assign=False, screen=s)) for s in (1, -1)]
    assert runs[0].trace[0]["gather_pairs"] >= n and runs[1].trace[0]["gather_pairs"] == 0
    a, b = (r.assign.long() for r in runs)
    Y = X[torch.as_tensor(idx, device="cuda")].double()
    # fp32 sums of d squares, and the split product's search: d 2^-24 of the sum, and 2^-20 of the norms' product (norms of 1)
    for r in range(0, n, 20_000):
        x = X[r:r + 20_000].double()
        da, db = (((x - Y[l[r:r + 20_000]]) ** 2).sum(1) for l in (a, b))
        assert (da <= db * (1 + 2 * d * 2.0 ** -24) + 2.0 ** -20).all() and (db <= da * (1 + 2 * d * 2.0 ** -24) + 2.0 ** -20).all()
        assert ((runs[0].dist[r:r + 20_000].double() - da).abs() <= 2 * d * 2.0 ** -24 * da + 1e-12).all()


# The lists of a row tile's columns are put together 8192 columns at a time: at that number, one more, several times as many, and
# tiles of which every column, few and hardly any are listed.
@pytest.mark.parametrize("good", [0, 1])     # the incumbents: the nearest centroids, or any
@pytest.mark.parametrize("n,d,k,dp", [(300, 64, 8192, 16), (257, 64, 8193, 32), (129, 80, 25_000, 48)])
def test_lists_of_many_columns(skm, dg, n, d, k, dp, good):  # noqa: F811
    say("lists", n, d, k, dp, good)
    X, Y = dg.mixture(n, d, 20, 5, "linear").cuda(), dg.mixture(k, d, 20, 5, "linear", sample_seed=9).cuda()
    g = torch.Generator("cuda").manual_seed(k)
    prev = skm.assign_exact(X, Y)[0] if good else torch.randint(0, k, (n,), generator=g, device="cuda", dtype=torch.int32)
    R = torch.eye(d, device="cuda")
    (a, da, ra), (b, db, rb) = (skm.assign(X, Y, prev, dp, skm.FitOptions(R=R, screen=s)) for s in (1, -1))
    assert ra["listed_tiles"] > 0 and ra["survivors"] == rb["survivors"] and ra["completed"] == rb["completed"]
    # (a pair finishes in a tile of split products or, handed over, in fp32: near-ties may fall either way, by d 2^-24 and 2^-20)
    dist = [((X.double() - Y.double()[l.long()]) ** 2).sum(1) for l in (a, b)]
    assert ((dist[0] - dist[1]).abs() <= 2 * d * 2.0 ** -24 * dist[1] + 2.0 ** -19 * float((X ** 2).sum(1).max())).all()


# The exact assignment through the one-product search: from 2048 centroids, rows of more than 128 dimensions and 2^34 multiply-adds
# on, 2^18 rows at a time; ragged and unaligned rows through a padded copy.
@pytest.mark.parametrize("n,d,k,shift", [(16_385, 256, 4100, 0), (262_145, 136, 2048, 0), (20_001, 515, 2100, 0), (9001, 400, 5001, 1),
                                         (262_144 + 16_000, 144, 2050, 1)])
def test_exact_assignment_through_the_search(skm, dg, n, d, k, shift):  # noqa: F811
    say("exact search", n, d, k, shift)
    X, Y = dg.mixture(n, d, 2 * k, 5, "embed").cuda(), dg.mixture(k, d, 2 * k, 5, "embed", sample_seed=3).cuda()
    if shift:
        at = torch.empty(n * d + 1, device="cuda")
        at[1:] = X.reshape(-1)
        X = at[1:].view(n, d)
    a, dist = skm.assign_exact(X, Y)
    alone = skm.assign_exact(X[:500], Y)[0]                     # (few rows: three products)
    for r in range(0, n, 16_384):
        x = X[r:r + 16_384].double()
        D = (x * x).sum(1, keepdim=True) - 2 * x @ Y.double().T + (Y.double() ** 2).sum(1)
        own = ((x - Y.double()[a[r:r + 16_384].long()]) ** 2).sum(1)
        # fp32 sums of d squares: d 2^-24 of the sum (and 2^-45 for the fp64 form of the matrix D, norms of 1)
        assert (own <= D.min(1).values * (1 + 2 * d * 2.0 ** -24) + 2.0 ** -45).all()
        assert ((dist[r:r + 16_384].double() - own).abs() <= 2 * d * 2.0 ** -24 * own + 1e-12).all()
    assert int((alone != a[:500]).sum()) <= 1


def test_exact_search_that_has_nothing_to_show(skm, dg):  # noqa: F811
    """Rows that are no numbers, and centroids that are all the same, take the other form: labels as for few rows."""
    n, d, k = 40_000, 256, 2100
    X, Y = dg.mixture(n, d, 500, 5, "embed").cuda(), dg.mixture(k, d, 500, 5, "embed", sample_seed=3).cuda()
    want, dist = skm.assign_exact(X, Y)
    X[7777] = float("nan")
    got, dist_got = skm.assign_exact(X, Y)
    keep = torch.arange(n, device="cuda") != 7777
    assert int((got[keep] != want[keep]).sum()) <= 1e-3 * n and int(got[7777]) == int(skm.assign_exact(X[7700:7800], Y)[0][77])
    same = got == want
    assert ((dist_got - dist)[same].abs() <= 4 * d * 2.0 ** -24 * dist[same] + 1e-12).all()
    X[7777] = X[0]
    Y[:] = Y[0].clone()
    assert int(skm.assign_exact(X, Y)[0].abs().max()) == 0


# Rows to a batch of the search follow from the bytes of its buffers: long rows go in several batches, whose block is one that the
# library keeps for the next call.
@pytest.mark.parametrize("n,d,k", [(262_200, 1401, 2048), (140_000, 2112, 2050)])
def test_exact_search_in_batches_of_long_rows(skm, dg, n, d, k):  # noqa: F811
    say("exact search, long rows", n, d, k)
    X, Y = dg.mixture(n, d, 2 * k, 5, "embed", "cuda"), dg.mixture(k, d, 2 * k, 5, "embed", "cuda", sample_seed=3)
    skm.release_memory()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    a, dist = skm.assign_exact(X, Y)
    assert (1 << 30) < before - torch.cuda.mem_get_info()[0] < (1 << 31) + (1 << 25)     # (labels and distances: 2 MB)
    Yd = Y.double()
    y2 = (Yd * Yd).sum(1)
    for r in range(0, n, 16_384):
        x = X[r:r + 16_384].double()
        D = (x * x).sum(1, keepdim=True) - 2 * x @ Yd.T + y2
        own = ((x - Yd[a[r:r + 16_384].long()]) ** 2).sum(1)
        # fp32 sums of d squares: d 2^-24 of the sum (and 2^-45 for the fp64 form of the matrix D, norms of 1)
        assert (own <= D.min(1).values * (1 + 2 * d * 2.0 ** -24) + 2.0 ** -45).all()
        assert ((dist[r:r + 16_384].double() - own).abs() <= 2 * d * 2.0 ** -24 * own + 1e-12).all()


# A row that is no number sends its own batch to the product of all pairs, not the others: rows half way between two centroids,
# whose nearest one is a matter of rounding, have the labels and distances that they have without it.
@pytest.mark.parametrize("with_dist", [True, False])
def test_exact_search_with_one_batch_that_fails(skm, with_dist):  # noqa: F811
    n, d, k = (1 << 18) + 1000, 144, 2048
    say("exact search, one batch fails", n, d, k, with_dist)
    g = torch.Generator("cuda").manual_seed(5)
    Y = torch.nn.functional.normalize(torch.randn(k, d, generator=g, device="cuda"), dim=1)
    near = torch.cdist(Y, Y).fill_diagonal_(9.0).argmin(1)
    a = torch.randint(0, k, (n,), generator=g, device="cuda")
    X = 0.5 * (Y[a] + Y[near[a]])

    def run(x):
        if with_dist:
            return skm.assign_exact(x, Y)
        labels = torch.empty(len(x), dtype=torch.int32, device="cuda")
        st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert skm.lib().skm_assign_exact(ctypes.c_void_p(x.data_ptr()), len(x), d, ctypes.c_void_p(Y.data_ptr()), k, st,
                                          ctypes.c_void_p(labels.data_ptr()), None) == 0
        return labels, None

    want, dist = run(X)
    few = run(X[:50_000])[0]                              # (too few rows for the search)
    assert not torch.equal(few, want[:50_000])            # (the rows do tell the two forms apart)
    X[n - 5] = float("nan")
    got, dist_got = run(X)
    first = slice(0, 1 << 18)
    assert torch.equal(got[first], want[first]) and (not with_dist or torch.equal(dist_got[first], dist[first]))
    rest = torch.arange(1 << 18, n, device="cuda")
    rest = rest[rest != n - 5]
    own = lambda l: ((X[rest].double() - Y.double()[l[rest].long()]) ** 2).sum(1)  # noqa: E731
    # split products and norms of 1: 2^-20 of a distance either way
    assert int(got[n - 5]) == 0 and bool(((own(got) - own(want)).abs() <= 2.0 ** -18).all())


# A step after one that cut a third to a half of the pairs lists every column without asking the filter, and multiplies in one
# product behind the first test: with 1200 tiles or more, and a test behind 95 % of the row.  Counts and labels are those of the
# dense tiles.
@pytest.mark.parametrize("n,d,k,components,recipe,lists", [(144_442, 1536, 1198, 3594, "embed", True), (72_645, 1024, 714, 2856, "embed", True),
                                                           (98_724, 768, 2009, 8036, "embed", True), (45_553, 768, 433, 1515, "embed", False),
                                                           (57_350, 1216, 1561, 4683, "linear", False)])
def test_every_column_listed(skm, dg, n, d, k, components, recipe, lists):  # noqa: F811
    say("every column", n, d, k, components)
    X = dg.mixture(n, d, components, 3, recipe, "cuda")
    R = skm.make_rotation(d, 2)
    fit, dense = (skm.fit(X, k, 3, 5, skm.FitOptions(R=R, screen=s)) for s in (0, -1))
    frac = [row["prune_frac"] for row in fit.trace]
    steps = [t for t in range(2, len(frac)) if 0.33 <= frac[t - 1] < 0.5]
    say("every column: pairs cut", frac)
    assert steps
    for t in steps:
        full, rest = divmod(k, 256)
        assert fit.trace[t]["listed_tiles"] == lists * -(-n // 128) * (2 * full + (rest > 0) + (rest > 128)) and dense.trace[t]["listed_tiles"] == 0
    for a, b in zip(fit.trace, dense.trace):   # (a near-tie that falls the other way moves a point)
        assert abs(a["survivors"] - b["survivors"]) <= 1e-4 * max(b["survivors"], n) and abs(a["completed"] - b["completed"]) <= 2 + 1e-3 * b["completed"]
    assert int((fit.assign != dense.assign).sum()) <= 2e-4 * n


# A step of poor incumbents through the listed tiles (most pairs survive, a tile is done again in three products and finished
# where it stands): a row's least distance is found in LDS, for the last, narrower list tile and the last rows too.
@pytest.mark.parametrize("n,d,k", [(40_001, 96, 300), (30_007, 160, 257), (35_000, 64, 386), (33_000, 112, 4099)])
def test_listed_tiles_that_finish_many_pairs(skm, n, d, k):  # noqa: F811
    say("listed tiles finished", n, d, k)
    g = torch.Generator().manual_seed(n)
    X = torch.randn(n, d, generator=g).cuda()
    Y = X[:k] + 0.1 * torch.randn(k, d, generator=g).cuda()
    prev = torch.randint(0, k, (n,), generator=g).int().cuda()
    prev[: n // 2] = 0     # the many rows of one cluster share their row tiles with one incumbent
    R = skm.make_rotation(d, 4)
    (a, da, ra), (c, dc, rc) = (skm.assign(X, Y, prev, opts=skm.FitOptions(R=R, screen=s)) for s in (1, -1))
    assert ra["listed_tiles"] > 0 and rc["listed_tiles"] == 0 and rc["completed"] > n * k // 8
    assert ra["survivors"] == rc["survivors"] and abs(ra["completed"] - rc["completed"]) <= 2 + 1e-5 * rc["completed"]
    assert int((a != c).sum()) <= 2e-4 * n     # (near-ties of two roundings)
    assert bool(((da - dc).abs() <= 2.0 ** -18 * (X.norm(dim=1) + Y.norm(dim=1).max()) ** 2).all())


# A step on its own orders its points by the class of their threshold, then by label: thresholds with a long tail, all of them
# alike, none above zero, a tail larger than half, and clusters of several row tiles (which have an order of their own inside).
# Counts, labels and distances are those of the points in the caller's order, and the same from run to run.
@pytest.mark.parametrize("n,d,k,form", [(33_001, 200, 4100, "tail"), (33_001, 200, 4100, "most"), (40_000, 64, 4096, "alike"),
                                        (32_768, 80, 4096, "zero"), (530_000, 48, 4097, "tail")])
def test_points_in_the_order_of_their_thresholds(skm, dg, n, d, k, form):  # noqa: F811
    say("threshold classes", n, d, k, form)
    g = torch.Generator().manual_seed(n + d)
    Y = dg.mixture(k, d, 64, 3, "embed").cuda()
    lab = torch.randint(0, k, (n,), generator=g).cuda()
    X = Y[lab].clone()
    if form == "alike":
        X[:, 0] += 0.25
    elif form != "zero":
        X += 0.02 * torch.randn(n, d, generator=g).cuda()
    prev = lab.int()
    if form in ("tail", "most"):
        far = torch.rand(n, generator=g).cuda() < (0.02 if form == "tail" else 0.7)
        prev = torch.where(far, torch.randint(0, k, (n,), generator=g).int().cuda(), prev)
    R = skm.make_rotation(d, 4)
    runs = [skm.assign(X, Y, prev, opts=skm.FitOptions(R=R, screen=s)) for s in (0, 0, -1)]
    (a, da, ra), (b, db, rb), (c, dc, rc) = runs
    assert torch.equal(a, b) and torch.equal(da, db) and ra["survivors"] == rb["survivors"]
    assert ra["listed_tiles"] > 0 and rc["listed_tiles"] == 0
    assert abs(ra["survivors"] - rc["survivors"]) <= 1e-5 * max(rc["survivors"], n)
    # a label that differs is a near-tie: the rounding of a split product, 2^-20 of the norms, either way
    bound = 2.0 ** -19 * (X.double().norm(dim=1) + Y.double().norm(dim=1).max()) ** 2
    moved = a != c
    exact = lambda l: ((X.double() - Y.double()[l.long()]) ** 2).sum(1)  # noqa: E731
    assert int(moved.sum()) <= 1e-3 * n and bool(((exact(a) - exact(c)).abs() <= bound)[moved].all())
    assert bool(((da.double() - exact(a)).abs() <= bound).all())


# The same from 2048 centroids on, where there are 2^40 products: with a tail the points are regrouped and the columns listed,
# without one the step stays as it is (all but the incumbent of a point cut: nothing to list).
@pytest.mark.parametrize("tail", [True, False])
def test_order_of_thresholds_with_fewer_centroids(skm, dg, tail):  # noqa: F811
    n, d, k = 4_194_400, 120, 2049
    say("fewer centroids", n, d, k, tail)
    g = torch.Generator(device="cuda").manual_seed(7)
    Y = dg.mixture(k, d, 64, 3, "embed").cuda()
    prev = torch.randint(0, k, (n,), generator=g, device="cuda").int()
    X = Y[prev.long()] + 0.02 * torch.randn(n, d, generator=g, device="cuda")
    if tail:
        prev = torch.where(torch.rand(n, generator=g, device="cuda") < 0.02, torch.randint(0, k, (n,), generator=g, device="cuda").int(), prev)
    R = skm.make_rotation(d, 4)
    (a, da, ra), (c, dc, rc) = (skm.assign(X, Y, prev, opts=skm.FitOptions(R=R, screen=s)) for s in (0, -1))
    assert (ra["listed_tiles"] > 0) == tail and rc["listed_tiles"] == 0
    assert abs(ra["survivors"] - rc["survivors"]) <= 1e-5 * max(rc["survivors"], n)
    bound = 2.0 ** -19 * (X.norm(dim=1).max() + Y.norm(dim=1).max()) ** 2     # as above
    assert int((a != c).sum()) <= 1e-3 * n and float((da - dc).abs().max()) <= 2 * float(bound)


# ... and where there is no memory for the regrouped copy the step is served without it.
def test_fewer_centroids_without_memory_for_the_order(skm, dg):  # noqa: F811
    n, d, k = 1_050_000, 512, 2052
    say("fewer centroids, a full device", n, d, k)
    g = torch.Generator(device="cuda").manual_seed(7)
    Y = dg.mixture(k, d, 64, 3, "embed", "cuda")
    prev = torch.randint(0, k, (n,), generator=g, device="cuda").int()
    X = Y[prev.long()] + 0.02 * torch.randn(n, d, generator=g, device="cuda")
    prev = torch.where(torch.rand(n, generator=g, device="cuda") < 0.02, torch.randint(0, k, (n,), generator=g, device="cuda").int(), prev)
    opts = skm.FitOptions(R=skm.make_rotation(d, 4), own_workspace=True)
    a, da, ra = skm.assign(X, Y, prev, opts=opts)
    skm.release_memory()
    # a call's memory but for half of the copy (a fit's is a few ten MB more)
    held = fill_device(skm.workspace_bytes(n, d, k) - n * d * 2)
    c, dc, rc = skm.assign(X, Y, prev, opts=opts)
    del held
    torch.cuda.empty_cache()
    assert ra["listed_tiles"] > 0 and rc["listed_tiles"] == 0
    assert abs(ra["survivors"] - rc["survivors"]) <= 1e-5 * max(rc["survivors"], n)
    bound = 2.0 ** -19 * (X.norm(dim=1).max() + Y.norm(dim=1).max()) ** 2     # as above
    assert int((a != c).sum()) <= 1e-3 * n and float((da - dc).abs().max()) <= 2 * float(bound)


# Tiles are dealt out to the XCDs in runs of 8 (below 2048 tiles) to 128 (from 16 384 on), eight runs a round, and what does not fill
# a round in eighths.  With a threshold that drops nothing every pair is finished, so a tile left out, or done in another's place,
# shows in the labels.  Tiles of listed columns: one a row tile here; the others are narrow: two.
@pytest.mark.parametrize("screen", [-1, 1])
@pytest.mark.parametrize("tiles", [1, 31, 63, 64, 65, 127, 129, 1023, 1024, 1025, 2049, 16393])
def test_tiles_dealt_out_in_runs(skm, tiles, screen):  # noqa: F811
    say("runs", tiles, screen)
    n, d, k = 128 * tiles - 3, 32, 256
    g = torch.Generator().manual_seed(tiles)
    X, Y = torch.randn(n, d, generator=g), torch.randn(k, d, generator=g)
    near = []
    for x in X.double().split(1 << 16):      # (all of the largest case at once are 4.3 GB a matrix)
        near.append(((x ** 2).sum(1)[:, None] + (Y.double() ** 2).sum(1)[None] - 2.0 * x @ Y.double().T).topk(2, 1, largest=False))
    D, want = (torch.cat(p) for p in zip(*near))
    prev = torch.randint(0, k, (n,), generator=g, dtype=torch.int32)
    a, dist, row = skm.assign(X.cuda(), Y.cuda(), prev.cuda(), 16, skm.FitOptions(rotate=False, screen=screen, eps0=100.0))
    assert (row["listed_tiles"] > 0) == (screen == 1)
    clear = D[:, 1] - D[:, 0] > 1e-4 * D[:, 0]      # fp32 distances of 22-bit products
    assert torch.equal(a.cpu()[clear].long(), want[clear, 0])
    assert float(((dist.cpu().double() - D[:, 0]).abs() / D[:, 0]).max()) < 1e-4


# A fit regroups its points by quarters of their distances and by label (by label alone below 2^34 products a step), and again once the
# labels have moved on where the rows are its own (rows that are not 16-byte aligned are copied); a caller's rows are regrouped
# once.  Behind an update from the changed points alone their order is made for it, by counting (n >= 8 k, k <= 8192) or by
# scattering.  Both fits add the same fp64 sums in another order.  Clusters of a few points and of several row tiles (those
# have an order of their own inside).
def regroupings(trace, n, k, iters):
    """Iterations in which the rule regroups the points again, each with the changed share behind which it does."""
    out, moved, tiles = [], 0, (n + 127) // 128 * ((k + 127) // 128)
    for t in range(4, iters + 1):
        before = trace[t - 2]
        moved += before["changed"]
        listed = before["listed_tiles"] / tiles or 1.0
        if 20 * moved >= n and 0.20 <= before["prune_frac"] < 0.98 and (iters - t + 2) * k * moved * listed >= 1500 * n:
            out.append((t, before["changed"] / n))
            moved = 0
    return out


@pytest.mark.parametrize("n,d,k,iters,comps", [(33_000, 256, 2100, 12, 4), (140_000, 256, 1024, 30, 4), (300_001, 64, 1024, 30, 4),
                                               (140_000, 64, 1024, 30, 4), (20_000, 64, 1024, 30, 4), (33_000, 64, 4200, 20, 2),
                                               (150_000, 64, 9000, 20, 4)])
def test_points_of_a_fit_regrouped_again(skm, dg, n, d, k, iters, comps):  # noqa: F811
    say("regrouped again", n, d, k, iters)
    X = dg.mixture(n, d, comps * k, 3, "embed", "cuda")
    own = torch.empty(n * d + 1, device="cuda")[1:].view(n, d).copy_(X)
    opts = skm.FitOptions(rotate=False)
    a, b, c = (skm.fit(x, k, iters, 5, opts) for x in (X, own, own))
    assert torch.equal(b.assign, c.assign) and torch.equal(b.centroids, c.centroids) and torch.equal(b.dist, c.dist)
    for ra, rb in zip(a.trace, b.trace):
        assert abs(ra["survivors"] - rb["survivors"]) <= 1e-4 * max(ra["survivors"], n)
    assert sum(r["listed_tiles"] for r in b.trace) < sum(r["listed_tiles"] for r in a.trace)
    # the first is in iteration 3; some later one lies behind an update of the changed points alone
    assert any(share <= 1 / 8 for _, share in regroupings(b.trace, n, k, iters))
    assert float((a.centroids - b.centroids).norm() / a.centroids.norm()) < 1e-4
    assert float((a.assign != b.assign).float().mean()) <= 1e-3
    # labels and distances belong to the points in the caller's order
    exact = ((X.double() - b.centroids.double()[b.assign.long()]) ** 2).sum(1)
    assert float((b.dist.double() - exact).abs().max()) <= 2.0 ** -18 * float(X.norm(dim=1).max() + b.centroids.norm(dim=1).max()) ** 2


# ... not where the steps have little left to save: the labels of a mixture with fewer components than clusters move for long, but
# the first test leaves next to nothing of the tiles.
@pytest.mark.parametrize("n,d,k,iters,comps", [(140_000, 128, 2048, 20, 1024), (200_000, 64, 2048, 20, 512), (100_000, 32, 8200, 20, 8200)])
def test_points_of_a_fit_not_regrouped_again(skm, dg, n, d, k, iters, comps):  # noqa: F811
    say("not regrouped again", n, d, k, iters)
    X = dg.mixture(n, d, comps, 3, "embed", "cuda")
    own = torch.empty(n * d + 1, device="cuda")[1:].view(n, d).copy_(X)
    a, b = (skm.fit(x, k, iters, 5, skm.FitOptions(rotate=False)) for x in (X, own))
    assert not regroupings(a.trace, n, k, iters)
    assert [r["listed_tiles"] for r in a.trace] == [r["listed_tiles"] for r in b.trace]
    assert torch.equal(a.assign, b.assign) and torch.equal(a.centroids, b.centroids) and torch.equal(a.dist, b.dist)


# ... and where there is no memory for the regrouped copy the fit is served without it.  Mixtures with fewer components than clusters
# are not regrouped in the first place, in four iterations, because the step before has cut more than 85 % of the pairs; in six, or
# into more clusters, they are.
@pytest.mark.parametrize("k,comps,iters,regrouped", [(2048, 4096, 4, True), (2048, 1024, 4, False), (4096, 1024, 6, True)])
def test_fit_without_memory_for_the_order(skm, dg, k, comps, iters, regrouped):  # noqa: F811
    n, d = 400_000, 512
    say("fit, a full device", n, d, k, comps)
    X = dg.mixture(n, d, comps, 3, "embed", "cuda")
    opts = skm.FitOptions(R=skm.make_rotation(d, 4), own_workspace=True)
    a = skm.fit(X, k, iters, 5, opts)
    skm.release_memory()
    held = fill_device(skm.workspace_bytes(n, d, k) - n * d * 2)
    b = skm.fit(X, k, iters, 5, opts)
    del held
    torch.cuda.empty_cache()
    tiles = [sum(r["listed_tiles"] for r in x.trace) for x in (a, b)]
    assert tiles[0] < tiles[1] if regrouped else tiles[0] == tiles[1] > 0
    assert float((a.centroids - b.centroids).norm() / a.centroids.norm()) < 1e-4
    assert float((a.assign != b.assign).float().mean()) <= 1e-3


# ... also a short one with recall, whose queries, ground truth and scores are taken after its points: where there is memory for those
# or for the regrouped copy, not for both, the fit gets what it cannot do without.
def test_short_fit_with_recall_without_memory_for_the_order(skm, dg):  # noqa: F811
    n, d, k, nq, topk = 400_000, 512, 2048, 16_000, 10
    say("short fit with recall, a full device", n, d, k)
    X = dg.mixture(n, d, 2 * k, 3, "embed", "cuda")
    Q = dg.mixture(nq, d, 2 * k, 3, "embed", "cuda", sample_seed=9)
    opts = skm.FitOptions(R=skm.make_rotation(d, 4), own_workspace=True, etr=True, queries=Q, topk=topk, etr_patience=10)
    a = skm.fit(X, k, 4, 5, opts)
    skm.release_memory()
    copy = n * d * 4
    # what is taken before the recall's buffers: the plan of a fit without recall but for a copy and for what that plan holds for the
    # making of a rotation and in reserve
    base = skm.workspace_bytes(n, d, k) - copy - 7 * d * d * 4 - d * 16384 - (32 << 20)
    # the recall's own: a chunk of points and the queries in 16 bits, a group's minima, 1024 candidates, keys, rotated queries, scores
    recall = nq * (65_536 // 64 * 4 + 1024 * 8 + topk * 8 + d * 6 + k * 4) + 131_072 * d * 2
    assert base + recall < base + copy + recall // 2
    held = fill_device(base + copy + recall // 2)
    b = skm.fit(X, k, 4, 5, opts)
    del held
    torch.cuda.empty_cache()
    assert sum(r["listed_tiles"] for r in a.trace) < sum(r["listed_tiles"] for r in b.trace)
    assert max(abs(p["recall"] - q["recall"]) for p, q in zip(a.trace[:4], b.trace[:4])) <= 1e-3
    assert float((a.centroids - b.centroids).norm() / a.centroids.norm()) < 1e-4
    assert float((a.assign != b.assign).float().mean()) <= 1e-3


# A call with a rotation multiplies its rows and its centroids in one launch, behind one that takes both bounds and the copies of
# the matrix (rows that are not aligned, and the tall form, in launches of their own).  On rows that were rotated before the call
# labels and distances are the same bits.
@pytest.mark.parametrize("n,k,d", [(1, 1, 32), (127, 129, 32), (128, 128, 48), (129, 1, 100), (300, 257, 128), (1000, 3, 132),
                                   (64, 100, 33), (257, 130, 30), (5000, 700, 272), (140_000, 40, 128), (3, 2, 16)])
def test_rows_and_centroids_rotated_together(skm, dg, n, k, d):  # noqa: F811
    say("rotated together", n, k, d)
    X = dg.mixture(n, d, 20, 3, "linear", "cuda")
    Y = dg.mixture(k, d, 20, 3, "linear", "cuda", sample_seed=4)
    R = skm.make_rotation(d, 9)
    prev = torch.randint(0, k, (n,), generator=torch.Generator().manual_seed(1)).int().cuda()
    for p in (None, prev):
        a, da, _ = skm.assign(X, Y, p, opts=skm.FitOptions(R=R))
        b, db, _ = skm.assign(skm.rotate(X, R), skm.rotate(Y, R), p, opts=skm.FitOptions(rotate=False))
        assert torch.equal(a, b) and torch.equal(da, db)


# The same launch with 256 x 256 tiles, where those of both fill the rounds of the device (a first, a part and a second round; ragged
# rows and columns).  A rotated coordinate is off by 2^-21 of its row in the 22-bit products and the rotation's own entries by
# fp32, so that a vector is by less than e = 2^-18 of both norms (256 to 1536 terms added in fp32) and its squared distance by
# 2 e dist + e^2; a distance from |x|^2 + |y|^2 - 2 x.y adds 2^-20 of the squares (22-bit operands, three fp32
# roundings) and 2^-24 for each of the d / 8 partial sums behind one another.  Tests that drop nothing leave the nearest centroid,
# by distances of that error.
@pytest.mark.parametrize("n,k,d", [(52_100, 300, 256), (60_000, 5, 224), (26_300, 1, 448), (9000, 257, 1536), (120_000, 300, 256)])
def test_rows_and_centroids_rotated_together_in_large_tiles(skm, dg, n, k, d):  # noqa: F811
    say("rotated together, large tiles", n, k, d)
    X = dg.mixture(n, d, 20, 3, "linear", "cuda")
    Y = dg.mixture(k, d, 20, 3, "linear", "cuda", sample_seed=4)
    prev = torch.randint(0, k, (n,), generator=torch.Generator().manual_seed(1)).int().cuda()
    for p in (None, prev):
        a, da, _ = skm.assign(X, Y, p, opts=skm.FitOptions(R=skm.make_rotation(d, 9), eps0=100.0))
        for i in range(0, n, 8192):
            x, y = X[i:i + 8192].double(), Y.double()
            D = torch.cdist(x, y, compute_mode="donot_use_mm_for_euclid_dist")
            e = 2.0 ** -18 * (x.norm(dim=1) + y.norm(dim=1).max())
            at = D.gather(1, a[i:i + 8192, None].long())[:, 0]
            off = 2 * at * e + e ** 2 + (2.0 ** -20 + d * 2.0 ** -27) * ((x ** 2).sum(1) + (y ** 2).sum(1).max())
            assert bool(((da[i:i + 8192].double() - at ** 2).abs() <= off).all())
            assert bool((at ** 2 <= D.min(1).values ** 2 + 2 * off).all())


# Up to 256 dimensions the thresholds of a step are taken in the launch that prepares its centroids (a form for each 128), beyond
# in one of their own.  With tests that drop nothing the last labels are the nearest centroids, at their direct distances.
@pytest.mark.parametrize("d", [16, 112, 128, 130, 144, 250, 256, 272])
def test_thresholds_beside_the_centroids(skm, d):  # noqa: F811
    say("thresholds beside the centroids", d)
    n, k = 3001, 37
    X = torch.randn(n, d, generator=torch.Generator().manual_seed(d)).cuda()
    r = skm.fit(X, k, 4, 3, skm.FitOptions(rotate=False, eps0=100.0))
    D = torch.cdist(X.double(), r.centroids.double(), compute_mode="donot_use_mm_for_euclid_dist") ** 2
    near, at = D.topk(2, 1, largest=False)
    clear = near[:, 1] - near[:, 0] > 1e-4 * near[:, 0]      # fp32 distances of 22-bit products
    assert torch.equal(r.assign[clear].long(), at[clear, 0])
    assert bool(((r.dist.double() - near[:, 0]).abs() <= 1e-4 * near[:, 0] + 1e-6).all())      # (a cluster of one point: 0)


# An update in which few points moved is launched before the host knows how many did, and does nothing where they are none or more
# than its form takes (2^25 / 2k / slices of 256 dimensions, or an eighth of the points).  It is launched where the step before says
# that it may be that form (some changed, and at most four times as many), so the labels that changed say which steps it was
# launched in and what it did there: it took effect, they were too many, or none.  The sums are fp64, so the means are
# those of full updates to the last bit of fp32; unit rows (the angular metric) add that of their length.  With most points
# on a few places clusters run empty in every step, and their splits follow an update that has run ahead.
@pytest.mark.parametrize("n,d,k,iters,places,angular,reached", [
    (100_000, 64, 4096, 12, 0, False, {"took", "many"}), (20_000, 128, 100, 14, 0, False, {"took", "none"}),
    (3000, 300, 30, 25, 0, False, {"took", "none"}), (1000, 520, 3, 12, 0, False, {"none"}), (40, 16, 4, 6, 0, False, {"none"}),
    (100_000, 64, 4096, 12, 0, True, {"took", "many"}), (1000, 520, 3, 12, 0, True, {"took", "none"}),
    (6000, 64, 60, 14, 40, False, {"split", "many"}), (6000, 64, 80, 14, 20, True, {"split", "many", "none"})])
def test_updates_ahead_of_the_report(skm, dg, n, d, k, iters, places, angular, reached):  # noqa: F811
    say("updates ahead", n, d, k, places, angular)
    X = dg.mixture(n, d, max(2, 2 * k), 5, "linear", "cpu" if places else "cuda")
    if places:
        g = torch.Generator().manual_seed(8)
        far, m = torch.randn(places, d, generator=g) * 3, n * 9 // 10
        X[:m] = far[torch.randint(0, places, (m,), generator=g)]
        X = X[torch.randperm(n, generator=g)].cuda()
    R = skm.make_rotation(d, 2)
    a, b = (skm.fit(X, k, iters, 4, skm.FitOptions(R=R, full_update=f, angular=angular)) for f in (False, True))
    assert a.timing["inc_updates"] >= 1 and b.timing["inc_updates"] == 0
    assert [r["changed"] for r in a.trace] == [r["changed"] for r in b.trace]
    assert [r["nempty"] for r in a.trace] == [r["nempty"] for r in b.trace]
    assert torch.equal(a.assign, b.assign)
    assert float((a.centroids - b.centroids).norm() / b.centroids.norm()) < 1e-6
    most = min(2 * (n // 8), 2**25 // (k * (((d + 15) // 16 * 16 + 255) // 256))) // 2
    seen = set()
    for before, step in zip(a.trace[1:iters], a.trace[2:iters]):   # from iteration 3 on
        if 0 < before["changed"] <= 4 * most:
            c = step["changed"]
            seen.add("none" if c == 0 else "many" if c > most else "split" if step["nempty"] else "took")
    assert seen >= reached


# A program that asks the runtime for blocking waits, before its first GPU call, keeps the core for itself in a fit as well: of 30 steps
# the host is busy for the launches and for what the runtime takes to block, 28 % of the time (68 % where the host watches the report
# for half a millisecond a step).
BLOCKING = """
import ctypes, time
import torch
from paper_2603_20009_amd import datagen, skm
with open("/proc/self/maps") as f:
    hip = ctypes.CDLL(next(p for p in f.read().split() if "libamdhip64" in p))
assert hip.hipSetDeviceFlags(ctypes.c_uint(4)) == 0       # hipDeviceScheduleBlockingSync
X = datagen.mixture(1_000_000, 768, 800, 3, "embed", "cuda")
opts = skm.FitOptions(R=skm.make_rotation(768, 4))
share = []
for _ in range(4):
    wall, cpu = time.perf_counter(), time.thread_time()
    skm.fit(X, 200, 30, 5, opts)
    share.append((time.thread_time() - cpu) / (time.perf_counter() - wall))
print(min(share[1:]))
"""


def test_fit_of_a_program_with_blocking_waits(skm):  # noqa: F811
    say("blocking waits")
    r = subprocess.run([sys.executable, "-c", BLOCKING], capture_output=True, text=True, timeout=100,
                       cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert r.returncode == 0, r.stderr
    assert float(r.stdout.split()[-1]) < 0.45, r.stdout
