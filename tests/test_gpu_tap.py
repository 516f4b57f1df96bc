"""GPU parity of the calibration-set clustering (include/qc_tap.h) against the oracle (oracle/tap.py), through the C
ABI, on seeded synthetic pools.  Floating-point results: fp32 arithmetic against fp64, tolerances stated at each check;
labels, permutations and votes: exact, except where a distance tie within fp32 rounding decides (then the label must be
one of the tied centres)."""
import hashlib
import os

import numpy as np
import pytest

from oracle import tap
from synthetic import tap_inputs as TI

pytestmark = pytest.mark.gpu


def _cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _work(qc, N, F, n, k, kb):
    import torch
    return torch.empty(qc.qc_tap_workspace_bytes(N, F, n, k, kb), dtype=torch.uint8, device="cuda")


@pytest.fixture(scope="module")
def qc():
    import paper_2503_02508_amd as m
    return m


# ------------------------------------------------------------------------------------------- similarity
@pytest.mark.parametrize("N,F,n,alpha,shuffle", [
    (300, 64, 40, 0.5, False),        # 3 row tiles with a ragged tail, 16-byte loads
    (300, 70, 37, 0.3, True),         # K not a multiple of 4: element loads; unsorted indices
    (517, 256, 150, 0.5, False),      # two column tiles
    (128, 32, 128, 1.0, False),       # whole pool as the subsample, cosine only: symmetric, unit diagonal
    (130, 8, 9, 0.0, True),           # temporal only
])
def test_similarity_and_degrees(qc, N, F, n, alpha, shuffle):
    import torch
    X, t, _, _ = TI.make_pool(N, F, 50, 16, seed=N + F)
    idx = TI.make_subsamples(N, n, 1, seed=n)[0]
    if shuffle:
        idx = np.random.default_rng(1).permutation(idx).astype(np.int32)
    A = torch.empty((N, n), device="cuda")
    dr, dc = torch.empty(N, device="cuda"), torch.empty(n, device="cuda")
    work = _work(qc, N, F, n, 8, 8)
    qc.qc_tap_similarity(_cuda(X), _cuda(t), _cuda(idx), alpha, A, dr, dc, work)
    want = tap.similarity(X, t, idx, alpha)
    got = A.cpu().numpy().astype(np.float64)
    # entries are at most 1 in magnitude: fp32 products over F terms, fp32 exp
    assert np.abs(got - want).max() <= 2e-6, np.abs(got - want).max()
    wr, wc = tap.degrees(want)
    assert np.allclose(dr.cpu().numpy(), wr, rtol=2e-6, atol=1e-6 * n)
    assert np.allclose(dc.cpu().numpy(), wc, rtol=2e-6, atol=1e-6 * N)
    if alpha == 1.0 and n == N:
        assert np.abs(got - got.T).max() <= 2e-6 and np.abs(np.diag(got) - 1.0).max() <= 2e-6


def test_similarity_rejects_bad_indices_and_handles_zero_rows(qc):
    import torch
    N, F, n = 200, 32, 16
    X, t, _, _ = TI.make_pool(N, F, 50, 16, seed=3)
    X[5] = 0.0
    idx = TI.make_subsamples(N, n, 1, seed=4)[0]
    A = torch.empty((N, n), device="cuda")
    dr, dc = torch.empty(N, device="cuda"), torch.empty(n, device="cuda")
    work = _work(qc, N, F, n, 8, 8)
    qc.qc_tap_similarity(_cuda(X), _cuda(t), _cuda(idx), 1.0, A, dr, dc, work)
    assert torch.isfinite(A).all() and (A[5] == 0).all()          # a zero vector has cosine 0 with everything
    bad = idx.copy()
    bad[3] = N
    with pytest.raises(qc.QCError) as e:
        qc.qc_tap_similarity(_cuda(X), _cuda(t), _cuda(bad), 0.5, A, dr, dc, work)
    assert e.value.code == -4
    bad[3] = -1
    with pytest.raises(qc.QCError):
        qc.qc_tap_similarity(_cuda(X), _cuda(t), _cuda(bad), 0.5, A, dr, dc, work)
    qc.qc_tap_similarity(_cuda(X), _cuda(t), _cuda(idx), 0.5, A, dr, dc, work)    # still usable afterwards
    assert torch.isfinite(A).all()


def test_normalise(qc):
    import torch
    rng = np.random.default_rng(5)
    N, n = 333, 45
    A = rng.uniform(0.05, 1.0, size=(N, n)).astype(np.float32)
    dr, dc = A.astype(np.float64).sum(1).astype(np.float32), A.astype(np.float64).sum(0).astype(np.float32)
    Ad = _cuda(A)
    work = _work(qc, N, 8, n, 8, 8)
    qc.qc_tap_normalise(Ad, _cuda(dr), _cuda(dc), work)
    want = tap.normalised(A)
    assert np.allclose(Ad.cpu().numpy(), want, rtol=1e-6, atol=0)
    # a non-positive degree is refused and the matrix left alone
    Ad = _cuda(A)
    dr_bad = dr.copy()
    dr_bad[7] = 0.0
    with pytest.raises(qc.QCError) as e:
        qc.qc_tap_normalise(Ad, _cuda(dr_bad), _cuda(dc), work)
    assert e.value.code == -4 and np.array_equal(Ad.cpu().numpy(), A)
    dc_bad = dc.copy()
    dc_bad[0] = np.nan
    with pytest.raises(qc.QCError):
        qc.qc_tap_normalise(Ad, _cuda(dr), _cuda(dc_bad), work)


# -------------------------------------------------------------------------------------------- embedding
def _planted_L(N, F, k, n, seed):
    X, t, truth = TI.make_planted(N, F, k, seed=seed)
    idx = TI.make_subsamples(N, n, 1, seed=seed + 1)[0]
    return tap.normalised(tap.similarity(X, t, idx, 0.5)).astype(np.float32), truth


@pytest.mark.parametrize("N,n,k,kb,iters", [(420, 56, 6, 8, 6), (700, 97, 5, 16, 4), (300, 130, 12, 24, 4), (400, 160, 3, 128, 2)])
def test_embedding_matches_singular_vectors(qc, N, n, k, kb, iters):
    import torch
    L, _ = _planted_L(N, 40, k, n, seed=N)
    U = torch.empty((N, k), device="cuda")
    sig = torch.empty(k, device="cuda")
    work = _work(qc, N, 40, n, k, kb)
    q0 = TI.make_start_block(kb, n, seed=9)
    qc.qc_tap_embed(_cuda(L), k, iters, _cuda(q0), U, sig, work)
    Uo, so = tap.embed(L, k + 1)
    gap = so[k - 1] / so[k]
    assert gap > 1.5, "the test pool must separate the k leading singular values (gap %.2f)" % gap
    Ud = U.cpu().numpy().astype(np.float64)
    assert np.allclose(sig.cpu().numpy(), so[:k], atol=2e-5), (sig.cpu().numpy(), so[:k])
    assert np.abs(Ud.T @ Ud - np.eye(k)).max() <= 1e-4                        # orthonormal columns
    # same subspace: every principal angle's cosine is 1 (signs and rotations inside equal singular values are free)
    cosines = np.linalg.svd(Ud.T @ Uo[:, :k], compute_uv=False)
    assert cosines.min() >= 1 - 1e-5, cosines
    # column by column where the singular values are well separated from their neighbours
    for j in range(k):
        lo = so[j] - so[j + 1]
        hi = so[j - 1] - so[j] if j else np.inf
        if min(lo, hi) > 1e-2:
            assert abs(abs(Ud[:, j] @ Uo[:, j]) - 1.0) <= 1e-4, j


def test_embedding_rejects_a_start_block_without_full_rank(qc):
    import torch
    N, n, k, kb = 200, 40, 4, 8
    L, _ = _planted_L(N, 24, k, n, seed=11)
    q0 = TI.make_start_block(kb, n, seed=12)
    q0[3] = 0.0                                                         # a zero start vector
    U, sig = torch.empty((N, k), device="cuda"), torch.empty(k, device="cuda")
    with pytest.raises(qc.QCError) as e:
        qc.qc_tap_embed(_cuda(L), k, 3, _cuda(q0), U, sig, _work(qc, N, 24, n, k, kb))
    assert e.value.code == -4


# ---------------------------------------------------------------------------------------------- k-means
def _check_labels(U, got, want_labels, centres):
    """Labels equal the oracle's, except rows whose two nearest centres are tied within fp32 rounding."""
    diff = np.flatnonzero(got != want_labels)
    if len(diff):
        d2 = ((U[diff, None, :].astype(np.float64) - centres[None]) ** 2).sum(-1)
        a, b = d2[np.arange(len(diff)), got[diff]], d2[np.arange(len(diff)), want_labels[diff]]
        assert np.all(np.abs(a - b) <= 1e-5 * np.maximum(a, b)), "labels differ beyond distance ties"
    return len(diff)


@pytest.mark.parametrize("N,d,k,spread", [(1000, 6, 5, 0.7), (777, 3, 4, 1.5), (4099, 100, 100, 0.3), (130, 128, 128, 0.5), (50, 1, 2, 1.0)])
def test_kmeans_matches_oracle(qc, N, d, k, spread):
    import torch
    rng = np.random.default_rng(N + d)
    means = rng.standard_normal((k, d)) * 3
    U = (means[rng.integers(0, k, size=N)] + spread * rng.standard_normal((N, d))).astype(np.float32)
    init = rng.choice(N, k, replace=False).astype(np.int32)
    labels = torch.empty(N, dtype=torch.int32, device="cuda")
    centres = torch.empty((k, d), device="cuda")
    passes = qc.qc_tap_kmeans(_cuda(U), _cuda(init), 100, labels, centres, _work(qc, max(N, 256), 8, 128, k, 128))
    wl, wc, wp = tap.kmeans(U, init, 100)
    nd = _check_labels(U, labels.cpu().numpy(), wl, wc)
    if nd == 0:
        assert passes == wp
        assert np.allclose(centres.cpu().numpy(), wc, rtol=1e-6, atol=1e-6)
    # fixed point whatever happened: every row sits with its nearest centre
    c = centres.cpu().numpy().astype(np.float64)
    d2 = ((U[:, None, :].astype(np.float64) - c[None]) ** 2).sum(-1) if N * k * d < 5e7 else None
    if d2 is not None and passes < 100:
        mine = d2[np.arange(N), labels.cpu().numpy()]
        assert np.all(mine <= d2.min(1) * (1 + 1e-5) + 1e-12)


def test_kmeans_pass_limit_duplicate_centres_and_bad_indices(qc):
    import torch
    U = np.array([[1.0], [1.0], [3.0]], dtype=np.float32)
    work = _work(qc, 256, 8, 128, 2, 128)
    labels, centres = torch.empty(3, dtype=torch.int32, device="cuda"), torch.empty((2, 1), device="cuda")
    # duplicate initial centres: the second stays empty in the first pass and keeps its centre
    assert qc.qc_tap_kmeans(_cuda(U), _cuda(np.array([0, 1], np.int32)), 1, labels, centres, work) == 1
    assert labels.cpu().tolist() == [0, 0, 0] and centres.cpu().numpy()[:, 0].tolist() == [np.float32(5.0 / 3), 1.0]
    wl, wc, wp = tap.kmeans(U, [0, 1], 10)
    assert qc.qc_tap_kmeans(_cuda(U), _cuda(np.array([0, 1], np.int32)), 10, labels, centres, work) == wp
    assert labels.cpu().tolist() == wl.tolist() and np.allclose(centres.cpu().numpy(), wc)
    with pytest.raises(qc.QCError) as e:
        qc.qc_tap_kmeans(_cuda(U), _cuda(np.array([0, 3], np.int32)), 10, labels, centres, work)
    assert e.value.code == -4
    # pass limits that fall inside and at the end of a group of passes the host enqueues ahead, on a problem that needs
    # more passes than any of them: the state after exactly that many passes
    rng = np.random.default_rng(77)
    N, d, k = 3000, 8, 12
    U = (rng.standard_normal((k, d))[rng.integers(0, k, size=N)] + 1.5 * rng.standard_normal((N, d))).astype(np.float32)
    init = rng.choice(N, k, replace=False).astype(np.int32)
    assert tap.kmeans(U, init, 100)[2] > 17
    labels, centres = torch.empty(N, dtype=torch.int32, device="cuda"), torch.empty((k, d), device="cuda")
    work = _work(qc, N, 8, 128, k, 128)
    for limit in (3, 8, 9, 17):
        wl, wc, wp = tap.kmeans(U, init, limit)
        assert wp == limit
        assert qc.qc_tap_kmeans(_cuda(U), _cuda(init), limit, labels, centres, work) == limit
        if _check_labels(U, labels.cpu().numpy(), wl, wc) == 0:
            assert np.allclose(centres.cpu().numpy(), wc, rtol=1e-6, atol=1e-6)


# ------------------------------------------------------------------------------------------ aggregation
@pytest.mark.parametrize("m,N,k,noise", [(3, 1000, 7, 0.1), (5, 3001, 100, 0.3), (1, 100, 4, 0.0), (2, 64, 128, 0.5), (8, 500, 3, 1.0)])
def test_aggregate_is_bit_exact(qc, m, N, k, noise):
    import torch
    rng = np.random.default_rng(m * 1000 + k)
    base = rng.integers(0, k, size=N)
    labels = []
    for i in range(m):
        lab = rng.permutation(k)[base]
        flip = rng.random(N) < noise                                # noise 1.0: independent labels, ties everywhere
        lab = np.where(flip, rng.integers(0, k, size=N), lab)
        labels.append(lab)
    labels = np.stack(labels).astype(np.int32)
    out = torch.empty(N, dtype=torch.int32, device="cuda")
    perm = torch.empty((m, k), dtype=torch.int32, device="cuda")
    qc.qc_tap_aggregate(_cuda(labels), k, out, _work(qc, 256, 8, 128, k, 128), perm)
    want = tap.aggregate(labels, k)
    assert np.array_equal(out.cpu().numpy(), want)
    p = perm.cpu().numpy()
    assert p[0].tolist() == list(range(k))
    for i in range(1, m):
        assert np.array_equal(p[i], tap.greedy_match(tap.contingency(labels[0], labels[i], k)))


# ------------------------------------------------------------------------------------- whole algorithm
@pytest.mark.parametrize("N,F,k,n,kb,m,slots", [(700, 96, 6, 80, 8, 3, 1), (1100, 64, 9, 140, 16, 3, 3), (900, 48, 5, 70, 8, 5, 2)])
def test_cluster_recovers_planted_groups_like_the_oracle(qc, N, F, k, n, kb, m, slots):
    """slots = subsamples worked on at a time (workspace of that many times the base size): same labels."""
    import torch
    X, t, truth = TI.make_planted(N, F, k, seed=N)
    subs = TI.make_subsamples(N, n, m, seed=N + 1)
    init = np.stack([[int(np.flatnonzero(truth == g)[i]) for g in range(k)] for i in range(m)]).astype(np.int32)
    q0 = TI.make_start_block(kb, n, seed=N + 2)
    final = torch.empty(N, dtype=torch.int32, device="cuda")
    per = torch.empty((m, N), dtype=torch.int32, device="cuda")
    base = (qc.qc_tap_workspace_bytes(N, F, n, k, kb) + 255) // 256 * 256
    work = torch.empty(slots * base, dtype=torch.uint8, device="cuda")
    qc.qc_tap_cluster(_cuda(X), _cuda(t), _cuda(subs), 0.5, k, 8, _cuda(q0), _cuda(init), 50, final, per, work)
    wf, wp = tap.tap(X, t, subs, 0.5, k, init, 50)
    # the oracle recovers the planted groups exactly (its own pin); the embedding's sign and rotation freedom does
    # not touch distances between rows, so the labels must be the same ones
    assert np.array_equal(per.cpu().numpy(), wp)
    assert np.array_equal(final.cpu().numpy(), wf)
    assert np.array_equal(final.cpu().numpy(), truth)                # centre g starts inside planted group g


def test_cluster_on_a_pool_without_planted_groups_gives_the_oracles_labels(qc):
    """The small workload's pool (diffusion-like samples of 16 classes at 50 noise levels, no planted groups: the
    singular values fall off smoothly after the third): with 100 rounds of the block iteration the embedding spans
    the oracle's subspace to 1 - cos <= 1e-6, and the whole algorithm (three subsamples, k-means, alignment, vote)
    returns the oracle's labels, per subsample and final, at the benchmark's 8 rounds and at 100."""
    import torch
    wl = TI.TAP_WORKLOADS["tap0"]
    kb = 32
    N, F, n, k, m = wl.N, wl.F, wl.n, wl.k, wl.m
    X, t, _, _ = TI.make_pool(N, F, wl.steps, wl.classes, wl.seed)
    subs = TI.make_subsamples(N, n, m, wl.seed + 1)
    init = TI.make_init(N, k, m, wl.seed + 2)
    q0 = TI.make_start_block(kb, n, wl.seed + 3)
    wf, wp = tap.tap(X, t, subs, wl.alpha, k, init, 100)
    assert len(np.unique(wf)) == k                                    # every cluster is used: not a degenerate pool
    work = _work(qc, N, F, n, k, kb)
    # subspace of the first subsample's embedding
    A = torch.empty((N, n), device="cuda")
    dr, dc = torch.empty(N, device="cuda"), torch.empty(n, device="cuda")
    qc.qc_tap_similarity(_cuda(X), _cuda(t), _cuda(subs[0]), wl.alpha, A, dr, dc, work)
    qc.qc_tap_normalise(A, dr, dc, work)
    U, sig = torch.empty((N, k), device="cuda"), torch.empty(k, device="cuda")
    qc.qc_tap_embed(A, k, 100, _cuda(q0), U, sig, work)
    Uo, so = tap.embed(tap.normalised(tap.similarity(X, t, subs[0], wl.alpha)), k + 1)
    assert so[k - 1] / so[k] > 1.01                                   # the k-th and (k+1)-th values are distinct
    cosines = np.linalg.svd(U.cpu().numpy().astype(np.float64).T @ Uo[:, :k], compute_uv=False)
    assert cosines.min() >= 1 - 1e-6, cosines
    assert np.allclose(sig.cpu().numpy(), so[:k], atol=2e-6)
    for iters in (8, 100):
        final = torch.empty(N, dtype=torch.int32, device="cuda")
        per = torch.empty((m, N), dtype=torch.int32, device="cuda")
        qc.qc_tap_cluster(_cuda(X), _cuda(t), _cuda(subs), wl.alpha, k, iters, _cuda(q0), _cuda(init), 100, final, per, work)
        assert np.array_equal(per.cpu().numpy(), wp), iters
        assert np.array_equal(final.cpu().numpy(), wf), iters


# ------------------------------------------------------- the paper's sizes, in the configuration bench.py times
def test_paper_sized_pool_sampled_outputs_and_properties(qc):
    """N = 32768 samples of 4096 features, subsamples of N / 20, 100 clusters, iteration block 128, 8 power
    iterations: entries, degrees and normalised entries on sampled rows and columns against the oracle one by one;
    the embedding and the k-means result through properties that hold at any size."""
    import torch
    wl = TI.TAP_WORKLOADS["tap1"]
    kb, iters = 128, 8
    N, F, n, k = wl.N, wl.F, wl.n, wl.k
    X, t, _, _ = TI.make_pool(N, F, wl.steps, wl.classes, wl.seed)
    idx = TI.make_subsamples(N, n, wl.m, wl.seed + 1)[0]
    rng = np.random.default_rng(77)
    R = np.sort(rng.choice(N, 24, replace=False))
    R[0], R[-1] = 0, N - 1                                           # first and last row tile
    H = np.array([0, 1, 127, 128, n // 2, n - 1])                    # tile edges and the ragged last column tile
    Xd, td = _cuda(X), _cuda(t)
    A = torch.empty((N, n), device="cuda")
    dr, dc = torch.empty(N, device="cuda"), torch.empty(n, device="cuda")
    work = _work(qc, N, F, n, k, kb)
    qc.qc_tap_similarity(Xd, td, _cuda(idx), wl.alpha, A, dr, dc, work)
    # sampled rows against all subsample columns (gives their degrees too)
    rows = tap.similarity(np.concatenate([X[R], X[idx]]), np.concatenate([t[R], t[idx]]), len(R) + np.arange(n), wl.alpha)[:len(R)]
    assert np.abs(A[_cuda(R)].cpu().numpy() - rows).max() <= 2e-6
    assert np.allclose(dr[_cuda(R)].cpu().numpy(), rows.sum(1), rtol=2e-6)
    # sampled columns against all pool rows
    cols = np.concatenate([tap.similarity(X, t, [int(idx[h])], wl.alpha) for h in H], axis=1)       # [N, len(H)]
    assert np.abs(A[:, _cuda(H)].cpu().numpy() - cols).max() <= 2e-6
    assert np.allclose(dc[_cuda(H)].cpu().numpy(), cols.sum(0), rtol=2e-6)
    qc.qc_tap_normalise(A, dr, dc, work)
    want = rows[:, H] / np.sqrt(rows.sum(1))[:, None] / np.sqrt(cols.sum(0))[None, :]
    got = A[_cuda(R)][:, _cuda(H)].cpu().numpy()
    assert np.allclose(got, want, rtol=5e-6)

    U = torch.empty((N, k), device="cuda")
    sig = torch.empty(k, device="cuda")
    qc.qc_tap_embed(A, k, iters, _cuda(TI.make_start_block(kb, n, wl.seed + 3)), U, sig, work)
    s = sig.cpu().numpy().astype(np.float64)
    assert abs(s[0] - 1.0) <= 1e-5 and np.all(np.diff(s) <= 1e-7) and s[-1] > 0      # sigma_1 = 1, descending
    Ud = U.double()
    assert float((Ud.T @ Ud - torch.eye(k, device="cuda", dtype=torch.float64)).abs().max()) <= 1e-5
    # the leading left singular vector of the normalised matrix is sqrt(d_r) up to scale
    u1 = torch.sqrt(dr.double() / dr.double().sum())
    assert abs(abs(float(u1 @ Ud[:, 0])) - 1.0) <= 1e-6
    # Convergence criterion of the block iteration, for ALL k pairs at the iteration count bench.py times (8 rounds
    # with a block of 128): || L L^T u_j - sigma_j^2 u_j || <= 2e-6 sigma_1^2 (measured: 6e-7 for the leading pair, whose
    # residual is fp32 rounding of entries of size 1, and below 2e-7 for all others), and every sigma_j within 5e-5 of
    # the singular values a library routine (float64 SVD of the device's own normalised matrix) returns; the trailing
    # values of this pool lie 1e-6 apart, so single vectors are not pinned there, the invariant subspace is.
    Ld = A.double()
    res = (Ld @ (Ld.T @ Ud) - Ud * torch.from_numpy(s ** 2).cuda()[None]).norm(dim=0).cpu().numpy()
    assert res.shape == (k,) and res.max() <= 2e-6 * s[0] ** 2, (int(res.argmax()), float(res.max()))
    sv = torch.linalg.svdvals(Ld).cpu().numpy()
    assert np.abs(s - sv[:k]).max() <= 5e-5, float(np.abs(s - sv[:k]).max())
    # 32 rounds bring every sigma_j to the library's within fp32 rounding
    U32, sig32 = torch.empty((N, k), device="cuda"), torch.empty(k, device="cuda")
    qc.qc_tap_embed(A, k, 32, _cuda(TI.make_start_block(kb, n, wl.seed + 3)), U32, sig32, work)
    assert np.abs(sig32.cpu().numpy().astype(np.float64) - sv[:k]).max() <= 5e-7
    res32 = (Ld @ (Ld.T @ U32.double()) - U32.double() * (sig32.double() ** 2)[None]).norm(dim=0)
    assert float(res32.max()) <= 2e-6
    del Ld, U32

    labels = torch.empty(N, dtype=torch.int32, device="cuda")
    centres = torch.empty((k, k), device="cuda")
    init = TI.make_init(N, k, wl.m, wl.seed + 2)[0]
    passes = qc.qc_tap_kmeans(U, _cuda(init), 100, labels, centres, work)
    assert 2 <= passes <= 100
    lab = labels.cpu().numpy()
    assert lab.min() >= 0 and lab.max() < k
    Uh, c = U.cpu().numpy().astype(np.float64), centres.cpu().numpy().astype(np.float64)
    if passes < 100:
        # converged: every sampled row sits with its nearest centre, every centre is the mean of its rows
        samp = rng.choice(N, 2000, replace=False)
        d2 = ((Uh[samp, None, :] - c[None]) ** 2).sum(-1)
        mine = d2[np.arange(len(samp)), lab[samp]]
        assert np.all(mine <= d2.min(1) * (1 + 1e-5) + 1e-14)
        for g in (0, k // 2, k - 1):
            members = Uh[lab == g]
            if len(members):
                assert np.allclose(c[g], members.mean(0), rtol=1e-5, atol=1e-7)


def test_paper_sized_aggregation_is_bit_exact(qc):
    import torch
    N, k, m = 32768, 100, 3
    rng = np.random.default_rng(78)
    base = rng.integers(0, k, size=N)
    labels = np.stack([np.where(rng.random(N) < 0.08, rng.integers(0, k, size=N), rng.permutation(k)[base]) for _ in range(m)]).astype(np.int32)
    out = torch.empty(N, dtype=torch.int32, device="cuda")
    qc.qc_tap_aggregate(_cuda(labels), k, out, _work(qc, 256, 8, 128, k, 128))
    assert np.array_equal(out.cpu().numpy(), tap.aggregate(labels, k))


def test_cluster_reports_deferred_errors(qc):
    """Inside the whole algorithm the data-dependent checks are read after the k-means of the subsample concerned."""
    import torch
    N, F, k, n, kb, m = 400, 32, 4, 48, 8, 3
    X, t, truth = TI.make_planted(N, F, k, seed=5)
    subs = TI.make_subsamples(N, n, m, seed=6)
    init = np.stack([[int(np.flatnonzero(truth == g)[i]) for g in range(k)] for i in range(m)]).astype(np.int32)
    q0 = TI.make_start_block(kb, n, seed=7)
    final = torch.empty(N, dtype=torch.int32, device="cuda")
    per = torch.empty((m, N), dtype=torch.int32, device="cuda")
    base = (qc.qc_tap_workspace_bytes(N, F, n, k, kb) + 255) // 256 * 256
    for slots in (1, 3):
        work = torch.empty(slots * base, dtype=torch.uint8, device="cuda")
        bad = subs.copy(); bad[1, 5] = N + 3
        with pytest.raises(qc.QCError) as e:
            qc.qc_tap_cluster(_cuda(X), _cuda(t), _cuda(bad), 0.5, k, 4, _cuda(q0), _cuda(init), 20, final, per, work)
        assert e.value.code == -4 and "subsample index" in str(e.value)
        badi = init.copy(); badi[2, 0] = -1
        with pytest.raises(qc.QCError) as e:
            qc.qc_tap_cluster(_cuda(X), _cuda(t), _cuda(subs), 0.5, k, 4, _cuda(q0), _cuda(badi), 20, final, per, work)
        assert e.value.code == -4 and "initial-centre" in str(e.value)
        q0z = q0.copy(); q0z[2] = 0.0
        with pytest.raises(qc.QCError) as e:
            qc.qc_tap_cluster(_cuda(X), _cuda(t), _cuda(subs), 0.5, k, 4, _cuda(q0z), _cuda(init), 20, final, per, work)
        assert e.value.code == -4 and "full rank" in str(e.value)
        Xneg = X.copy(); Xneg[: N // 2] *= -1.0                       # opposite halves, cosine weight 1: negative degrees
        with pytest.raises(qc.QCError) as e:
            qc.qc_tap_cluster(_cuda(Xneg), _cuda(t), _cuda(subs), 1.0, k, 4, _cuda(q0), _cuda(init), 20, final, per, work)
        assert e.value.code == -4
        # and the context-free library is usable afterwards
        qc.qc_tap_cluster(_cuda(X), _cuda(t), _cuda(subs), 0.5, k, 8, _cuda(q0), _cuda(init), 50, final, per, work)
        assert np.array_equal(final.cpu().numpy(), truth)


# ------------------------------------------------------------------------------------------------ edge cases
def test_edge_shapes(qc):
    """Smallest and degenerate shapes: iteration block = subsample = k, one cluster, one subsample, a pool smaller
    than a tile."""
    import torch
    # embedding with kb == n == k (the block spans the whole column space: no iteration needed, iters = 0)
    N, n, k = 40, 8, 8
    L, _ = _planted_L(N, 12, 4, n, seed=21)
    U, sig = torch.empty((N, k), device="cuda"), torch.empty(k, device="cuda")
    qc.qc_tap_embed(_cuda(L), k, 0, _cuda(TI.make_start_block(8, n, seed=22)), U, sig, _work(qc, N, 12, n, k, 8))
    Uo, so = tap.embed(L, k)
    lead = so > 1e-3 * so[0]                                          # trailing values sit at fp32 rounding level
    assert np.allclose(sig.cpu().numpy()[lead], so[lead], atol=2e-5)
    Ud = U.cpu().numpy().astype(np.float64)[:, lead]
    assert np.linalg.svd(Ud.T @ Uo[:, lead], compute_uv=False).min() >= 1 - 1e-4
    # k-means with one cluster: everything lands in it after one pass, the centre is the mean
    Uk = np.random.default_rng(23).standard_normal((33, 5)).astype(np.float32)
    labels, centres = torch.empty(33, dtype=torch.int32, device="cuda"), torch.empty((1, 5), device="cuda")
    passes = qc.qc_tap_kmeans(_cuda(Uk), _cuda(np.array([7], np.int32)), 10, labels, centres, _work(qc, 256, 8, 128, 1, 128))
    assert passes == 2 and labels.cpu().tolist() == [0] * 33
    assert np.allclose(centres.cpu().numpy()[0], Uk.astype(np.float64).mean(0), rtol=1e-6, atol=1e-7)
    # the whole algorithm with a single subsample: the merge is the identity
    N, F, k, n, kb = 150, 20, 3, 24, 8
    X, t, truth = TI.make_planted(N, F, k, seed=24)
    subs = TI.make_subsamples(N, n, 1, seed=25)
    init = np.array([[int(np.flatnonzero(truth == g)[0]) for g in range(k)]], dtype=np.int32)
    final, per = torch.empty(N, dtype=torch.int32, device="cuda"), torch.empty((1, N), dtype=torch.int32, device="cuda")
    qc.qc_tap_cluster(_cuda(X), _cuda(t), _cuda(subs), 0.5, k, 6, _cuda(TI.make_start_block(kb, n, seed=26)), _cuda(init), 30,
                      final, per, _work(qc, N, F, n, k, kb))
    assert torch.equal(final, per[0]) and np.array_equal(final.cpu().numpy(), truth)
    wf, _ = tap.tap(X, t, subs, 0.5, k, init, 30)
    assert np.array_equal(final.cpu().numpy(), wf)
    # similarity with the whole pool as subsample (n == N), N below one tile
    N, F = 24, 10
    X, t, _, _ = TI.make_pool(N, F, 50, 4, seed=27)
    idx = np.arange(N, dtype=np.int32)
    A = torch.empty((N, N), device="cuda")
    dr, dc = torch.empty(N, device="cuda"), torch.empty(N, device="cuda")
    qc.qc_tap_similarity(_cuda(X), _cuda(t), _cuda(idx), 0.7, A, dr, dc, _work(qc, N, F, N, 8, 8))
    want = tap.similarity(X, t, idx, 0.7)
    assert np.abs(A.cpu().numpy() - want).max() <= 2e-6
    assert np.allclose(dr.cpu().numpy(), want.sum(1), rtol=2e-6) and np.allclose(dc.cpu().numpy(), want.sum(0), rtol=2e-6)


# --------------------------------------------------------------------- forms that the sizes pick
@pytest.mark.parametrize("N,d,k", [
    (70000, 8, 4),            # ranges of 274 rows, two batches each; centres formed by the passes themselves (256 x 32 sums)
    (70000, 7, 6),            # the same ranges, element loads, centres by a kernel of their own
    (65536, 4, 10),           # the largest ranges of one batch, whose rows stay in LDS
    (5000, 13, 39),           # the same, element loads, more centres than a turn of the threads forms
    (2600, 31, 10),           # element loads, two chunks of 16 dimensions
    (1537, 24, 40),           # 6720 sums
    (1537, 24, 72),           # 12096: beyond the rule
    (600, 128, 128), (300, 5, 1), (257, 16, 16)])
def test_kmeans_forms(qc, N, d, k):
    import torch
    rng = np.random.default_rng(N + d + k)
    means = rng.standard_normal((k, d)) * 2
    U = (means[rng.integers(0, k, size=N)] + 0.8 * rng.standard_normal((N, d))).astype(np.float32)
    init = rng.choice(N, k, replace=False).astype(np.int32)
    if k > 2:
        U[init[1]] = U[init[0]]                    # equal centres: the second has no rows in the first pass
    labels, centres = torch.empty(N, dtype=torch.int32, device="cuda"), torch.empty((k, d), device="cuda")
    for limit in (1, 2, 10):
        wl, wc, wp = tap.kmeans(U, init, limit)
        passes = qc.qc_tap_kmeans(_cuda(U), _cuda(init), limit, labels, centres, _work(qc, max(N, 256), 8, 128, k, 128))
        if _check_labels(U, labels.cpu().numpy(), wl, wc) == 0:
            assert passes == wp
            assert np.allclose(centres.cpu().numpy(), wc, rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("N,F,n", [(211, 24, 191), (211, 24, 192), (211, 24, 193), (1701, 16, 1664), (1701, 16, 1665), (900, 20, 260)])
def test_degree_sums_of_every_width(qc, N, F, n):
    test_similarity_and_degrees(qc, N, F, n, 0.5, False)


@pytest.mark.parametrize("N,n,k,kb,iters", [
    (501, 64, 4, 8, 6), (601, 129, 5, 40, 4), (901, 300, 6, 72, 3),     # 1, 3 and 5 ranges: 64, 4800 and 25920 partial sums
    (1203, 520, 8, 112, 3), (655, 192, 5, 56, 3), (655, 193, 5, 32, 3)])
def test_embedding_of_every_block_size(qc, N, n, k, kb, iters):
    test_embedding_matches_singular_vectors(qc, N, n, k, kb, iters)


# ------------------------------------------------------------------------------------------- bits that stay
# Digests of an embedding and of a whole clustering (three subsamples), or "refused", a pool a row.  Lloyd's iteration amplifies the last
# bits of the embedding, which stands behind a matrix of condition up to 1e12, so another order of roundings in the Gram
# matrices, their factors or the rotations gives other labels (and refuses other pools of numerically deficient rank).
# The digests are those of the plain forms: one ascending chain of multiply-adds an entry and range, one column at a time, ranges of a multiple of 32
# elements, K split by the unpadded length.
DIGESTS = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "clustering_digests.txt")


def clustering_digests(qc, N, F, n, k, kb, alpha, slots):
    """Digests of the normalised matrix of the first subsample, of its embedding and of the clustering's labels."""
    import torch
    X, t, _, _ = TI.make_pool(N, F, 50, max(2, k * 4 // 5), seed=N + n)
    if alpha == 1.0:
        X = np.abs(X)                   # positive degrees; the matrix has at most F independent columns
    subs, init = TI.make_subsamples(N, n, 3, seed=N + k), TI.make_init(N, k, 3, seed=N + kb)
    X, t, subs, init, q0 = (_cuda(v) for v in (X, t, subs, init, TI.make_start_block(kb, n, seed=n + kb)))
    size = (qc.qc_tap_workspace_bytes(N, F, n, k, kb) + 255) // 256 * 256
    work = torch.empty(slots * size, dtype=torch.uint8, device="cuda")

    def digest(call, *outs):
        try:
            call()
        except qc.QCError as e:
            if e.code != -4:
                raise
            return "refused"
        return hashlib.sha1(b"".join(o.cpu().numpy().tobytes() for o in outs)).hexdigest()[:16]

    A, dr, dc = (torch.empty(shape, device="cuda") for shape in ((N, n), (N,), (n,)))

    def matrix():
        qc.qc_tap_similarity(X, t, subs[0], alpha, A, dr, dc, work)
        qc.qc_tap_normalise(A, dr, dc, work)

    U, sigma = torch.empty((N, k), device="cuda"), torch.empty(k, device="cuda")
    final, per = torch.empty(N, dtype=torch.int32, device="cuda"), torch.empty((3, N), dtype=torch.int32, device="cuda")
    return [digest(matrix, A), digest(lambda: qc.qc_tap_embed(A, k, 8, q0, U, sigma, work), U, sigma),
            digest(lambda: qc.qc_tap_cluster(X, t, subs, alpha, k, 8, q0, init, 100, final, per, work), final, per)]


@pytest.mark.parametrize("N,F,n,k,kb", [
    (70001, 8, 130, 4, 32),             # 256 ranges, two batches of rows each, centres formed by the passes: 768 workgroups for three
    (66000, 12, 129, 9, 40)])           # centres by a kernel of their own
def test_subsamples_of_a_group_equal_single_ones(qc, N, F, n, k, kb):
    """Per-subsample labels, one, two and three subsamples a launch."""
    import torch
    X, t, _, _ = TI.make_pool(N, F, 50, 6, seed=N)
    args = [_cuda(v) for v in (X, t, TI.make_subsamples(N, n, 3, seed=1))], _cuda(TI.make_start_block(kb, n, seed=2)), _cuda(TI.make_init(N, k, 3, seed=3))
    size = (qc.qc_tap_workspace_bytes(N, F, n, k, kb) + 255) // 256 * 256
    want = None
    for slots in (1, 2, 3, 3):
        work = torch.empty(slots * size, dtype=torch.uint8, device="cuda")
        final, per = torch.empty(N, dtype=torch.int32, device="cuda"), torch.empty((3, N), dtype=torch.int32, device="cuda")
        qc.qc_tap_cluster(*args[0], 0.5, k, 6, args[1], args[2], 60, final, per, work)
        want = want or (final, per)
        assert torch.equal(final, want[0]) and torch.equal(per, want[1]), slots


@pytest.mark.parametrize("row", [line.split() for line in open(DIGESTS) if not line.startswith("#")], ids=lambda r: "-".join(r[:6]))
def test_embeddings_and_labels_keep_their_bits(qc, row):
    N, F, n, k, kb, slots = (int(v) for v in row[:5] + [row[6]])
    assert clustering_digests(qc, N, F, n, k, kb, float(row[5]), slots) == row[7:]


@pytest.mark.parametrize("k,kind", [(1, "chain"), (2, "chain"), (7, "chain"), (100, "chain"), (128, "chain"), (128, "ties"), (33, "ties"), (64, "empty")])
def test_renaming_in_rounds(qc, k, kind):
    """Tables that need as many rounds as labels (every entry but the last is larger than the one that waits for it), equal counts
    (the lowest row and column first) and empty rows and columns."""
    import torch
    if kind == "chain":
        T = np.zeros((k, k), dtype=np.int64)
        for i in range(k):
            T[i, i] = 2 * (k - i)
            if i + 1 < k:
                T[i, i + 1] = 2 * (k - i) - 1
    elif kind == "ties":
        T = np.random.default_rng(k).integers(0, 3, size=(k, k))
    else:
        T = np.zeros((k, k), dtype=np.int64)
        T[3, 5] = T[5, 3] = T[9, 9] = 4
    perm_rows, perm_cols = np.random.default_rng(k + 1).permutation(k), np.random.default_rng(k + 2).permutation(k)
    T = T[perm_rows][:, perm_cols]
    a, b = np.repeat(np.arange(k * k) // k, T.ravel()), np.repeat(np.arange(k * k) % k, T.ravel())
    labels = np.stack([a, b]).astype(np.int32)
    N = labels.shape[1]
    out, perm = torch.empty(N, dtype=torch.int32, device="cuda"), torch.empty((2, k), dtype=torch.int32, device="cuda")
    qc.qc_tap_aggregate(_cuda(labels), k, out, _work(qc, 256, 8, 128, k, 128), perm)
    assert np.array_equal(perm.cpu().numpy()[1], tap.greedy_match(T))
    assert np.array_equal(out.cpu().numpy(), tap.aggregate(labels, k))


def test_small_clusterings_beside_a_sampler(qc):
    """Clusterings whose passes form the centres themselves (few sums), on one stream while a sampling run fills the chip from another, so
    that workgroups of a launch start late: the labels, centres and number of passes that they give alone."""
    import torch
    from synthetic import dit_inputs as I
    from qc_testlib import make_pair, oracle_calibration
    m = I.ModelDesc(depth=4, hidden=1152, heads=16, mlp_dim=4608, patch=2, latent_c=4, latent_h=32, latent_w=32)
    w, B = I.make_weights(m, 61), 24
    lat, lab = I.make_latents(B, m, 62), I.make_labels(B, m, 63)
    qp, _, _ = oracle_calibration(m, w, lat=lat[:1], lab=lab[:1], t=np.array([400]))
    _, ctx = make_pair(m, w, qp, B, 1)
    x, ld = _cuda(lat), _cuda(lab)

    problems = []
    for N, d, k, seed in ((70000, 8, 4, 1), (3000, 8, 12, 2), (1537, 24, 40, 3), (12345, 4, 40, 4)):
        rng = np.random.default_rng(seed)
        U = (rng.standard_normal((k, d))[rng.integers(0, k, size=N)] + 1.2 * rng.standard_normal((N, d))).astype(np.float32)
        init = rng.choice(N, k, replace=False).astype(np.int32)
        problems.append((_cuda(U), _cuda(init), k, _work(qc, max(N, 256), 8, 128, k, 128)))
    wl = TI.TAP_WORKLOADS["tap0"]
    kb = 32
    X, t, _, _ = TI.make_pool(wl.N, wl.F, wl.steps, wl.classes, wl.seed)
    pool = [_cuda(v) for v in (X, t, TI.make_subsamples(wl.N, wl.n, wl.m, wl.seed + 1), TI.make_start_block(kb, wl.n, wl.seed + 3),
                               TI.make_init(wl.N, wl.k, wl.m, wl.seed + 2))]
    base = (qc.qc_tap_workspace_bytes(wl.N, wl.F, wl.n, wl.k, kb) + 255) // 256 * 256
    work = torch.empty(3 * base, dtype=torch.uint8, device="cuda")

    def once():
        out = []
        for U, init, k, wk in problems:
            labels, centres = torch.empty(U.shape[0], dtype=torch.int32, device="cuda"), torch.empty((k, U.shape[1]), device="cuda")
            out += [qc.qc_tap_kmeans(U, init, 60, labels, centres, wk), labels, centres]
        final, per = torch.empty(wl.N, dtype=torch.int32, device="cuda"), torch.empty((wl.m, wl.N), dtype=torch.int32, device="cuda")
        qc.qc_tap_cluster(pool[0], pool[1], pool[2], wl.alpha, wl.k, 8, pool[3], pool[4], 100, final, per, work)
        return out + [final, per]

    want = once()
    torch.cuda.synchronize()
    side, done, beside = torch.cuda.Stream(), torch.cuda.Event(), 0
    for _ in range(3):
        with torch.cuda.stream(side):
            ctx.sample(x, ld, 20)
            done.record()
        for _ in range(40):
            got = once()
            assert all(a == b if isinstance(a, int) else torch.equal(a, b) for a, b in zip(got, want))
            if done.query():
                break
            beside += 1
        side.synchronize()
    assert beside >= 3
    ctx.close()
