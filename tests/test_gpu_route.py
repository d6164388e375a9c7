"""GPU parity of prefix routing against the oracle's fp64 argmin."""
import math

import numpy as np
import pytest
import torch

import dipaco_inputs as gen
import paper_2403_10616_amd as dp
from oracle import dipaco_oracle as orc
from gpu_util import DEV, dev, fma32, host, median_us, rel_l2

pytestmark = pytest.mark.gpu

TIE = 1e-4   # squared-distance gap below which fp32 and fp64 may legitimately order two centroids differently


def _run(z, c):
    N, D = z.shape
    K = c.shape[0]
    idx = torch.full((max(N, 1),), -1, dtype=torch.int32, device=DEV)
    hist = torch.full((K,), -7, dtype=torch.int64, device=DEV)
    margin = torch.zeros(max(N, 1), dtype=torch.float32, device=DEV)
    zd = dev(z) if N else torch.zeros((1, D), dtype=torch.float32, device=DEV)
    dp.dipaco_route_prefix(zd, dev(c), N, D, K, idx, hist, margin)
    return host(idx)[:N], host(hist), host(margin)[:N]


def _check(z, c, scale=1.0):
    idx, hist, margin = _run(z, c)
    o_idx, o_hist, o_margin = orc.route_prefix(z, c)
    clear = o_margin > TIE * scale
    assert np.array_equal(idx[clear], o_idx[clear])
    for n in np.nonzero(~clear)[0]:           # near-ties: the GPU's pick must be one of the oracle's two best
        d = ((z[n].astype(np.float64) - c.astype(np.float64)) ** 2).sum(1)
        assert idx[n] in np.argsort(d, kind="stable")[:2], (n, o_margin[n])
    assert hist.sum() == len(z) and np.array_equal(hist, np.bincount(idx, minlength=len(c)))
    moved = int((idx != o_idx).sum())
    assert np.abs(hist - o_hist).sum() <= 2 * moved
    fin = clear & np.isfinite(o_margin)
    assert np.abs(margin[fin] - o_margin[fin]).max(initial=0.0) <= 2e-4 * scale
    assert np.array_equal(np.isinf(margin), np.isinf(o_margin))
    return moved, int((~clear).sum())


@pytest.mark.parametrize("N,D,K", [(1000, 768, 256), (129, 64, 8), (4096, 32, 300), (777, 100, 1), (5, 4, 3),
                                   (2500, 768, 1000)])
def test_route_matches_oracle(N, D, K):
    print(f"route N={N} D={D} K={K}", flush=True)
    z, c, _ = gen.gaussian_mixture(N, D, K, 0.3, seed=4)
    _check(z, c)


def test_route_exact_ties_pick_lowest_index_and_empty_input():
    rng = np.random.default_rng(0)
    c = rng.integers(-3, 4, size=(16, 8)).astype(np.float32)
    c[11] = c[4]
    z = rng.integers(-3, 4, size=(300, 8)).astype(np.float32)
    z[:16] = c
    idx, hist, margin = _run(z, c)                   # small integers: fp32 scores are exact
    o_idx, o_hist, o_margin = orc.route_prefix(z, c)
    assert np.array_equal(idx, o_idx) and np.array_equal(hist, o_hist)
    assert np.array_equal(margin.astype(np.float64), o_margin)
    assert idx[11] == 4 and hist[11] == 0
    idx, hist, _ = _run(np.zeros((0, 8), np.float32), c)
    assert len(idx) == 0 and np.array_equal(hist, np.zeros(16, np.int64))


# ---- top-2 assignment, strided rows (product k-means), k-means update ----------------------------------------------
def _run_top(z_full, ldz, off, D, c, n_best):
    N = z_full.shape[0]
    K = c.shape[0]
    idx = torch.full((max(N, 1) * n_best,), -9, dtype=torch.int32, device=DEV)
    hist = torch.full((K,), -7, dtype=torch.int64, device=DEV)
    margin = torch.zeros(max(N, 1), dtype=torch.float32, device=DEV)
    dp.dipaco_route_prefix_top(dev(z_full), ldz, dev(c), N, D, K, n_best, idx, hist, margin, z_offset=off)
    out = host(idx)[:N * n_best]
    return (out.reshape(N, 2) if n_best == 2 else out), host(hist), host(margin)[:N]


@pytest.mark.parametrize("N,D,K", [(1000, 768, 256), (129, 64, 8), (777, 100, 1), (5, 4, 3), (2500, 64, 600)])
def test_route_top2_matches_oracle(N, D, K):
    print(f"route top2 N={N} D={D} K={K}", flush=True)
    z, c, _ = gen.gaussian_mixture(N, D, K, 0.3, seed=14)
    idx2, hist, margin = _run_top(z, D, 0, D, c, 2)
    o_idx2, o_hist = orc.route_prefix_top2(z, c)
    d = ((z.astype(np.float64)[:, None, :] - c.astype(np.float64)[None, :, :]) ** 2).sum(-1) if N * K <= 2_000_000 else None
    moved = 0
    for n in range(N):
        if np.array_equal(idx2[n], o_idx2[n]):
            continue
        moved += 1                                  # only near-ties may differ: compare distances, not indices
        dn = ((z[n].astype(np.float64) - c.astype(np.float64)) ** 2).sum(1) if d is None else d[n]
        assert idx2[n, 0] != idx2[n, 1]
        for j in range(2):
            assert abs(dn[idx2[n, j]] - dn[o_idx2[n, j]]) <= TIE, (n, j)
    assert moved <= max(2, N // 100)
    assert np.array_equal(hist, np.bincount(idx2[idx2 >= 0], minlength=K))
    assert np.abs(hist - o_hist).sum() <= 4 * moved
    if K > 1:
        o_margin = orc.route_prefix(z, c)[2]
        assert np.abs(margin - o_margin).max() <= 2e-4
    else:
        assert np.all(idx2[:, 1] == -1) and np.all(np.isinf(margin))


def test_route_top2_exact_ties_and_single_best_mode():
    rng = np.random.default_rng(1)
    c = rng.integers(-3, 4, size=(16, 8)).astype(np.float32)
    c[11] = c[4]
    z = rng.integers(-3, 4, size=(300, 8)).astype(np.float32)
    idx2, hist, _ = _run_top(z, 8, 0, 8, c, 2)          # small integers: fp32 scores are exact
    o_idx2, o_hist = orc.route_prefix_top2(z, c)
    assert np.array_equal(idx2, o_idx2) and np.array_equal(hist, o_hist)
    idx1, hist1, _ = _run_top(z, 8, 0, 8, c, 1)
    assert np.array_equal(idx1, o_idx2[:, 0]) and hist1.sum() == 300


def test_route_strided_halves_give_product_kmeans_pairs():
    """Product k-means: the two halves of the features are routed in place against their own centroid sets."""
    N, D, K = 700, 64, 12
    z, _, _ = gen.gaussian_mixture(N, D, K, 0.3, seed=15)
    c1 = gen.gaussian_mixture(1, D // 2, K, 0.3, seed=16)[1]
    c2 = gen.gaussian_mixture(1, D // 2, K, 0.3, seed=17)[1]
    i1, _, _ = _run_top(z, D, 0, D // 2, c1, 1)
    i2, _, _ = _run_top(z, D, D // 2, D // 2, c2, 1)
    o1, _, m1 = orc.route_prefix(z[:, :D // 2], c1)
    o2, _, m2 = orc.route_prefix(z[:, D // 2:], c2)
    assert np.array_equal(i1[m1 > TIE], o1[m1 > TIE]) and np.array_equal(i2[m2 > TIE], o2[m2 > TIE])
    pair = [dp.dipaco_path_index([int(a), int(b)], [K, K]) for a, b in zip(i1[:5], i2[:5])]
    assert pair == [int(a) * K + int(b) for a, b in zip(i1[:5], i2[:5])]


def _kmeans_gpu(z_full, ldz, off, D, idx, c_prev):
    N, K = z_full.shape[0], c_prev.shape[0]
    cd = dev(c_prev.copy())
    counts = torch.full((K,), -3, dtype=torch.int64, device=DEV)
    ws = torch.empty(dp.dipaco_kmeans_workspace_bytes(N, D, K), dtype=torch.uint8, device=DEV)
    zd = dev(z_full) if N else torch.zeros((1, max(ldz, 4)), dtype=torch.float32, device=DEV)
    idd = dev(idx.astype(np.int32)) if N else torch.zeros(1, dtype=torch.int32, device=DEV)
    dp.dipaco_kmeans_update(zd, ldz, idd, N, D, K, cd, counts, ws, z_offset=off)
    return host(cd), host(counts)


@pytest.mark.parametrize("N,D,K", [(5000, 768, 256), (3, 4, 2), (2049, 100, 7), (40000, 32, 300), (0, 8, 5),
                                   (9000, 1028, 3)])
def test_kmeans_update_matches_oracle(N, D, K):
    print(f"kmeans update N={N} D={D} K={K}", flush=True)
    z, c, _ = gen.gaussian_mixture(max(N, 1), D, K, 0.3, seed=24)
    z = z[:N]
    rng = np.random.default_rng(25)
    idx = rng.integers(0, K, size=N)
    if K > 2 and N > 0:
        idx[idx == 1] = 0                           # an empty cluster
    got, counts = _kmeans_gpu(z, D, 0, D, idx, c)
    want, o_counts = orc.kmeans_update(z, idx, c)
    assert np.array_equal(counts, o_counts)
    assert rel_l2(got, want) <= 1e-6
    assert np.abs(got - want).max() <= 1e-5
    empty = o_counts == 0
    assert np.array_equal(got[empty], c[empty])     # untouched, bit for bit
    again, _ = _kmeans_gpu(z, D, 0, D, idx, c)
    assert np.array_equal(got, again)               # fixed summation order


def test_kmeans_update_strided_rows_and_lloyd_iteration_lowers_objective():
    N, D, K = 6000, 48, 10
    z, c_true, _ = gen.gaussian_mixture(N, D, K, 0.3, seed=26)
    wide = np.zeros((N, 80), dtype=np.float32)
    wide[:, 16:16 + D] = z
    wide[:, :16] = 99.0                             # must not be read
    c = (c_true + 0.3 * np.random.default_rng(27).standard_normal(c_true.shape)).astype(np.float32)
    prev = np.inf
    for _ in range(3):
        idx, _, _ = _run_top(wide, 80, 16, D, c, 1)
        c, counts = _kmeans_gpu(wide, 80, 16, D, idx, c)
        obj = orc.kmeans_objective(z, idx, c)
        assert obj < prev
        prev = obj
        want, o_counts = orc.kmeans_update(z, idx, c)   # a fixed point of the update for this assignment
        assert rel_l2(c, want) <= 1e-6 and np.array_equal(counts, o_counts)


# ---- discriminative router: linear logistic classifier --------------------------------------------------------------
def _labelled_mixture(N, D, K, seed):
    z, c, comp = gen.gaussian_mixture(N, D, K, 0.3, seed=seed)
    return z, c, comp.astype(np.int32)


@pytest.mark.parametrize("N,D,K", [(1000, 768, 256), (130, 64, 8), (4100, 32, 304), (777, 104, 1), (5, 4, 3)])
def test_route_linear_matches_oracle(N, D, K):
    print(f"route_linear N={N} D={D} K={K}", flush=True)
    rng = np.random.default_rng(50 + K)
    z, c, _ = _labelled_mixture(N, D, K, 6)
    W = (2.0 * c + 0.05 * rng.standard_normal(c.shape)).astype(np.float32)
    b = (-(c.astype(np.float64) ** 2).sum(1) + 0.1 * rng.standard_normal(K)).astype(np.float32)
    idx = torch.full((N,), -1, dtype=torch.int32, device=DEV)
    hist = torch.full((K,), -7, dtype=torch.int64, device=DEV)
    margin = torch.zeros(N, dtype=torch.float32, device=DEV)
    dp.dipaco_route_linear(dev(z), D, dev(W), dev(b), N, D, K, idx, hist, margin)
    idx, hist, margin = host(idx), host(hist), host(margin)
    o_idx, o_hist, o_margin = orc.route_linear(z, W, b)
    clear = o_margin > TIE
    assert np.array_equal(idx[clear], o_idx[clear])
    for n in np.nonzero(~clear)[0]:           # near-ties: the GPU's pick must be one of the oracle's two best
        logit = W.astype(np.float64) @ z[n].astype(np.float64) + b
        assert idx[n] in np.argsort(-logit, kind="stable")[:2]
    assert hist.sum() == N and np.array_equal(hist, np.bincount(idx, minlength=K))
    fin = clear & np.isfinite(o_margin)
    assert np.abs(margin[fin] - o_margin[fin]).max(initial=0.0) <= 2e-4
    assert np.array_equal(np.isinf(margin), np.isinf(o_margin))


def test_route_linear_exact_ties_pick_lowest_index():
    rng = np.random.default_rng(1)
    W = rng.integers(-2, 3, size=(16, 8)).astype(np.float32)
    b = rng.integers(-2, 3, size=16).astype(np.float32)
    W[11], b[11] = W[4], b[4]
    z = rng.integers(-3, 4, size=(300, 8)).astype(np.float32)
    idx = torch.empty(300, dtype=torch.int32, device=DEV)
    hist = torch.empty(16, dtype=torch.int64, device=DEV)
    margin = torch.empty(300, dtype=torch.float32, device=DEV)
    dp.dipaco_route_linear(dev(z), 8, dev(W), dev(b), 300, 8, 16, idx, hist, margin)   # small integers: exact in fp32
    o_idx, o_hist, o_margin = orc.route_linear(z, W, b)
    assert np.array_equal(host(idx), o_idx) and np.array_equal(host(hist), o_hist)
    assert np.array_equal(host(margin).astype(np.float64), o_margin) and host(hist)[11] == 0


def _logistic(z, y, W, b, want_dw=True):
    N, D = z.shape
    K = W.shape[0]
    nbytes = dp.dipaco_router_workspace_bytes(N, D, K)
    assert nbytes > 0
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    loss = torch.zeros(4, dtype=torch.float32, device=DEV)
    dW = torch.full((K, D), 9.0, dtype=torch.float32, device=DEV) if want_dw else None
    db = torch.full((K,), 9.0, dtype=torch.float32, device=DEV)
    dp.dipaco_router_logistic_grad(dev(z), dev(y), dev(W), dev(b), N, D, K, loss, dW, db, ws, nbytes)
    return float(host(loss)[0]), (host(dW) if want_dw else None), host(db)


@pytest.mark.parametrize("N,D,K", [(1000, 768, 256), (129, 64, 8), (3000, 32, 304), (7, 8, 8), (2500, 104, 1000)])
def test_logistic_loss_and_gradients_match_oracle(N, D, K):
    print(f"logistic N={N} D={D} K={K}", flush=True)
    rng = np.random.default_rng(60 + K)
    z, c, y = _labelled_mixture(N, D, K, 8)
    y = y.copy()
    if N > 100:
        y[::97] = -1                                            # dropped documents
        y[5] = K
    W = (c + 0.1 * rng.standard_normal(c.shape)).astype(np.float32)
    b = (0.1 * rng.standard_normal(K)).astype(np.float32)
    loss, dW, db = _logistic(z, y, W, b)
    o_loss, o_dW, o_db = orc.logistic_loss_grad(z, y, W, b)
    assert abs(loss - o_loss) <= 1e-5 * max(1.0, abs(o_loss))
    assert rel_l2(dW, o_dW) <= 1e-5
    assert np.abs(db - o_db).max() <= 1e-6
    _, none_dW, db2 = _logistic(z, y, W, b, want_dw=False)        # bias-only mode
    assert none_dW is None and np.array_equal(db2, db)


@pytest.mark.parametrize("N,D,K", [(31, 8, 256), (33, 16, 200), (32768, 16, 256), (32769, 16, 256), (70001, 8, 120), (65568, 8, 8)])
def test_logistic_sums_over_several_rounds_of_rows(N, D, K):
    """Up to 1024 workgroups take 32 rows of 129 to 256 classes at a time, 64 of 65 to 128, 128 of 33 to 64, else 256: the sums of whole and ragged rounds."""
    test_logistic_loss_and_gradients_match_oracle(N, D, K)


@pytest.mark.parametrize("N,D,K", [(1, 8, 8), (15, 8, 64), (129, 8, 64), (131073, 8, 64), (130, 16, 72), (65, 8, 128), (65537, 8, 128),
                                   (63, 8, 136), (63, 8, 24), (257, 8, 32), (262145, 8, 16), (140000, 8, 40), (17, 8, 264), (33000, 8, 512),
                                   (5, 8, 520), (20000, 8, 1024), (9, 8, 1032)])
def test_logistic_rows_that_share_a_vector(N, D, K):
    """Eight rows of up to 32 classes, four of up to 64, two of up to 128, one above, which takes two vectors from 257 on and four
    from 513 on: ragged vectors and groups, one round of the workgroups and more."""
    test_logistic_loss_and_gradients_match_oracle(N, D, K)


@pytest.mark.parametrize("N,K", [(900, 256), (20000, 64), (40000, 120)])
def test_logistic_loss_is_off_by_little_more_than_its_rounding(N, K):
    """Over 24 draws, against 64 bits: rounding the result is off by 2^-24 / sqrt(3) at most (root mean square); half as much again is left for
    the rows' own errors and the spread of 24 draws."""
    D, errors = 8, []
    for seed in range(24):
        rng = np.random.default_rng(seed)
        z, W = rng.standard_normal((N, D)).astype(np.float32), (0.05 * (seed + 4) * rng.standard_normal((K, D))).astype(np.float32)
        b, y = rng.standard_normal(K).astype(np.float32), rng.integers(0, K, N).astype(np.int32)
        loss = _logistic(z, y, W, b, want_dw=False)[0]
        o_loss = orc.logistic_loss_grad(z, y, W, b)[0]
        errors.append((loss - o_loss) / o_loss)
    rms = float(np.sqrt(np.mean(np.square(errors))))
    print(f"logistic N={N} K={K}: rms error {rms:.2e}", flush=True)
    assert rms <= 1.5 * 2.0 ** -24 / 3 ** 0.5


@pytest.mark.parametrize("K", [64, 256, 264, 512, 1024])
def test_a_long_sum_of_like_rows_does_not_drift(K):
    """2^20 rows of the same probabilities (weights not yet trained): up to 256 rows a lane, which in one fp32 chain leave the bias gradient off by 6e-7
    (64 classes) to 3e-6 (1024) of the summands' magnitude.  Bound: four roundings of a row's own value (exponential, sum, quotient, product),
    alike in every row; 1.4e-7 - 1.6e-7 measured."""
    N, D = 1 << 20, 8
    rng = np.random.default_rng(K)
    b, y = rng.standard_normal(K).astype(np.float32), rng.integers(0, K, N).astype(np.int32)
    _, _, db = _logistic(np.zeros((N, D), np.float32), y, np.zeros((K, D), np.float32), b, want_dw=False)
    p = np.exp(b.astype(np.float64) - b.max())
    p /= p.sum()
    hits = np.bincount(y, minlength=K) / N
    off = float(np.abs((db - (p - hits)) / (p * (1.0 - hits) + (1.0 - p) * hits)).max())
    print(f"logistic bias gradient K={K}: off by {off:.2e} of the magnitudes", flush=True)
    assert off <= 4 * 2.0 ** -24


def test_bias_fit_on_gpu_gradients_matches_label_distribution_and_refills_empty_paths():
    """Weights frozen, bias descended with the GPU's dbias: the mean predicted distribution reaches the labels',
    and classes the unfitted classifier never picked get documents again."""
    rng = np.random.default_rng(70)
    N, D, K = 4000, 16, 8
    z = rng.standard_normal((N, D)).astype(np.float32)
    W = (0.3 * rng.standard_normal((K, D))).astype(np.float32)
    b0 = np.zeros(K, dtype=np.float32)
    b0[6:] = -3.0                                                 # classes 6, 7 start out nearly unreachable
    logits = z @ W.T
    y = np.argmax(logits + rng.gumbel(size=logits.shape), axis=1).astype(np.int32)   # labels spread over all classes
    q = np.bincount(y, minlength=K) / N
    b = b0.copy()
    for _ in range(400):
        _, _, db = _logistic(z, y, W, b, want_dw=False)
        b = (b - 4.0 * db).astype(np.float32)
    _, _, db = _logistic(z, y, W, b, want_dw=False)
    assert np.abs(db).max() < 2e-4                                # mean softmax - q
    o_db = orc.logistic_loss_grad(z, y, W, b)[2]
    assert np.abs(db - o_db).max() <= 1e-6
    h0 = orc.route_linear(z, W, b0)[1]
    idx = torch.empty(N, dtype=torch.int32, device=DEV)
    hist = torch.empty(K, dtype=torch.int64, device=DEV)
    dp.dipaco_route_linear(dev(z), D, dev(W), dev(b), N, D, K, idx, hist, None)
    h1 = host(hist)
    assert h0[6:].sum() < 0.2 * N * q[6:].sum() and h1[6:].sum() > 0.5 * N * q[6:].sum()


def test_router_entry_points_reject_bad_arguments():
    t = torch.zeros(64, dtype=torch.float32, device=DEV)
    i = torch.zeros(64, dtype=torch.int32, device=DEV)
    h = torch.zeros(8, dtype=torch.int64, device=DEV)
    assert dp.dipaco_router_workspace_bytes(8, 12, 8) == 0 and dp.dipaco_router_workspace_bytes(8, 8, 12) == 0
    with pytest.raises(dp.DipacoError):
        dp.dipaco_router_logistic_grad(t, i, t, t, 8, 8, 8, t, t, t, t, 16)         # workspace too small
    with pytest.raises(dp.DipacoError):
        dp.dipaco_route_linear(t, 6, t, t, 8, 8, 8, i, h, None)                     # ldz < D
    with pytest.raises(dp.DipacoError):
        dp.dipaco_route_linear(t, 8, t, None, 8, 8, 8, i, h, None)                  # bias missing


# ---- routing more often at evaluation -------------------------------------------------------------------------------
@pytest.mark.parametrize("P,B,S,L,W", [(4, 3, 300, 64, 128), (16, 16, 2048, 1024, 128), (1, 2, 5, 3, 2), (5, 2, 257, 1000, 257),
                                       (3, 40, 17, 1, 1)])
def test_window_targets_and_chunk_routed_scores_match_oracle(P, B, S, L, W):
    print(f"reroute P={P} B={B} S={S} L={L} W={W}", flush=True)
    rng = np.random.default_rng(80 + P)
    nll = rng.uniform(0.2, 9.0, size=(P, B, S)).astype(np.float32)
    nll[:, :, ::11] = 0.0                                         # ignored positions
    if P > 2:
        nll[2, 0] = nll[0, 0]                                     # exact ties on one document: lowest path wins
    nbytes = dp.dipaco_reroute_workspace_bytes(P, B, S)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    tg = torch.full((B, S), -1, dtype=torch.int32, device=DEV)
    nd = dev(nll)
    dp.dipaco_window_targets(nd, P, B, S, L, tg, ws, nbytes)
    got = host(tg)
    scores = -nll.astype(np.float64)
    want = orc.window_targets(scores, L)
    diff = np.argwhere(got != want)
    for b, j in diff:            # a different label must be a tie up to the rounding of a window sum of fp64 values
        hi = min(S, j + L)
        assert abs(scores[got[b, j], b, j:hi].sum() - scores[want[b, j], b, j:hi].sum()) <= 1e-9
    assert len(diff) <= 0.001 * B * S
    if P > 2:
        assert not np.any(got[0] == 2)
    n_chunks = (S + W - 1) // W
    choice = np.stack([want[:, min(S - 1, c * W)] for c in range(n_chunks)], axis=1).astype(np.int32)
    out = torch.zeros(B, dtype=torch.float32, device=DEV)
    dp.dipaco_chunk_routed_score(nd, dev(choice), P, B, S, W, out, ws, nbytes)
    o = orc.chunk_routed_scores(scores, choice, W)
    assert np.abs(host(out) - o).max() <= 1e-6 * np.abs(o).max()
    # one chunk, path 0 for every document: the plain document score
    dp.dipaco_chunk_routed_score(nd, dev(np.zeros((B, 1), np.int32)), P, B, S, S, out, ws, nbytes)
    assert np.abs(host(out) + nll[0].astype(np.float64).sum(1)).max() <= 1e-6 * nll[0].sum(1).max()
    with pytest.raises(dp.DipacoError):
        dp.dipaco_window_targets(nd, P, B, S, 0, tg, ws, nbytes)
    with pytest.raises(dp.DipacoError):
        dp.dipaco_chunk_routed_score(nd, dev(choice), P, B, S, W, out, ws, 8)


# ---- exact comparison on integer points over many ragged shapes --------------------------------------------------
_EXACT_SHAPES = [(1, 4, 1), (2, 4, 2), (255, 8, 7), (256, 8, 64), (257, 12, 65), (511, 4, 255), (513, 36, 256),
                 (700, 8, 257), (1025, 32, 300), (300, 40, 511), (64, 4, 513), (2049, 8, 33), (90, 68, 1030)]


@pytest.mark.parametrize("N,D,K", _EXACT_SHAPES)
def test_route_and_top2_are_exact_on_integer_points(N, D, K):
    """Small-integer coordinates make every fp32 score exact, and ties between centroids are the rule: the kernel's
    selection (fold over a lane's columns, reduction over the lanes of a row, merge of the waves and of the centroid
    tiles) must then give the oracle's indices, histogram and margins bit for bit, whatever part of a tile is empty."""
    print(f"exact route N={N} D={D} K={K}", flush=True)
    rng = np.random.default_rng(1000 * N + K)
    z = rng.integers(-2, 3, size=(N, D)).astype(np.float32)
    c = rng.integers(-2, 3, size=(K, D)).astype(np.float32)
    idx, hist, margin = _run(z, c)
    o_idx, o_hist, o_margin = orc.route_prefix(z, c)
    assert np.array_equal(idx, o_idx) and np.array_equal(hist, o_hist)
    assert np.array_equal(margin.astype(np.float64), o_margin)
    idx2, hist2, margin2 = _run_top(z, D, 0, D, c, 2)
    o_idx2, o_hist2 = orc.route_prefix_top2(z, c)
    assert np.array_equal(idx2, o_idx2) and np.array_equal(hist2, o_hist2)
    assert np.array_equal(margin2.astype(np.float64), o_margin)


def test_rows_without_a_nearest_centroid_go_to_centroid_zero_with_nan_margin():
    """A document whose features hold a NaN (a diverged path) has no nearest centroid: every score is NaN.  The library
    routes it to centroid 0 (second choice 1), counts it there and marks it with a NaN margin -- what the plain
    definition's argmin over a row of NaN distances gives -- and the other rows are not disturbed.  Infinite features
    also end in NaN scores when they meet centroid entries of both signs; a row they leave with scores of -inf gets
    some index in range, and the histogram stays consistent."""
    print("route: rows with NaN / infinite features", flush=True)
    z, c, _ = gen.gaussian_mixture(700, 64, 40, 0.3, seed=9)
    bad = [3, 255, 699]
    z[3, 5] = np.nan
    z[255, :] = np.inf
    z[699, 63] = np.nan
    z[256, 0] = -np.inf                      # one infinite entry: unspecified, but in range and counted once
    good = np.setdiff1d(np.arange(700), bad + [256])
    idx, hist, margin = _run(z, c)
    with np.errstate(invalid="ignore"):
        o_idx, o_hist, o_margin = orc.route_prefix(z, c)
    assert np.array_equal(o_idx[bad], [0, 0, 0]) and np.all(np.isnan(o_margin[bad]))      # the definition's own answer
    assert np.array_equal(idx[bad], [0, 0, 0]) and np.all(np.isnan(margin[bad]))
    assert np.array_equal(idx[good], o_idx[good]) and 0 <= idx[256] < 40
    assert hist.sum() == 700 and np.array_equal(hist, np.bincount(idx, minlength=40))
    # top-2 form: (0, 1) for such rows, both memberships counted
    idx2 = torch.full((700 * 2,), -5, dtype=torch.int32, device=DEV)
    hist2 = torch.full((40,), -7, dtype=torch.int64, device=DEV)
    m2 = torch.zeros(700, dtype=torch.float32, device=DEV)
    dp.dipaco_route_prefix_top(dev(z), 64, dev(c), 700, 64, 40, 2, idx2, hist2, m2)
    i2 = host(idx2).reshape(700, 2)
    with np.errstate(invalid="ignore"):
        o2, _ = orc.route_prefix_top2(z, c)
    assert np.array_equal(o2[[3, 699]], [[0, 1]] * 2)          # NaN rows: the definition's own answer
    assert np.array_equal(i2[bad], [[0, 1]] * 3) and np.all(np.isnan(host(m2)[bad]))
    assert np.array_equal(i2[good], o2[good]) and i2[256].min() >= 0 and i2[256].max() < 40
    assert np.array_equal(host(hist2), np.bincount(i2.ravel(), minlength=40)) and host(hist2).sum() == 1400


@pytest.mark.parametrize("N,D,K,bias", [
    (4096, 36, 256, False), (16, 4, 33, False), (1, 896, 129, True), (30000, 20, 32, False),      # 16 points per wave
    (4097, 36, 256, False), (40001, 100, 20, False), (9000, 20, 65, True), (70000, 20, 257, False),   # 32 points per wave
    (66000, 16, 256, False), (140000, 12, 250, True),                                              # 256 points per workgroup
])
def test_route_kernels_agree_with_fp64_on_both_sides_of_every_size_rule(N, D, K, bias):
    """Integer points and centroids: every fp32 score is exact (|score| < 2^24), so indices, ties, counts and margins are."""
    print(f"route rule N={N} D={D} K={K} bias={bias}", flush=True)
    g = torch.Generator().manual_seed(N + K)
    z = torch.randint(-3, 4, (N, D), generator=g).float().to(DEV)
    c = torch.randint(-3, 4, (K, D), generator=g).float().to(DEV)
    b = torch.randint(-5, 6, (K,), generator=g).float().to(DEV)
    score = -(z.double() @ c.double().T + b.double()) if bias else (c.double() ** 2).sum(1) - 2 * z.double() @ c.double().T
    order = torch.sort(score, dim=1, stable=True)
    for n_best in ((1,) if bias else (1, 2)):
        idx = torch.full((N * n_best,), -9, dtype=torch.int32, device=DEV)
        hist = torch.full((K,), -7, dtype=torch.int64, device=DEV)
        margin = torch.zeros(N, device=DEV)
        if bias:
            dp.dipaco_route_linear(z, D, c, b, N, D, K, idx, hist, margin)
        else:
            dp.dipaco_route_prefix_top(z, D, c, N, D, K, n_best, idx, hist, margin)
        want = order.indices[:, :n_best].reshape(-1)
        assert torch.equal(idx.long(), want)
        assert torch.equal(hist, torch.bincount(want, minlength=K))
        assert torch.equal(margin.double(), order.values[:, 1] - order.values[:, 0])


@pytest.mark.parametrize("N,D,K,bias", [(45000, 64, 129, False), (45057, 36, 256, True), (50001, 100, 257, False), (41500, 896, 200, False),
                                        (45056, 4, 130, True), (45000, 16, 4096, False)])
def test_tiles_of_bf16_parts_route_as_fp64_does(N, D, K, bias):
    """128 points x 128 centroids a tile, whole ones and remainders in points, centroids and features.  Whole numbers are one bf16
    part each, so every score is exact, and so are those of the ties, which are taken again in fp32."""
    test_route_kernels_agree_with_fp64_on_both_sides_of_every_size_rule(N, D, K, bias)


def test_tiles_of_bf16_parts_with_values_that_are_not_finite():
    """An infinity has no bf16 parts that multiply as it does: points that meet one are taken again in fp32.  Expected: the smallest score that is
    not NaN, the lowest index among equals; rows without one go to centroid 0 with a NaN margin."""
    N, D, K = 45000, 68, 130
    g = torch.Generator().manual_seed(5)
    z = torch.randint(-3, 4, (N, D), generator=g).float()
    c = torch.randint(1, 4, (K, D), generator=g).float()
    z[5, 3], z[700, 67], z[701, 0] = math.inf, -math.inf, math.nan
    z[900, 1], z[900, 2] = math.inf, -math.inf
    z[1234, 7] = 3.4e38              # finite, but its first bf16 part is not
    c[129, 5] = math.inf             # never the nearest
    z[0:N:97, 5] = 0.0               # 0 x inf
    score = (c.double() ** 2).sum(1) - 2 * z.double() @ c.double().T
    score = torch.where(score.isnan(), math.inf, score)
    order = torch.sort(score, dim=1, stable=True)
    idx, hist, margin = (torch.empty(N, dtype=torch.int32, device=DEV), torch.empty(K, dtype=torch.int64, device=DEV),
                         torch.empty(N, device=DEV))
    dp.dipaco_route_prefix(z.to(DEV), c.to(DEV), N, D, K, idx, hist, margin)
    idx, margin = idx.cpu().long(), margin.cpu()
    none = order.values[:, 0] == math.inf
    assert none.nonzero().flatten().tolist() == [700, 701, 900] and bool((idx[none] == 0).all()) and bool(margin[none].isnan().all())
    plain = ~none & order.values[:, 0].isfinite()
    plain[1234] = False              # every score beyond fp32: -inf
    assert torch.equal(idx[plain], order.indices[plain, 0])
    assert torch.equal(margin[plain].double(), (order.values[:, 1] - order.values[:, 0])[plain])
    assert idx[5] == 0 and idx[1234] == 0
    assert torch.equal(hist.cpu(), torch.bincount(idx, minlength=K))


def _near_tie_groups(linear, N, D, K, seed):
    """Centroids in groups whose scores lie 1e-5 apart for every point: two that differ in feature 3, in the lower half four that differ in
    features 3 and 29.  linear: weights and a bias, and points with a common offset that the bias takes out of the scores again."""
    rng = np.random.default_rng(seed)
    c = (rng.standard_normal((K, D)) * 4).astype(np.float32)
    k = np.arange(K)
    first = np.where(k < K // 2, k // 4 * 4, k // 2 * 2)
    c = c[first]
    c[:, 3] = 2 + k % 2
    c[: K // 2, 29] = -5 + k[: K // 2] // 2 % 2
    z = rng.standard_normal((N, D)).astype(np.float32)
    bias = None
    if linear:
        z += np.float32(4)
        rest = np.delete(c.astype(np.float64), (3, 29), axis=1).sum(1)
        bias = (-4.0 * rest - 2.5 * c[:, 3] + 4.5 * c[:, 29]).astype(np.float32)
    z[:, 3] = 2.5 + rng.standard_normal(N) * 1e-5
    z[:, 29] = -4.5 + rng.standard_normal(N) * 1e-5
    return z, c, bias


def _chain_norm(c):
    """|c|^2 as the kernels add it: pieces of four features, each eighth piece into one of eight sums, then a tree."""
    sums = np.zeros((8, len(c)), np.float32)
    for p in range(c.shape[1] // 4):
        x, y, z, w = c[:, 4 * p:4 * p + 4].T
        sums[p % 8] += fma32(w, w, fma32(z, z, fma32(y, y, x * x)))
    pairs = sums[0::2] + sums[1::2]
    return (pairs[0] + pairs[1]) + (pairs[2] + pairs[3])


@pytest.mark.parametrize("form", ["nearest", "two nearest", "linear"])
@pytest.mark.parametrize("D", [64, 100])
def test_near_ties_of_bf16_parts_are_decided_by_the_fp32_instruction(form, D):
    """Every point is a near-tie of two or four centroids that a chain of fp32 multiply-adds orders differently from 64 bits for many
    points.  The answers are those of the chain, bit for bit: indices, and the gaps of the two best."""
    N, K = 45000, 256
    z, c, bias = _near_tie_groups(form == "linear", N, D, K, 8)
    score = -(z.astype(np.float64) @ c.T + bias) if form == "linear" else (c.astype(np.float64) ** 2).sum(1) - 2 * z.astype(np.float64) @ c.T
    best = np.argsort(score, axis=1, kind="stable")[:, :6]
    best.sort(axis=1)                                        # ties go to the lower index
    s64 = np.sort(np.take_along_axis(score, best, 1), axis=1)
    four = score.argmin(1) < K // 2
    apart = np.where(four, s64[:, 4], s64[:, 2]) - s64[:, 0] > 1e-2   # the next group is not in the tie
    rows = np.nonzero(apart)[0][:12000]
    cand = best[rows]
    dot = np.zeros(cand.shape, np.float32)
    for base in range(0, D, 8):                              # the order of v_mfma_f32_32x32x2_f32 over chunks of four
        for k in (0, 4, 1, 5, 2, 6, 3, 7):
            if base + k < D:
                dot = fma32(np.broadcast_to(z[rows, base + k][:, None], dot.shape), c[cand, base + k], dot)
    start = -bias[cand] if form == "linear" else _chain_norm(c)[cand]
    s32 = fma32(np.full_like(dot, -1.0 if form == "linear" else -2.0), dot, start)
    order = np.argsort(s32, axis=1, kind="stable")
    want = np.take_along_axis(cand, order, 1)
    gap = np.take_along_axis(s32, order, 1)
    gap = gap[:, 1] - gap[:, 0]
    turned = want[:, 0] != score[rows].argmin(1)
    assert turned.sum() > 100 and turned[four[rows]].sum() > 50, (turned.sum(), turned[four[rows]].sum())
    n_best = 2 if form == "two nearest" else 1
    idx, hist, margin = (torch.empty((N, n_best), dtype=torch.int32, device=DEV), torch.empty(K, dtype=torch.int64, device=DEV),
                         torch.empty(N, device=DEV))
    if form == "linear":
        dp.dipaco_route_linear(dev(z), D, dev(c), dev(bias), N, D, K, idx, hist, margin)
    else:
        dp.dipaco_route_prefix_top(dev(z), D, dev(c), N, D, K, n_best, idx, hist, margin)
    got = host(idx)
    assert np.array_equal(got[rows], want[:, :n_best])
    assert np.array_equal(host(margin)[rows], gap)
    assert np.array_equal(host(hist), np.bincount(got.ravel(), minlength=K))


@pytest.mark.parametrize("linear", [False, True])
def test_centroids_of_small_numbers_keep_their_bits(linear):
    """Centroids (weights) around 2^-118: three bf16 parts hold 16 bits of them, the fp32 instruction 24.  Gaps err by a few 2^-24 of the
    sums, D 2^-24 of the absolute products at the most."""
    N, D, K = 45000, 64, 256
    rng = np.random.default_rng(9)
    z = rng.standard_normal((N, D)).astype(np.float32)
    c = (rng.standard_normal((K, D)) * 2.0 ** -118).astype(np.float32)
    dot = z.astype(np.float64) @ c.T.astype(np.float64)
    score = -dot if linear else (c.astype(np.float64) ** 2).sum(1) - 2 * dot
    order = np.argsort(score, axis=1)
    gap = np.take_along_axis(score, order, 1)
    gap = gap[:, 1] - gap[:, 0]
    idx, hist, margin = torch.empty(N, dtype=torch.int32, device=DEV), torch.empty(K, dtype=torch.int64, device=DEV), torch.empty(N, device=DEV)
    if linear:
        dp.dipaco_route_linear(dev(z), D, dev(c), torch.zeros(K, device=DEV), N, D, K, idx, hist, margin)
    else:
        dp.dipaco_route_prefix(dev(z), dev(c), N, D, K, idx, hist, margin)
    bound = 2 * 2 * math.sqrt(D) * 2.0 ** -24 * np.linalg.norm(z, axis=1) * np.linalg.norm(c.astype(np.float64), axis=1).max()
    clear = gap > bound
    assert clear.mean() > 0.99
    assert np.array_equal(host(idx)[clear], order[clear, 0])
    assert (np.abs(host(margin) - gap) <= bound).all()


def test_rows_that_are_not_finite_do_not_hold_the_others_up():
    """Rows of NaN have no scores and are not multiplied again; infinite ones are, by their wave alone."""
    N, D, K = 65536, 256, 256
    g = torch.Generator().manual_seed(5)
    z, c = torch.randn((N, D), generator=g).to(DEV), torch.randn((K, D), generator=g).to(DEV)
    idx, hist = torch.empty(N, dtype=torch.int32, device=DEV), torch.empty(K, dtype=torch.int64, device=DEV)
    run = lambda: dp.dipaco_route_prefix(z, c, N, D, K, idx, hist, None)
    finite = median_us(run)
    want = idx.clone()
    z[::64, 3] = math.nan
    times = [median_us(run)]
    keep = torch.arange(N, device=DEV) % 64 != 0
    assert torch.equal(idx[keep], want[keep]) and not bool(idx[~keep].any())
    z[::64, 3] = math.inf
    times.append(median_us(run))
    assert torch.equal(idx[keep], want[keep])
    print(f"route us finite {finite:.0f} NaN {times[0]:.0f} infinite {times[1]:.0f}", flush=True)
    assert times[0] <= 1.5 * finite and times[1] <= 6 * finite


@pytest.mark.parametrize("D,K", [(4, 3), (28, 64), (36, 65), (896, 128), (100, 129), (32, 256), (64, 257), (256, 1000)])
def test_a_batch_routes_as_its_points_do_among_others(D, K):
    """Batches of up to 256, 512 or 1024 points (by K) have a kernel of their own, whose scores are those of the larger ones' bit for bit."""
    N = 1100
    rng = np.random.default_rng(K)
    z, c = (rng.standard_normal((n, D)).astype(np.float32) for n in (N, K))
    z[7, D - 1], z[9, 0] = np.nan, np.inf
    c[K // 2] = c[0]
    bias = dev(rng.standard_normal(K).astype(np.float32))
    zd, cd = dev(z), dev(c)

    def route(lo, hi, form):
        n = hi - lo
        idx = torch.full((n, 2) if form == "two nearest" else (n,), -7, dtype=torch.int32, device=DEV)
        hist, gap = torch.full((K,), -7, dtype=torch.int64, device=DEV), torch.empty(n, dtype=torch.float32, device=DEV)
        if form == "linear":
            dp.dipaco_route_linear(zd[lo:hi], D, cd, bias, n, D, K, idx, hist, gap)
        else:
            dp.dipaco_route_prefix_top(zd[lo:hi], D, cd, n, D, K, idx.numel() // n, idx, hist, gap)
        assert np.array_equal(host(hist), np.bincount(host(idx).ravel(), minlength=K))
        return host(idx), host(gap).view(np.int32)

    for form in ("nearest", "two nearest", "linear"):
        idx, gap = route(0, N, form)
        nan = np.isnan(gap.view(np.float32))
        lo = 0
        for n in (1, 2, 3, 8, 65, 255, 256):   # each starts behind the one before; one and two points a wave, a last wave that is not full
            got_idx, got_gap = route(lo, lo + n, form)
            assert np.array_equal(got_idx, idx[lo:lo + n]) and np.array_equal(got_gap[~nan[lo:lo + n]], gap[lo:lo + n][~nan[lo:lo + n]])
            lo += n
        for n in (257, 511, 512, 513, 1023, 1024, 1025):
            got_idx, got_gap = route(0, n, form)
            assert np.array_equal(got_idx, idx[:n]) and np.array_equal(got_gap[~nan[:n]], gap[:n][~nan[:n]])


def test_points_of_one_centroid_take_a_batch_no_longer():
    """Added to a histogram in memory, 1800 indices of the same line are 27 us; 64 points take 11."""
    D, K = 64, 4
    c = np.random.default_rng(3).standard_normal((K, D)).astype(np.float32)
    times = {}
    for N in (64, 900):
        idx, hist = torch.empty((N, 2), dtype=torch.int32, device=DEV), torch.empty(K, dtype=torch.int64, device=DEV)
        z, cd = dev(np.repeat(c[1:2], N, axis=0)), dev(c)
        times[N] = median_us(lambda: dp.dipaco_route_prefix_top(z, D, cd, N, D, K, 2, idx, hist, None), n=50)
        assert host(hist)[1] == N and host(hist).sum() == 2 * N and (host(idx)[:, 0] == 1).all()
    print(f"two nearest of 4: 64 points {times[64]:.1f} us, 900 {times[900]:.1f}", flush=True)
    assert times[900] <= 1.5 * times[64]


def test_more_points_than_one_launch_of_small_workgroups_holds():
    """600,000,000 points and 100 centroids: 64 points a workgroup of 512 threads would pass 2^32 threads in a launch."""
    N, D, K = 600_000_000, 4, 100
    g = torch.Generator(DEV).manual_seed(3)
    c = torch.randint(-9, 10, (K, D), generator=g, device=DEV).float()
    z = torch.empty((N, D), device=DEV).normal_(generator=g).mul_(4.0).round_()
    idx = torch.full((N,), -9, dtype=torch.int32, device=DEV)
    hist = torch.full((K,), -7, dtype=torch.int64, device=DEV)
    dp.dipaco_route_prefix(z, c, N, D, K, idx, hist, None)
    assert int(hist.sum()) == N
    for at in (0, N // 2, N - 4096):     # whole numbers: scores and ties are exact
        part = z[at:at + 4096].double()
        score = (c.double() ** 2).sum(1) - 2 * part @ c.double().T
        assert torch.equal(idx[at:at + 4096].long(), torch.sort(score, dim=1, stable=True).indices[:, 0])


def test_window_labels_of_more_documents_than_one_launch_holds():
    """17,000,000 documents x 1 position: a workgroup of threads per document and path passes 2^32 threads in a launch."""
    P, B = 2, 17_000_000
    nll = torch.rand((P, B, 1), device=DEV, generator=torch.Generator(DEV).manual_seed(4))
    nbytes = dp.dipaco_reroute_workspace_bytes(P, B, 1)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    labels = torch.full((B, 1), -3, dtype=torch.int32, device=DEV)
    dp.dipaco_window_targets(nll, P, B, 1, 1, labels, ws, nbytes)
    want = (nll[1, :, 0] < nll[0, :, 0]).long()
    assert torch.equal(labels[:, 0].long(), want)
    out = torch.full((B,), 9.0, device=DEV)
    dp.dipaco_chunk_routed_score(nll, labels, P, B, 1, 1, out, ws, nbytes)
    assert torch.equal(out, -nll[:, :, 0].amin(0))
