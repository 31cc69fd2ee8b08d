"""Sizer calls beyond the kept workspaces: small calls are staged through pinned memory, larger ones copy
from and to the caller's arrays, the largest also allocate device memory of their own.  Every size against
the FP64 reference, small calls between large ones on one sizer, and no size class that is slow for its
number of samples."""
import time

import numpy as np
import pytest

from oracle import mlp_ref as R
from tests.test_sizer import _magnitudes

pytestmark = pytest.mark.gpu


# staging ends at 2^18 floats in and out, kept device memory at 2^24 floats: per sample 22 + K and
# 22 + 3 K + 4 H of them
@pytest.mark.parametrize("H,K,sizes", [(4, 2, (100, 10922, 10923, 381000, 390000, 99)), (64, 8, (8738, 8739, 51000, 58000, 50))])
def test_predictions_around_the_limits(H, K, sizes):
    import paper_2609_32308_amd as sd
    ctx = sd.Context(0)
    z = sd.Sizer(ctx, H, K, seed=5)
    flat = z.get_params()
    for n in sizes:
        print("sizer", H, K, "samples", n, flush=True)
        X = np.random.default_rng(n).random((n, 22)).astype(np.float32)
        Y = np.full((n, K), 0.25, np.float32)
        _, _, ry = R.loss_and_grad(flat, X, Y, H, K)
        _, mag_y, _ = _magnitudes(flat, X, Y, H, K)
        # FP32 rounding of each term and sum, per entry
        assert np.all(np.abs(z.predict(X) - ry) <= 4 * (H + 26) * 2.0 ** -24 * mag_y + 2e-7)
        loss, g = z.gradient(X, Y)
        l2, g2 = z.gradient(X, Y)
        assert loss == l2 and np.array_equal(g, g2)
        assert abs(loss - np.mean((ry - Y) ** 2)) <= 1e-5 * max(1e-3, loss)
    ctx.close()


def rows_clear_of_kinks(n, K, flat, H, seed):
    """Random rows whose FP64 pre-activations all sit clear of the ReLU kink."""
    W1, b1, W2, b2, _, _ = R.unpack(flat, H, K)
    rng = np.random.default_rng(seed)
    X = np.zeros((0, 22), np.float32)
    while len(X) < n:
        x = rng.random((4 * n, 22)).astype(np.float32)
        z1 = x.astype(np.float64) @ W1.T + b1
        z2 = np.maximum(z1, 0.0) @ W2.T + b2
        X = np.concatenate([X, x[np.minimum(np.abs(z1).min(1), np.abs(z2).min(1)) > 1e-4]])
    return X[:n], rng.random((n, K)).astype(np.float32)


# a layer of H * H + H sums is split into at most 2^18 / (H * H + H) chunks: 6 of up to 33, 34 and 67
# samples, the last one ragged; 63 of up to 72
@pytest.mark.parametrize("H,K,n", [(200, 1, 193), (200, 1, 200), (200, 1, 400), (64, 8, 4500)])
def test_gradient_with_as_many_chunks_as_allowed(H, K, n):
    import paper_2609_32308_amd as sd
    ctx = sd.Context(0)
    z = sd.Sizer(ctx, H, K, seed=3)
    flat = z.get_params()
    X, Y = rows_clear_of_kinks(n, K, flat, H, n)
    print("sizer", H, K, "samples", n, flush=True)
    loss, g = z.gradient(X, Y)
    rl, rg, _ = R.loss_and_grad(flat, X, Y, H, K)
    mag, _, _ = _magnitudes(flat, X, Y, H, K)
    assert abs(loss - rl) <= 1e-5 * max(1e-3, abs(rl))
    # FP32 rounding of each term and sum, per entry, as for the chunks of 32 samples
    tol = 4 * (max(n, H, 22) + 4) * 2.0 ** -24 * mag + 1e-4 * np.abs(rg) + 1e-12
    bad = np.flatnonzero(np.abs(g - rg) > tol)
    assert bad.size == 0, (bad[:10], g[bad[:10]], rg[bad[:10]])
    ctx.close()


def test_smallest_network_with_the_most_samples():
    # two parameters in the last layer: more chunks of 32 samples than a launch has workgroups in y
    import paper_2609_32308_amd as sd
    n, H, K = 65535 * 32 + 40000, 1, 1
    ctx = sd.Context(0)
    z = sd.Sizer(ctx, H, K, seed=5)
    flat = z.get_params()
    rng = np.random.default_rng(3)
    X, Y = rng.random((n, 22), np.float32), rng.random((n, K), np.float32)
    print("sizer", H, K, "samples", n, flush=True)
    loss, g = z.gradient(X, Y)
    rl, rg, _ = R.loss_and_grad(flat, X, Y, H, K)
    mag, _, _ = _magnitudes(flat, X, Y, H, K)
    # a chunk's sum, then the chunks' sums, and the terms of each sample
    tol = 4 * (64 + 65535 + 22) * 2.0 ** -24 * mag + 1e-12
    assert abs(loss - rl) <= 1e-3 * rl
    assert np.all(np.abs(g - rg) <= tol), (g - rg, tol)
    ctx.close()


def test_time_grows_with_the_samples():
    # a prediction copies 120 bytes per sample; pinning those on every call took six times as long
    import paper_2609_32308_amd as sd
    ctx = sd.Context(0)
    z = sd.Sizer(ctx, 8, 8, seed=5)
    best = {}
    for n in (100000, 600000):
        X = np.random.default_rng(n).random((n, 22)).astype(np.float32)
        z.predict(X)
        ts = []
        for _ in range(7):
            t0 = time.perf_counter()
            z.predict(X)
            ts.append(time.perf_counter() - t0)
        best[n] = min(ts)
        print("sizer", n, best[n], flush=True)
    ctx.close()
    assert best[600000] <= 3 * 6 * best[100000]
