"""Sizer gradients whose sample sums are split: every entry against the FP64 reference at the edges of
the sample chunks, for a wide and a narrow network, and repeated calls of growing and shrinking
sizes on one sizer (its workspace is kept between calls)."""
import numpy as np
import pytest

from oracle import mlp_ref as R
from tests.test_sizer import _inputs_clear_of_kinks, _magnitudes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,K", [(64, 8), (5, 3), (200, 1)])
def test_gradient_at_chunk_edges(H, K):
    import paper_2609_32308_amd as sd
    ctx = sd.Context(0)
    z = sd.Sizer(ctx, H, K, seed=3)
    flat = z.get_params()
    for n in (32, 33, 64, 65, 257 if H <= 64 else 66, 31):
        print("sizer", H, K, "samples", n, flush=True)
        X, Y = _inputs_clear_of_kinks(n, K, flat, H, 5 + n)
        loss, g = z.gradient(X, Y)
        rl, rg, ry = R.loss_and_grad(flat, X, Y, H, K)
        mag, mag_y, _ = _magnitudes(flat, X, Y, H, K)
        assert abs(loss - rl) <= 1e-5 * max(1e-3, abs(rl))
        # FP32 rounding of each term and sum, per entry (as in the unsplit test)
        tol = 4 * (max(n, H, 22) + 4) * 2.0 ** -24 * mag + 1e-4 * np.abs(rg) + 1e-12
        bad = np.flatnonzero(np.abs(g - rg) > tol)
        assert bad.size == 0, (n, bad[:10], g[bad[:10]], rg[bad[:10]])
        assert np.array_equal(g, z.gradient(X, Y)[1])  # the sums run in a fixed order
        assert np.all(np.abs(z.predict(X) - ry) <= 4 * (H + 26) * 2.0 ** -24 * mag_y + 2e-7)
    ctx.close()
