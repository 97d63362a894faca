"""GPU (-m gpu): small fp32 weight gradients with the bias gradient and both updates in one launch: rows that are no whole vectors (whose
inputs are fetched one by one), remainders of k, tiles over both edges, programs of no, one and two inputs.  Against 64 bits, 1e-6 of
the sum of magnitudes: sums of at most 1000 terms over eight shares, each addition 6e-8, and three more operations."""
import numpy as np
import pytest

from test_gpu_parity import ctx, rng  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 15, 16, 17, 40, 128, 1000])
@pytest.mark.parametrize("m,n", [(5, 1), (31, 3), (64, 10), (33, 32), (100, 100), (260, 33), (7, 4)])
@pytest.mark.parametrize("form", ["plain", "update", "two inputs"])
def test_gradients_and_updates(ctx, m, n, k, form):  # noqa: F811
    g = rng(m * 1009 + n * 31 + k)
    x, dy, w, z = (g.standard_normal(s, dtype=np.float32) for s in ((k, m), (k, n), (m, n), (m, n)))
    b = g.standard_normal(n, dtype=np.float32)
    X, D, W, Bv, Z = ctx.tensor(x), ctx.tensor(dy), ctx.tensor(w, donatable=True), ctx.tensor(b, donatable=True), ctx.tensor(z)
    dw, db = ctx.matmul(X, D, trans_a=True), ctx.sum(D, axis=0)
    if form != "plain":
        new = ctx.sub(W, ctx.mul(dw, 0.5))
        ctx.assign(W, new if form == "update" else ctx.add(new, ctx.mul(Z, Bv)))
        ctx.assign(Bv, ctx.sub(Bv, ctx.mul(db, 0.5)))
        dw, db = W, Bv
    ctx.set_profiling(True)
    ctx.barrier()
    names = [r["kernel"] for r in ctx.last_launches()]
    ctx.set_profiling(False)
    if n > 1 and k >= 32:      # (one column is a row as well)
        assert "small" in names[0], names
    x, dy, w, b, z = (t.astype(np.float64) for t in (x, dy, w, b, z))
    ew, mw, eb, mb = x.T @ dy, np.abs(x.T) @ np.abs(dy), dy.sum(0), np.abs(dy).sum(0)
    if form != "plain":
        ew, mw = w - 0.5 * ew, np.abs(w) + 0.5 * mw
        if form == "two inputs":
            ew, mw = ew + z * b, mw + np.abs(z * b)
        eb, mb = b - 0.5 * eb, np.abs(b) + 0.5 * mb
    assert np.all(np.abs(ctx.fetch(dw) - ew) <= 1e-6 * mw)
    assert np.all(np.abs(ctx.fetch(db) - eb) <= 1e-6 * mb)
