"""GPU (-m gpu): column sums that ride with the contraction of the same tensor.  Against 64 bits: the sums' own error, fp32 partial
sums of up to a few hundred terms added pairwise, 1e-6 of the sum of magnitudes (each addition 6e-8), a bf16 result 4e-3 of its value."""
import numpy as np
import pytest

from oracle.numeric import round_to_bf16
from test_gpu_parity import ctx, rng  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu

# rows, columns of x and dy: (unsplit, split, halves) x (whole tiles, over the edges, k no multiple of a slice, one slice or less)
SHAPES = [(512, 2048, 2048), (1000, 1500, 2052), (4096, 1024, 1024), (8192, 300, 520), (2048, 1024, 1000), (2050, 700, 1300),
          (33, 1300, 1400), (31, 1100, 1500), (1, 1024, 1100), (96, 1030, 1028), (70, 1100, 999)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows,m,n", SHAPES)
@pytest.mark.parametrize("form", ["sum", "mean, first", "update"])
def test_sums_next_to_a_weight_gradient(ctx, dt, rows, m, n, form):  # noqa: F811
    g = rng(rows * 31 + m * 7 + n)
    x, dy = (g.standard_normal((rows, c), dtype=np.float32) for c in (m, n))
    b = g.standard_normal(n, dtype=np.float32)
    if dt == "bf16":
        x, dy, b = round_to_bf16(x), round_to_bf16(dy), round_to_bf16(b)
    X, D, P = ctx.tensor(x, dtype=dt), ctx.tensor(dy, dtype=dt), ctx.tensor(b, dtype=dt, donatable=True)
    db = ctx.mean(D, axis=0) if form == "mean, first" else None
    dw = ctx.matmul(X, D, trans_a=True)
    if db is None:
        db = ctx.sum(D, axis=0)
    if form == "update":
        ctx.assign(P, ctx.sub(P, ctx.mul(db, 0.01)))
        db = P
    ctx.set_profiling(True)
    ctx.barrier()
    names = [r["kernel"] for r in ctx.last_launches()]
    ctx.set_profiling(False)
    assert any("sums" in k for k in names) or any("small" in k for k in names) or any("col_reduce" in k for k in names), names
    if "lt_gemm_small" not in names[0] and (n % 4 == 0 or len(names) == 1):
        assert any("sums" in k for k in names) and not any("col_reduce" in k for k in names), names
    exact, mass = dy.astype(np.float64).sum(0), np.abs(dy.astype(np.float64)).sum(0)
    got = ctx.fetch(db).astype(np.float64)
    if form == "mean, first":
        exact, mass = exact / rows, mass / rows
    if form == "update":
        exact, mass = b - 0.01 * exact, np.abs(b) + 0.01 * mass
    bound = 1e-6 * mass + (4e-3 * np.abs(exact) if dt == "bf16" else 0.0)
    assert np.all(np.abs(got - exact) <= bound), np.max(np.abs(got - exact) / bound)
    ref = x.astype(np.float64).T @ dy.astype(np.float64)
    err = np.linalg.norm(ctx.fetch(dw).astype(np.float64) - ref) / np.linalg.norm(ref)
    assert err <= (4e-3 if dt == "bf16" else 2e-6), err


def test_infinities_and_nan_pass(ctx):  # noqa: F811
    dy = np.ones((512, 2048), np.float32)
    dy[7, 3], dy[100, 5], dy[101, 5], dy[200, 9] = np.inf, np.inf, -np.inf, np.nan
    for dt in ("f32", "bf16"):
        D = ctx.tensor(dy, dtype=dt)
        dw, db = ctx.matmul(ctx.tensor(np.ones((512, 2048), np.float32), dtype=dt), D, trans_a=True), ctx.sum(D, axis=0)
        ctx.barrier()
        got = ctx.fetch(db)
        assert got[3] == np.inf and np.isnan(got[5]) and np.isnan(got[9]) and got[0] == 512 and got[2047] == 512
