"""GPU (-m gpu): errors against 64 bits, where a path computes something in its own way."""
import numpy as np
import pytest

from test_gpu_parity import ctx, rng  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi,rms,most", [(1e-6, 1e-3, 0.253, 0.51), (1e-3, 0.1, 0.290, 0.56), (0.1, 0.3, 0.292, 0.59), (0.3, 0.625, 0.295, 0.78),
                                            (0.625, 0.8, 0.440, 1.41), (0.8, 1.0, 0.396, 1.13), (1.0, 1.5, 0.321, 1.0), (1.5, 2.0, 0.2945, 0.66), (2.0, 4.0, 0.290, 0.57),
                                            (4.0, 9.0, 0.290, 0.51)])
def test_tanh(ctx, lo, hi, rms, most):  # noqa: F811
    """Root mean square and largest error in last places: at most what the device library's tanhf shows on
    the same points (measured, rounded up in the third digit)."""
    x = np.linspace(lo, hi, 1 << 20).astype(np.float32)
    x[::2] *= -1
    y = ctx.fetch(ctx.tanh(ctx.tensor(x))).astype(np.float64)
    e = np.tanh(x.astype(np.float64))
    d = np.abs(y - e) / np.spacing(np.abs(e).astype(np.float32))
    assert np.sqrt(np.mean(d * d)) <= rms and d.max() <= most, (np.sqrt(np.mean(d * d)), d.max())


def test_tanh_of_special_values(ctx):  # noqa: F811
    x = np.array([0.0, -0.0, 1e-40, -1e-40, 9.5, -9.5, 44.0, -100.0, 3e38, -3e38, np.inf, -np.inf, np.nan], np.float32)
    y, e = ctx.fetch(ctx.tanh(ctx.tensor(x))), np.tanh(x.astype(np.float64)).astype(np.float32)
    assert np.array_equal(y, e, equal_nan=True) and np.array_equal(np.signbit(y[:-1]), np.signbit(e[:-1]))


def lanes_one_by_one(x, lanes):
    """Row sums as `lanes` lanes add them up: each its groups of four columns one by one, then all of them pairwise."""
    rows, cols = x.shape
    steps = -(-cols // (4 * lanes))
    t = np.zeros((rows, steps * 4 * lanes), np.float32)
    t[:, :cols] = x
    t = t.reshape(rows, steps, lanes, 4)
    acc = np.zeros((rows, lanes), np.float32)
    for s in range(steps):
        for e in range(4):
            acc = acc + t[:, s, :, e]
    while acc.shape[1] > 1:
        acc = acc[:, 0::2] + acc[:, 1::2]
    return acc[:, 0]


@pytest.mark.parametrize("rows,cols", [(4000, 100), (4000, 200), (3000, 513), (3001, 1777), (1500, 2000), (2100, 4097), (2100, 8192), (600, 8192), (1024, 1024)])
def test_row_sums(ctx, rows, cols):  # noqa: F811
    """Error of the sums of N(0, 1) terms: not above that of 256 lanes (64 below 512 columns) adding one by
    one, the arrangement that gives a lane the fewest terms, but for what the estimate over so many rows scatters
    (a relative 1 / sqrt(2 rows) each, 4 of them)."""
    x = rng(rows + cols).standard_normal((rows, cols), dtype=np.float32)
    e = x.astype(np.float64).sum(1)
    got = ctx.fetch(ctx.sum(ctx.mul(ctx.tensor(x), ctx.tensor(np.ones(cols, np.float32))), axis=1))
    ref = lanes_one_by_one(x, 256 if cols >= 512 else 64)
    err = lambda s: np.linalg.norm(s - e) / np.linalg.norm(e)                                   # noqa: E731
    assert err(got) <= err(ref) * (1 + 4 / np.sqrt(2 * rows)), (err(got), err(ref))
