"""GPU (-m gpu): column sums that ride with a weight gradient are no further from 64 bits than in a launch of their own, over long columns,
rows aligned and not, unsplit, split and in halves.  Root mean square over the columns, of which a thousand fix it to a few per
cent: hence 1.1."""
import numpy as np
import pytest

from test_gpu_parity import ctx  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


def error(ctx, rows, m, n, mean, dt, ride):  # noqa: F811
    """Distance of the sums from 64 bits; the contraction's kernel."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(rows + n)
    dy = torch.randn(rows, n, device="cuda", generator=gen).add_(mean).to(torch.float32 if dt == "f32" else torch.bfloat16)
    x = torch.zeros(rows, m, device="cuda", dtype=dy.dtype)
    exact = torch.zeros(n, dtype=torch.float64, device="cuda")
    for part in dy.split(8192):
        exact += part.double().sum(0)
    D, zero = ctx.tensor(dy, dtype=dt), ctx.tensor(torch.zeros(n, device="cuda"))
    dw = ctx.matmul(ctx.tensor(x, dtype=dt), D, trans_a=True) if ride else None
    db = ctx.sum(D, axis=0)
    if dt == "bf16":                 # (the sum itself is of 32 bits; what is stored would be rounded to 16)
        db = ctx.add(ctx.cast(db, "f32"), zero)
    ctx.set_profiling(True)
    ctx.barrier()
    names = [r["kernel"] for r in ctx.last_launches()]
    ctx.set_profiling(False)
    assert any("sums" in k for k in names) == ride, names
    got = ctx.fetch(db).astype(np.float64)
    del dw
    exact = exact.cpu().numpy()
    return np.linalg.norm(got - exact) / np.linalg.norm(exact), names[0]


def closer(ctx, rows, m, n, mean, dt):  # noqa: F811
    (own, _), (riding, name) = error(ctx, rows, m, n, mean, dt, False), error(ctx, rows, m, n, mean, dt, True)
    assert riding <= 1.1 * own, (riding, own)
    return name


@pytest.mark.parametrize("rows,m,n,aligned", [(4096, 1030, 1030, False), (8192, 1030, 1030, False), (8209, 1030, 1030, False), (8192, 1030, 2052, False),
                                              (4096, 1030, 4100, False), (65536, 1030, 1030, False), (8192, 1024, 1024, True), (65536, 1024, 1024, True),
                                              (65536, 2048, 4096, True)])
@pytest.mark.parametrize("mean", [0.0, 1.0])
def test_long_columns_in_fp32(ctx, rows, m, n, aligned, mean):  # noqa: F811
    assert closer(ctx, rows, m, n, mean, "f32").split(",")[4].startswith("true" if aligned else "false")


@pytest.mark.parametrize("rows,m,n,kernel", [(65536, 2048, 2048, "true,2>"), (32768, 2048, 4096, "true,1>"), (65536, 2050, 4098, "false,1>"), (8192, 1030, 1032, "false,2>"),
                                             (16384, 1024, 1024, "true,2>"), (70, 1030, 2052, "false,1>")])
@pytest.mark.parametrize("mean", [0.0, 1.0])
def test_long_columns_in_bf16(ctx, rows, m, n, kernel, mean):  # noqa: F811
    assert closer(ctx, rows, m, n, mean, "bf16").endswith(kernel)


@pytest.mark.parametrize("dt,unit", [("f32", 2.0 ** -149), ("bf16", 2.0 ** -133)])
@pytest.mark.parametrize("n", [2048, 2052])
def test_subnormal_columns(ctx, dt, unit, n):  # noqa: F811
    """Sums that stay subnormal and sums that become normal: both exact."""
    dy = np.zeros((512, n), np.float32)
    dy[:, 3] = 3 * unit
    dy[[7, 300], 5] = unit, 2 * unit
    dy[::2, 9], dy[1::2, 9] = 5 * unit, -4 * unit
    x, D = ctx.tensor(np.zeros((512, 2048), np.float32), dtype=dt), ctx.tensor(dy, dtype=dt)
    dw, db = ctx.matmul(x, D, trans_a=True), ctx.sum(D, axis=0)
    ctx.set_profiling(True)
    ctx.barrier()
    names = [r["kernel"] for r in ctx.last_launches()]
    ctx.set_profiling(False)
    assert "sums" in names[0], names
    got = ctx.fetch(db).astype(np.float64)
    assert got[3] == 1536 * unit and got[5] == 3 * unit and got[9] == 256 * unit and got[0] == 0


def small_sums(dy):
    """The order of a small product's riding sums: eight shares of k, each half of a wave every other four rows of its share; four groups
    of those at a time, then one after the other; the shares in order, the lower half before the upper."""
    rows, n = dy.shape
    per = -(-(-(-rows // 8)) // 8)
    padded = np.zeros((8 * per * 8, n), np.float32)
    padded[:rows] = dy
    v = padded.reshape(8, per, 2, 4, n)
    group = (v[:, :, :, 0] + v[:, :, :, 1]) + (v[:, :, :, 2] + v[:, :, :, 3])
    share = np.zeros((8, 2, n), np.float32)
    for first in range(0, per, 4):
        four = np.zeros((8, 2, n), np.float32)
        for g in range(first, min(first + 4, per)):
            four = four + group[:, g]
        share = share + four
    total = np.zeros(n, np.float32)
    for w in range(8):
        total = total + share[w, 0] + share[w, 1]
    return total


@pytest.mark.parametrize("rows,m,n", [(1000, 100, 100), (1024, 300, 333), (700, 250, 40), (40, 64, 10), (129, 512, 784)])
def test_small_products_add_up_in_fours(ctx, rows, m, n):  # noqa: F811
    """Bit for bit: with running sums joined group by group, or two by two, a thousand rows are an eighth further from 64 bits."""
    dy = np.random.default_rng(rows).standard_normal((rows, n), dtype=np.float32)
    D = ctx.tensor(dy)
    dw, db = ctx.matmul(ctx.tensor(np.ones((rows, m), np.float32)), D, trans_a=True), ctx.sum(D, axis=0)
    ctx.set_profiling(True)
    ctx.barrier()
    names = [r["kernel"] for r in ctx.last_launches()]
    ctx.set_profiling(False)
    assert len(names) == 1 and "small" in names[0], names
    assert np.array_equal(ctx.fetch(db), small_sums(dy))


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows,m,n", [(8192, 1030, 1032), (8192, 1024, 2048), (5001, 1030, 4100)])
def test_infinite_totals_stay(ctx, dt, rows, m, n):  # noqa: F811
    """What a total keeps of its additions' losses is nothing once it is infinite; largest values next to each other do not overflow it."""
    dy = np.ones((rows, n), np.float32)
    dy[70, 3], dy[rows - 2, 4], dy[100, 5], dy[rows - 1, 5], dy[9, 6] = np.inf, -np.inf, np.inf, -np.inf, np.nan
    big = np.float32(2.0 ** 127)
    dy[:, 7] = 0.0
    dy[5, 7], dy[6, 7], dy[4000, 7] = big, -big, big
    x, D = ctx.tensor(np.zeros((rows, m), np.float32), dtype=dt), ctx.tensor(dy, dtype=dt)
    dw, db = ctx.matmul(x, D, trans_a=True), ctx.sum(D, axis=0)
    ctx.set_profiling(True)
    ctx.barrier()
    names = [r["kernel"] for r in ctx.last_launches()]
    ctx.set_profiling(False)
    assert "sums" in names[0], names
    got = ctx.fetch(db).astype(np.float64)
    assert got[3] == np.inf and got[4] == -np.inf and np.isnan(got[5]) and np.isnan(got[6]) and got[7] == float(big)
    assert abs(got[0] - rows) <= (0 if dt == "f32" else 2 ** -8 * rows)
