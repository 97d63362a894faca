"""Whether a context that was never told how many streams to use spreads a plan (host logic, null device): layer steps on both
sides of the estimate, and what lt_set_streams makes of either."""
import re

import numpy as np
import pytest

from paper_2102_13267_amd import Context
from workloads import programs


def layer_step(ctx, batch, seq, d):
    vector = ("bq", "bk", "bv", "bo", "b2", "g1", "be1", "g2", "be2")
    shapes = {"Wq": (d, d), "Wk": (d, d), "Wv": (d, d), "Wo": (d, d), "W1": (d, 4 * d), "W2": (4 * d, d), "b1": (4 * d,), **{k: (d,) for k in vector}}
    new = lambda shape, dt: ctx.tensor(np.zeros(shape, np.float32), dtype=dt, donatable=True)   # noqa: E731
    P, M, V = ({k: new(s, dt) for k, s in shapes.items()} for dt in ("bf16", "f32", "f32"))
    out = programs.c3_step(ctx, new((batch, seq, d), "bf16"), new((batch, seq, d), "bf16"), P, M, V, d // 64)
    ctx.barrier()
    return out


@pytest.mark.parametrize("size,pays", [((4, 128, 512), False), ((32, 256, 256), False), ((32, 256, 512), False), ((4, 256, 1024), False),
                                       ((1, 64, 1024), False), ((1, 100, 1024), True), ((2, 128, 1024), True), ((16, 256, 1024), True), ((32, 256, 1024), True)])
def test_layer_steps(size, pays):
    ctx = Context()
    assert ctx.plan_streams() == 0
    keep = layer_step(ctx, *size)
    sched = ctx.dump_schedule()
    streams = 1 + max(int(s) for s in re.findall(r" stream=(\d) ", sched))
    assert streams > 1 and len(sched.splitlines()) >= 24          # (there is something to decide)
    assert ctx.plan_streams() == (streams if pays else 1)
    ctx.set_streams(4)
    assert ctx.plan_streams() == streams                          # asked for: the estimate has no say
    ctx.set_streams(1)
    assert ctx.plan_streams() == 1
    del keep


def test_short_plans_do_not_spread():
    ctx = Context()
    ctx.set_streams(4)
    x = ctx.tensor(np.zeros((4096, 1024), np.float32))
    keep = [ctx.sum(ctx.mul(x, float(i + 2)), axis=0) for i in range(4)]
    ctx.barrier()
    assert ctx.plan_streams() == 1
    del keep


def products_and_sums(ctx, rows, cols):
    """fp32 products next to column sums, three times over."""
    new = lambda *shape: ctx.tensor(np.zeros(shape, np.float32))   # noqa: E731
    x, w, w2, out = new(rows, cols), new(cols, cols // 2), new(cols, cols), []
    for i in range(3):
        xi = ctx.mul(x, 1.0 + 0.5 * i)
        s = ctx.sum(ctx.square(xi), axis=0)
        out += [ctx.matmul(xi, w), s, ctx.add(ctx.matmul(xi, w2), s)] + [ctx.sum(ctx.mul(xi, float(k + 2)), axis=0) for k in range(5)]
    ctx.barrier()
    return out


@pytest.mark.parametrize("rows,cols,pays", [(1024, 512, False), (3000, 1024, True), (4096, 1024, True), (8192, 1024, True)])
def test_fp32_products_and_column_sums(rows, cols, pays):
    ctx = Context()
    keep = products_and_sums(ctx, rows, cols)
    assert len(ctx.dump_schedule().splitlines()) >= 24
    assert (ctx.plan_streams() > 1) == pays
    del keep


@pytest.mark.parametrize("products,spread", [(11, False), (12, True)])
def test_riding_sums_count_as_launches(products, spread):
    ctx = Context()
    ctx.set_streams(4)
    x, keep = ctx.tensor(np.zeros((1024, 1024), np.float32)), []
    for _ in range(products):
        dy = ctx.tensor(np.zeros((1024, 2048), np.float32))
        keep += [ctx.matmul(x, dy, trans_a=True), ctx.sum(dy, axis=0)]
    ctx.barrier()
    assert len(ctx.dump_schedule().splitlines()) == products
    assert (ctx.plan_streams() > 1) == spread
    del keep
