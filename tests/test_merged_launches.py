"""Launches that take another region's work along, and the programs where they must not (host logic, null device):
which launches a plan has and what they read and write."""
import numpy as np
import pytest

from paper_2102_13267_amd import Context
from test_launches import check_launches
from test_schedule import hazards_are_ordered, invariants, parse


def schedule(build):
    ctx = Context()

    def mk(shape, dtype="f32", donatable=False):
        return ctx.tensor(np.zeros(shape, np.int32 if dtype == "s32" else np.float32), dtype=dtype, donatable=donatable)
    keep = build(ctx, mk)
    info = ctx.barrier()
    sched = parse(ctx.dump_schedule())
    invariants(sched)
    hazards_are_ordered(sched)
    check_launches(ctx.dump_key(), info.n_nodes, ctx.dump_plan(), sched)
    del keep
    return sched


def kinds(sched):
    return [l["kind"] for l in sched]


# ---- a norm's column reductions behind its input gradient ----------------------------------------------
def norm_gradient(reduce, dt="f32", rows=64, cols=256, between=None):
    """The input gradient, then `reduce` of dy * xhat over the rows."""
    def build(B, mk):
        x, dy = mk((rows, cols), dt, True), mk((rows, cols), dt, True)
        y, mu, rs = B.layer_norm(x, mk((cols,), dt), mk((cols,), dt), eps=1e-5)
        dx = B.layer_norm_grad(dy, x, mk((cols,), dt), mu, rs)
        out = [between(B, x, dy)] if between else []
        xhat = B.mul(B.sub(x, B.reshape(mu, (rows, 1))), B.reshape(rs, (rows, 1)))
        return [y, dx, getattr(B, reduce)(B.mul(dy, xhat), axis=0), x, dy] + out
    return build


def column_operands(sched):
    """How many tensors the column launch reads."""
    (col,) = [l for l in sched if l["kind"] == "COL"]
    return len(col["reads"])


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("reduce,operands", [("sum", 1), ("mean", 1), ("amax", 4)])
def test_sums_and_means_ride_with_a_norms_gradient(dt, reduce, operands):
    """(one operand: the partial sums that the gradient's launch has left)"""
    assert column_operands(schedule(norm_gradient(reduce, dt))) == operands
