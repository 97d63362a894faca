"""In-place updates of a tensor that the updating region itself reads: only where every reader of an
element is the one that overwrites it.  Plans on the null device against the oracle and the checker,
then (-m gpu) values against the oracle."""
import numpy as np
import pytest

from oracle.structural import Tracer
from paper_2102_13267_amd import Context
from plan_check import check_plan


def plans(build):
    """The plan of `build(B, mk)` on the null device (checked), which must be the structural oracle's."""
    ctx, T = Context(), Tracer()
    keep = build(ctx, lambda shape, donatable=False: ctx.tensor(np.zeros(shape, np.float32), donatable=donatable))
    info = ctx.barrier()
    plan = ctx.dump_plan()
    check_plan(ctx.dump_key(), info.n_nodes, plan)
    keep2 = build(T, lambda shape, donatable=False: T.tensor(shape, "f32", donatable=donatable))
    assert T.barrier()["plan"] == plan
    del keep, keep2
    return plan


@pytest.mark.parametrize("axis,shape", [(1, (64,)), (0, (64,)), (None, ())])
def test_a_broadcast_operand_is_not_overwritten(axis, shape):
    """x * b summed into b: with as many rows as columns b has the result's shape, and other workgroups
    still read all of it while one writes its part."""
    def build(B, mk):
        x, b = mk((64, 64)), mk(shape, True)
        B.assign(b, B.sum(B.mul(x, b), axis))
        return b
    assert "->p" not in plans(build)


def test_an_aligned_operand_is():
    def build(B, mk):
        x, b = mk((64, 64)), mk((64,), True)
        B.assign(b, B.sub(b, B.sum(x, axis=0)))
        return b
    assert "->p" in plans(build)


def values(build, data, tol=1e-5):
    """`build(B, *tensors)` three times over on the GPU and on the oracle (tensors whose entry is a pair are donatable)."""
    from oracle.numeric import Eager
    ctx, E = Context(device=0, workspace_bytes=256 << 20), Eager()
    mk = lambda B: [B.tensor(t[0].copy(), donatable=True) if isinstance(t, tuple) else B.tensor(t) for t in data]   # noqa: E731
    got, ref = mk(ctx), mk(E)
    for _ in range(3):
        for x, y in zip(build(ctx, *got), build(E, *ref)):
            a, b = np.asarray(ctx.fetch(x), np.float64), np.asarray(E.fetch(y), np.float64)
            assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b)
    ctx.close()


@pytest.mark.gpu
def test_broadcast_operand_values():
    """1e-5 of the norm: sums of 640 positive terms, rounded in another order."""
    g = np.random.Generator(np.random.PCG64(5))
    x, b = g.random((640, 640), dtype=np.float32), g.random(640, dtype=np.float32)

    def build(B, x, b):
        B.assign(b, B.mul(B.sum(B.mul(x, b), 1), 1 / 320))
        return [b]
    values(build, [x, (b,)])


def running_scale(B, x, s):
    """A running maximum kept in s, and x scaled by it."""
    r = B.add(B.mul(s, 0.9), B.mul(B.amax(B.abs(x)), 0.1))
    out = B.div(x, r)
    B.assign(s, r)
    return [out, s]


@pytest.mark.parametrize("n,in_place", [(1, True), (4, False), (1000, False), (2048, False), (2052, False), (65536, False), (65537, True)])
def test_a_running_scalar_that_a_finaliser_reads(n, in_place):
    """Up to 65,536 elements x / r is the finaliser of the maximum and computes r for each of its
    elements; beyond, and for a single one, r is computed once."""
    plan = plans(lambda B, mk: running_scale(B, mk((n,)), mk((), True)))
    assert ("->p" in plan) == in_place, plan


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 5, 1000, 1025, 2048, 2052, 65536, 65537])
def test_running_scalar_values(n):
    """1e-5 of the norm: a handful of fp32 roundings."""
    x = np.random.Generator(np.random.PCG64(n)).standard_normal(n).astype(np.float32)
    values(running_scale, [x, (np.float32(3.0).reshape(()),)])
