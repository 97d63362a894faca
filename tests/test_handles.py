"""What the binding says of handles: element type, shape and device address of results, released ones, closed contexts, foreign objects
(null device)."""
import types

import numpy as np
import pytest

from paper_2102_13267_amd import Context
from paper_2102_13267_amd.lt import LtError


def make():
    ctx = Context()
    t = ctx.add(ctx.tensor(np.zeros((3, 5), np.float32)), 1.0)
    ctx.barrier()
    return ctx, t


def test_results():
    ctx, t = make()
    assert t.dtype == "f32" and t.shape == (3, 5) and isinstance(ctx.device_ptr(t), int)
    s = ctx.sum(t)                       # not evaluated yet
    assert s.shape == ()
    with pytest.raises(LtError, match="not materialised"):
        ctx.device_ptr(s)


def test_anything_with_an_id_has_an_address():
    ctx, t = make()
    assert ctx.device_ptr(types.SimpleNamespace(tid=t.tid)) == ctx.device_ptr(t)
    for foreign in ("text", 7, None):
        with pytest.raises(AttributeError):
            ctx.device_ptr(foreign)


def test_assign_takes_tensors_only():
    ctx, t = make()
    foreign = types.SimpleNamespace(tid=t.tid, ctx=ctx, dtype="f32", shape=(3, 5))
    for dst, src in ((foreign, t), (t, foreign)):
        with pytest.raises((TypeError, AttributeError, LtError)):
            ctx.assign(dst, src)


def test_released_and_closed():
    ctx, t = make()
    u = ctx.mul(t, 2.0)
    ctx._check(ctx._lib.lt_release(ctx._h, u.tid))
    with pytest.raises(LtError, match="unknown or released"):
        u.shape
    with pytest.raises(LtError, match="unknown or released"):
        ctx.device_ptr(u)
    ctx.barrier()
    ctx.close()
    with pytest.raises(LtError):
        ctx.device_ptr(t)
