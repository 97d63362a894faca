"""The attention core as the lowering sees it (host logic, null device)."""
import numpy as np

from paper_2102_13267_amd import Context
from test_schedule import hazards_are_ordered, invariants, parse


def launches(dt, sq, sk, h=2, d=64, backward=True):
    """Kinds of the launches of the core, forward or forward and backward."""
    ctx = Context()

    def record():
        head = lambda s: ctx.permute(ctx.reshape(ctx.tensor(np.zeros((s, h * d), np.float32), dtype=dt), (1, s, h, d)), (0, 2, 1, 3))   # noqa: E731
        q, k, v, dy = head(sq), head(sk), head(sk), head(sq)
        p = ctx.softmax(ctx.matmul(q, k, trans_b=True))
        out = [ctx.matmul(p, v)]
        if backward:
            ds = ctx.softmax_grad(ctx.matmul(dy, v, trans_b=True), p)
            out += [ctx.matmul(ds, k), ctx.matmul(ds, q, trans_a=True), ctx.matmul(p, dy, trans_a=True)]
        return out
    out = record()
    ctx.barrier()
    sched = parse(ctx.dump_schedule())
    invariants(sched)
    hazards_are_ordered(sched)
    del out
    return [l["kind"] for l in sched]


def test_schedule_names_the_launches_of_the_core():
    assert launches("bf16", 128, 128) == ["ATTN"] * 3
    assert launches("f32", 70, 33, backward=False) == ["ATTN"]


def test_empty_sides_keep_the_parts():
    """No keys (a context of zeros), no queries: the parts' launches take them."""
    for sq, sk in ((128, 0), (0, 128)):
        assert "ATTN" not in launches("f32", sq, sk) and "ATTN" not in launches("bf16", sq, sk, backward=False)
