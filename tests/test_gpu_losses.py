"""GPU parity (-m gpu) of a cross-entropy and its gradient, which share a launch when they read the same logits and
labels, against the CPU oracle.  Tolerance 1e-5 of the largest value in fp32, 1e-2 in bf16 (one rounding of each)."""
import numpy as np
import pytest

from oracle.numeric import Eager, round_to_bf16
from test_gpu_parity import check, ctx, rng  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu


def step(B, z, w, labels, other, form):
    z = B.mul(z, 2.0)
    d, loss = None, None
    if form == "loss first":
        loss = B.mean(B.xent(z, labels))
        d = B.xent_grad(z, labels, 0.25)
    elif form == "gradient overwrites logits":
        loss, d = B.xent(w, labels), B.xent_grad(w, labels, 0.25)
        B.assign(w, d)
        d = w
    elif form == "gradient into a parameter":
        loss, d = B.xent(z, labels), B.xent_grad(z, labels, 0.25)
        B.assign(w, d)
        d = w
    elif form == "other labels":
        d, loss = B.xent_grad(z, labels, 0.25), B.xent(z, other)
    else:
        d, loss = B.xent_grad(z, labels, 0.25), B.xent(z, labels)
    return [d, loss, B.sum(d, axis=0)] + ([B.sum(loss)] if form == "gradient first" else [])


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows,cols", [(1, 2), (17, 10), (33, 256), (5, 257), (40, 1000), (3, 1025), (2, 4096), (512, 300), (513, 300)])
@pytest.mark.parametrize("form", ["gradient first", "loss first", "gradient overwrites logits", "gradient into a parameter", "other labels"])
def test_loss_with_its_gradient(ctx, dt, rows, cols, form):  # noqa: F811
    E, g = Eager(), rng(rows * 5000 + cols)
    z, w = (g.standard_normal((rows, cols), dtype=np.float32) * 3 for _ in range(2))
    if dt == "bf16":
        z, w = round_to_bf16(z), round_to_bf16(w)
    labels, other = (g.integers(0, cols, rows).astype(np.int32) for _ in range(2))
    for _ in range(2):     # (the second step finds the plan of the first)
        out = []
        for B in (ctx, E):
            mk = dict(donatable=True) if B is ctx else {}
            out.append(step(B, B.tensor(z, dtype=dt), B.tensor(w, dtype=dt, **mk), B.tensor(labels), B.tensor(other), form))
        ctx.set_profiling(True)
        ctx.barrier()
        names = [r["kernel"] for r in ctx.last_launches()]
        n, totals = sum("row_op" in k for k in names), sum("all_reduce" in k for k in names)
        ctx.set_profiling(False)
        # (one loss is its own sum; a launch of more than 128 workgroups leaves the sum to another)
        assert totals == (form in ("gradient first", "loss first") and (rows == 1 or rows == 513)), names
        # (the gradient does not overwrite the logits that it reads; into a parameter that nobody reads it comes first, and the losses join it)
        assert n == (2 if form == "other labels" else 1), names
        for i, (x, y) in enumerate(zip(*out)):
            check(ctx, E, x, y, 1e-2 if dt == "bf16" else 1e-5, i)
