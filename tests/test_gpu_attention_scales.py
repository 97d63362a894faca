"""GPU parity (-m gpu) of attention over few keys (all of them in LDS at once), and of cores whose queries and query
gradients are scaled by the launches that load and store them.

Tolerances: bf16 2e-2 of the largest value (probabilities and their gradients rounded once each), fp32 1e-5 for the
context and 2e-5 for the gradients (two nested sums feed every element)."""
import numpy as np
import pytest

from oracle.numeric import Eager
from test_gpu_attention import kinds, operands
from test_gpu_parity import check, ctx  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu


def scaled_core(B, q, k, v, dy, b, sq, sk, h, d, scale, form):
    split = lambda t, s: B.permute(B.reshape(t, (b, s, h, d)), (0, 2, 1, 3))                  # noqa: E731
    merge = lambda t, s: B.reshape(B.permute(t, (0, 2, 1, 3)), (b * s, h * d))                # noqa: E731
    qs = B.mul(q, scale)
    qh, kh, vh, dh = split(qs, sq), split(k, sk), split(v, sk), split(dy, sq)
    p = B.softmax(B.matmul(qh, kh, trans_b=True))
    ds = B.softmax_grad(B.matmul(dh, vh, trans_b=True), p)
    dq = merge(B.matmul(ds, kh), sq)
    out = [merge(B.matmul(p, vh), sq), B.mul(dq, scale), merge(B.matmul(ds, qh, trans_a=True), sk), merge(B.matmul(p, dh, trans_a=True), sk)]
    if form == "read elsewhere":      # another reader of each
        out += [B.sum(qs, axis=1), B.sum(dq, axis=1)]
    elif form == "results":           # the host has both
        out += [qs, dq]
    elif form == "overwritten":       # the unscaled queries change in the same step
        B.assign(q, B.add(q, 1.0))
        out.append(q)
    return out


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("b,sq,sk,h,d", [(1, 1, 1, 1, 32), (2, 31, 33, 2, 64), (1, 130, 64, 2, 32), (2, 64, 65, 1, 64), (1, 127, 128, 2, 64), (1, 129, 129, 2, 32),
                                         (1, 200, 255, 2, 64), (1, 65, 256, 2, 32), (1, 97, 257, 1, 64), (1, 40, 70, 1, 128)])
def test_scaled_cores(ctx, dt, b, sq, sk, h, d):  # noqa: F811
    data, E = operands(sq * 1000 + sk + d, dt, b, sq, sk, h, d, growth=4.0), Eager()
    args = (b, sq, sk, h, d, 0.7, "")
    got = scaled_core(ctx, *(ctx.tensor(t, dtype=dt) for t in data), *args)
    names = kinds(ctx)
    assert len(names) == 3 and all(n.startswith("lt_attention") for n in names), names
    ref = scaled_core(E, *(E.tensor(t, dtype=dt) for t in data), *args)
    for i, (x, y) in enumerate(zip(got, ref)):
        check(ctx, E, x, y, 2e-2 if dt == "bf16" else 1e-5 if i == 0 else 2e-5, i)


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("form,extra", [("read elsewhere", 4), ("results", 2), ("overwritten", 2)])
def test_scalings_that_others_see(ctx, dt, form, extra):  # noqa: F811
    b, s, h, d = 2, 70, 2, 64
    data, E = operands(7, dt, b, s, s, h, d), Eager()
    for scale in (0.125, 1.7):     # (the second step finds the plan of the first)
        mk = lambda B, i, t: B.tensor(t, dtype=dt, donatable=form == "overwritten" and i == 0) if B is ctx else B.tensor(t, dtype=dt)   # noqa: E731
        got = scaled_core(ctx, *(mk(ctx, i, t) for i, t in enumerate(data)), b, s, s, h, d, scale, form)
        names = kinds(ctx)
        assert len(names) == 3 + extra, names
        ref = scaled_core(E, *(mk(E, i, t) for i, t in enumerate(data)), b, s, s, h, d, scale, form)
        for i, (x, y) in enumerate(zip(got, ref)):
            check(ctx, E, x, y, 2e-2 if dt == "bf16" else 2e-5, i)


@pytest.mark.parametrize("heads,sk,d,forward,dq", [(4, 64, 64, "walk", 1), (4, 65, 64, "walk", 2), (4, 128, 64, "walk", 2), (4, 129, 64, "short", 4), (4, 256, 32, "short", 4),
                                                   (4, 257, 64, "walk", 0), (4, 200, 128, "walk", 0), (384, 130, 64, "short", 4), (385, 130, 64, "walk", 4),
                                                   (768, 130, 64, "walk", 4), (769, 130, 64, "walk", 0), (2048, 130, 32, "walk", 4), (2049, 130, 32, "walk", 0),
                                                   (2049, 20, 32, "walk", 1)])
def test_kernels_on_both_sides_of_a_line(ctx, heads, sk, d, forward, dq):  # noqa: F811
    """All keys at once only where that was measured to be faster: by pass, keys and workgroups (three queries: one for each head)."""
    data, E = operands(heads + sk, "bf16", heads, 3, sk, 1, d), Eager()
    args = (heads, 3, sk, 1, d, 0.7, "")
    got = scaled_core(ctx, *(ctx.tensor(t, dtype="bf16") for t in data), *args)
    names = kinds(ctx)
    assert names[0] == (f"lt_attention_kernel_short<bf16, {d}, 4>" if forward == "short" else f"lt_attention_kernel<bf16, {d}>"), names
    assert names[1] == (f"lt_attention_dq_kernel_short<bf16, {d}, {dq}>" if dq else f"lt_attention_dq_kernel<bf16, {d}>"), names
    ref = scaled_core(E, *(E.tensor(t, dtype="bf16") for t in data), *args)
    for i, (x, y) in enumerate(zip(got, ref)):
        check(ctx, E, x, y, 2e-2, i)
