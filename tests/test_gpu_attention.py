"""GPU parity (-m gpu) of the attention core that is lowered as a whole (forward, dq, dk and dv) against
the CPU oracle and against the same trace with its regions kept apart.

Tolerances: bf16 2e-2 of the largest value (probabilities and their gradients rounded once each), fp32
1e-5 for the context and 2e-5 for the gradients (two nested sums feed every element, as in a layer
norm's gradient)."""
import numpy as np
import pytest

from oracle.numeric import Eager, round_to_bf16
from test_gpu_parity import check, ctx, rng  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu


def core(B, q, k, v, dy, b, sq, sk, h, d, backward=True, keep_prob=False):
    split = lambda t, s: B.permute(B.reshape(t, (b, s, h, d)), (0, 2, 1, 3))                  # noqa: E731
    merge = lambda t, s: B.reshape(B.permute(t, (0, 2, 1, 3)), (b * s, h * d))                # noqa: E731
    qh, kh, vh, dh = split(q, sq), split(k, sk), split(v, sk), split(dy, sq)
    p = B.softmax(B.matmul(qh, kh, trans_b=True))
    out = [merge(B.matmul(p, vh), sq)]
    if backward:
        ds = B.softmax_grad(B.matmul(dh, vh, trans_b=True), p)
        out += [B.mul(merge(B.matmul(ds, kh), sq), 0.5), merge(B.matmul(ds, qh, trans_a=True), sk), merge(B.matmul(p, dh, trans_a=True), sk)]
    return out + ([p] if keep_prob else [])


def operands(seed, dt, b, sq, sk, h, d, growth=1.0):
    g, rnd = rng(seed), (round_to_bf16 if dt == "bf16" else (lambda x: x))
    q, dy = (g.standard_normal((b * sq, h * d), dtype=np.float32) for _ in range(2))
    k, v = (g.standard_normal((b * sk, h * d), dtype=np.float32) for _ in range(2))
    # scores of about N(0, growth^2) whose row maxima move to later keys
    q *= np.float32(d ** -0.5)
    k *= np.linspace(0.2, growth, sk, dtype=np.float32).repeat(1)[np.tile(np.arange(sk), b)][:, None]
    return [rnd(np.ascontiguousarray(t)) for t in (q, k, v, dy)]


def kinds(ctx):  # noqa: F811
    ctx.set_profiling(True)
    ctx.barrier()
    names = [r["kernel"] for r in ctx.last_launches()]
    ctx.set_profiling(False)
    return names


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("b,sq,sk,h,d", [(1, 1, 1, 1, 64), (2, 7, 7, 3, 32), (1, 32, 32, 2, 128), (2, 33, 33, 2, 64), (1, 64, 65, 2, 64), (2, 127, 130, 2, 32),
                                         (1, 200, 200, 3, 64), (3, 129, 63, 2, 128), (1, 513, 257, 2, 64), (1, 300, 301, 2, 128)])
def test_attention_core(ctx, dt, b, sq, sk, h, d):  # noqa: F811
    E = Eager()
    data = operands(sq * 1000 + sk + d, dt, b, sq, sk, h, d, growth=4.0)
    got = core(ctx, *(ctx.tensor(t, dtype=dt) for t in data), b, sq, sk, h, d)
    names = kinds(ctx)
    assert sum(n.startswith("lt_attention") for n in names) == 3 and not any("row_op" in n for n in names), names
    ref = core(E, *(E.tensor(t, dtype=dt) for t in data), b, sq, sk, h, d)
    for i, (x, y) in enumerate(zip(got, ref)):
        check(ctx, E, x, y, 2e-2 if dt == "bf16" else 1e-5 if i == 0 else 2e-5, i)


@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_attention_forward_only_in_place_and_kept_apart(ctx, dt):  # noqa: F811
    """Forward alone; probabilities that are a result of their own, another reader of the scores and a
    head width without a kernel keep the parts; a context that overwrites v's own buffer."""
    E, b, s, h = Eager(), 2, 70, 2
    for d, backward, keep in ((64, False, False), (64, False, True), (64, True, True), (96, True, False), (16, False, False)):
        data = operands(d + backward * 2 + keep, dt, b, s, s, h, d)
        got = core(ctx, *(ctx.tensor(t, dtype=dt) for t in data), b, s, s, h, d, backward, keep)
        names = kinds(ctx)
        assert any(n.startswith("lt_attention") for n in names) == (d == 64 and not keep), (d, names)
        ref = core(E, *(E.tensor(t, dtype=dt) for t in data), b, s, s, h, d, backward, keep)
        for i, (x, y) in enumerate(zip(got, ref)):
            check(ctx, E, x, y, 2e-2 if dt == "bf16" else 2e-5, i)
    data = operands(5, dt, 1, s, s, 1, 64)

    def update(B, mk):
        q, k, v = (mk(t) for t in data[:3])
        B.assign(v, B.matmul(B.softmax(B.matmul(q, k, trans_b=True)), v))
        return v
    got, ref = update(ctx, lambda t: ctx.tensor(t, dtype=dt, donatable=True)), update(E, lambda t: E.tensor(t, dtype=dt))
    check(ctx, E, got, ref, 2e-2 if dt == "bf16" else 1e-5)


def test_attention_core_same_as_its_parts(ctx):  # noqa: F811
    """One region per op against the whole core, fp32: 2e-5 of the largest value."""
    from paper_2102_13267_amd import Context
    b, sq, sk, h, d = 2, 150, 90, 3, 64
    data = operands(99, "f32", b, sq, sk, h, d, growth=3.0)
    other = Context(device=0, workspace_bytes=256 << 20)
    other.set_fusion(False)
    res = []
    for c in (ctx, other):
        out = core(c, *(c.tensor(t) for t in data), b, sq, sk, h, d)
        c.barrier()
        res.append([c.fetch(t).copy() for t in out])
    other.close()
    for x, y in zip(*res):
        assert np.max(np.abs(x - y)) <= 2e-5 * np.max(np.abs(y))


def test_results_that_are_other_shapes_of_a_computed_value(ctx):  # noqa: F811
    """A reshaped result takes the memory of the value it reshapes when it can: a value with other
    readers, two reshapes of one value, a value that is a result too, a permuted one; and updating one
    of them in place afterwards changes none of the others."""
    E, g = Eager(), rng(77)
    a, b = (g.standard_normal((24, 24), dtype=np.float32) for _ in range(2))

    def prog(B, a, b):
        y = B.matmul(a, b)
        e = B.mul(a, 2.0)
        p = B.matmul(B.reshape(a, (2, 12, 24)), B.reshape(b, (2, 12, 24)), trans_b=True)
        r = [B.reshape(y, (12, 48)), B.reshape(y, (576,)), B.sum(B.relu(y), axis=1), e, B.reshape(e, (4, 144)), B.reshape(B.permute(p, (1, 0, 2)), (12, 24)),
             B.reshape(B.softmax(b), (8, 72))]
        if B is ctx:
            ctx.barrier()
        B.assign(r[0], B.mul(r[0], -1.0))
        B.assign(r[4], B.add(r[4], 1.0))
        return r
    got, ref = prog(ctx, ctx.tensor(a), ctx.tensor(b)), prog(E, E.tensor(a), E.tensor(b))
    for i, (x, y) in enumerate(zip(got, ref)):
        check(ctx, E, x, y, 1e-5, i)


def test_no_keys(ctx):  # noqa: F811
    """A context over no keys at all is zero, as the parts give it."""
    z = lambda n: ctx.tensor(np.ones((n, 64), np.float32))                                   # noqa: E731
    assert not np.any(ctx.fetch(ctx.matmul(ctx.softmax(ctx.matmul(z(70), z(0), trans_b=True)), z(0))))


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("s,d", [(64, 64), (70, 64), (33, 32), (129, 128)])
def test_a_key_that_no_query_attends_to(ctx, s, d, dt):  # noqa: F811
    """A key with minus infinity in a column where every query is positive has probability 0 and gets
    gradients of 0, whether or not the last block of queries is whole; its neighbours are unaffected.  (dq is 0 * inf.)"""
    E = Eager()
    q, k, v, dy = operands(s + d, dt, 1, s, s, 1, d)
    q[:, 3] = np.abs(q[:, 3]) + 0.5
    q = round_to_bf16(q) if dt == "bf16" else q
    k[5, 3] = -np.inf
    out = []
    for B in (ctx, E):
        qt, kt, vt, dt_ = (B.tensor(t, dtype=dt) for t in (q, k, v, dy))
        p = B.softmax(B.matmul(qt, kt, trans_b=True))
        ds = B.softmax_grad(B.matmul(dt_, vt, trans_b=True), p)
        out.append([B.matmul(p, vt), B.matmul(ds, kt), B.matmul(ds, qt, trans_a=True), B.matmul(p, dt_, trans_a=True)])
    assert sum(n.startswith("lt_attention") for n in kinds(ctx)) == 3
    for i in (0, 2, 3):
        x, y = ctx.fetch(out[0][i]), E.fetch(out[1][i])
        assert np.all(np.isfinite(x)), i
        assert np.max(np.abs(x - y)) <= (2e-2 if dt == "bf16" else 2e-5) * np.max(np.abs(y)), i
    assert not np.any(ctx.fetch(out[0][2])[5]) and not np.any(ctx.fetch(out[0][3])[5])


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("s", [1, 3, 200, 1025])
def test_values_near_the_largest(ctx, s, dt):  # noqa: F811
    """An average of values near the type's largest is finite."""
    E, d = Eager(), 64
    q, k, _, _ = operands(s, dt, 1, s, s, 1, d)
    v = np.full((s, d), 2.0 ** 127, np.float32)
    out = []
    for B in (ctx, E):
        qt, kt, vt = (B.tensor(t, dtype=dt) for t in (q, k, v))
        out.append(B.matmul(B.softmax(B.matmul(qt, kt, trans_b=True)), vt))
    assert kinds(ctx)[0].startswith("lt_attention_kernel")
    check(ctx, E, *out, 2e-2 if dt == "bf16" else 1e-5)
