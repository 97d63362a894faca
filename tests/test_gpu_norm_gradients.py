"""GPU parity (-m gpu) of a layer norm's weight and bias gradients, which share a launch when they can,
against the CPU oracle.  Bar: 2e-5 (fp32; sums of N(0,1) terms, scaled by the square root of their
number as they cancel) or 2e-2 (bf16) of the largest value."""
import numpy as np
import pytest

from oracle.numeric import Eager, round_to_bf16
from test_gpu_parity import check, ctx, rng  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu


def operands(rows, cols, dt):
    g, rnd = rng(rows * 31 + cols), (round_to_bf16 if dt == "bf16" else (lambda t: t))
    x, dy = (rnd(g.standard_normal((rows, cols), dtype=np.float32)) for _ in range(2))
    w, b = (rnd(g.standard_normal(cols, dtype=np.float32)) for _ in range(2))
    return x, dy, w, b


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows,cols", [(1, 4), (7, 256), (64, 260), (65, 500), (129, 1024), (1000, 1028), (4099, 1024), (8192, 512), (300, 4096), (40, 30)])
def test_weight_and_bias_gradient(ctx, rows, cols, dt):  # noqa: F811
    """One slab and many, a rest of rows, a rest of a strip, columns that are no multiple of four (launches
    of their own); results, and an update of the parameters in place, twice."""
    E, data = Eager(), operands(rows, cols, dt)
    tol = 2e-2 if dt == "bf16" else 2e-5 * max(1.0, rows ** 0.5 / 8)

    def run(B, mk):
        x, dy, w, b = (mk(t) for t in data)
        out = []
        for _ in range(2):
            y, mu, rs = B.layer_norm(x, w, b, eps=1e-5)
            dg = B.sum(B.mul(dy, B.mul(B.sub(x, B.reshape(mu, (rows, 1))), B.reshape(rs, (rows, 1)))), axis=0)
            db = B.sum(dy, axis=0)
            out += [dg, db]
            low = (lambda t: B.cast(t, "bf16")) if dt == "bf16" else (lambda t: t)
            B.assign(w, low(B.sub(w, B.mul(dg, 1e-3))))
            B.assign(b, low(B.sub(b, B.mul(db, 1e-3))))
            if B is ctx:
                info = ctx.barrier()
                # (a single row's mean is a scalar, not one value per row: the general form)
                assert rows == 1 or cols % 4 or info.n_launches == info.n_regions - 1
        return out + [w, b]
    got, ref = run(ctx, lambda t: ctx.tensor(t, dtype=dt, donatable=True)), run(E, lambda t: E.tensor(t, dtype=dt))
    for i, (p, q) in enumerate(zip(got, ref)):
        check(ctx, E, p, q, tol, i)


def test_bias_gradient_keeps_its_own_launch_when_it_must(ctx):  # noqa: F811
    """Its program reads the weight gradient, or overwrites what a launch in between reads; another
    tensor's sum; a mean; other forms of the weight gradient."""
    E, rows, cols = Eager(), 256, 128
    x, dy, w, b = operands(rows, cols, "f32")

    def prog(B, variant):
        mk = lambda t: B.tensor(t.copy(), donatable=True)                                     # noqa: E731
        tx, tdy, tw, tb = mk(x), mk(dy), mk(w), mk(b)
        _, mu, rs = B.layer_norm(tx, tw, tb, eps=1e-5)
        mu, rs = B.reshape(mu, (rows, 1)), B.reshape(rs, (rows, 1))
        dg = B.sum(B.mul(B.mul(rs, B.sub(tx, mu)), tdy) if variant != 5 else B.mul(B.mul(B.sub(mu, tx), rs), tdy), axis=0)
        if variant == 0:
            return dg, B.add(B.sum(tdy, axis=0), dg)
        if variant == 1:
            z = B.matmul(B.reshape(tb, (1, cols)), B.tensor(x[:cols, :16].copy()))
            db = B.sum(tdy, axis=0)
            B.assign(tb, B.sub(tb, db))
            return dg, z, tb
        if variant == 2:
            return dg, B.sum(tx, axis=0)
        if variant == 3:
            return dg, B.mean(tdy, axis=0)
        if variant == 4:
            return dg, B.sum(tdy, axis=0), B.sum(B.mul(tdy, tdy), axis=0), B.mul(B.sum(tdy, axis=0), 2.0)
        return dg, B.sum(tdy, axis=0)
    for variant in range(6):
        for i, (p, q) in enumerate(zip(prog(ctx, variant), prog(E, variant))):
            check(ctx, E, p, q, 4e-5, (variant, i))


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows,cols", [(1, 8), (3, 256), (5, 504), (4097, 512), (130, 520), (4100, 1024), (33, 1032), (70, 2048), (9, 2056), (6, 4096), (5, 1028)])
def test_norm_forward_and_backward(ctx, rows, cols, dt):  # noqa: F811
    """One to eight chunks per lane, a last chunk that few lanes have, more rows than waves (a wave walks
    several), columns that are no whole chunks; a row of large equal values next to a row of minus ones."""
    E, data = Eager(), operands(rows, cols, dt)
    data[0][-1] = 1000.0 + np.arange(cols) % 2 * 8                       # (a large mean: 8 is representable next to it in bf16)

    def prog(B):
        x, dy, w, b = (B.tensor(t, dtype=dt) for t in data)
        y, mu, rs = B.layer_norm(x, w, b, eps=1e-5)
        return y, mu, rs, B.layer_norm_grad(dy, x, w, mu, rs)
    for i, (p, q) in enumerate(zip(prog(ctx), prog(E))):
        check(ctx, E, p, q, 2e-2 if dt == "bf16" else 2e-5, i)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows,cols", [(2, 8), (31, 256), (33, 504), (257, 512), (8193, 520), (16500, 1024), (300, 1032), (2100, 2048), (70, 2056), (5, 1028), (64, 1030)])
def test_sums_that_ride_with_the_input_gradient(ctx, rows, cols, dt):  # noqa: F811
    """One to more than 512 workgroups' partial sums, a wave with a row more than another, the last chunk that few lanes
    have, rows too long for it or of no whole chunks (launches of their own); both sums, one alone, parameters updated in
    place by them, and x overwritten between the input gradient and the sums (which then take the new x, in a launch of their own)."""
    chunk = 8 if dt == "bf16" else 4
    rides = cols % chunk == 0 and cols <= 4 * 64 * chunk
    E, data = Eager(), operands(rows, cols, dt)
    tol = 2e-2 if dt == "bf16" else 2e-5 * max(1.0, rows ** 0.5 / 8)

    def run(B, mk, variant):
        x, dy, w, b = (mk(t) for t in data)
        y, mu, rs = B.layer_norm(x, w, b, eps=1e-5)
        dx = B.layer_norm_grad(dy, x, w, mu, rs)
        if variant == 3:
            B.assign(x, B.mul(x, 0.5))
        dg = B.sum(B.mul(dy, B.mul(B.sub(x, B.reshape(mu, (rows, 1))), B.reshape(rs, (rows, 1)))), axis=0)
        if variant == 1:
            return [dx, dg]
        db = B.sum(dy, axis=0)
        if variant == 2:
            low = (lambda t: B.cast(t, "bf16")) if dt == "bf16" else (lambda t: t)
            B.assign(w, low(B.sub(w, B.mul(dg, 1e-3))))
            B.assign(b, low(B.sub(b, B.mul(db, 1e-3))))
            return [dx, w, b]
        return [y, dx, dg, db, x]
    for variant in range(4):
        got = run(ctx, lambda t: ctx.tensor(t, dtype=dt, donatable=True), variant)
        ctx.set_profiling(True)
        ctx.barrier()
        names = [r["kernel"] for r in ctx.last_launches()]
        ctx.set_profiling(False)
        (sums,) = [int(n[:-1].split(", ")[-1]) for n in names if n.startswith("lt_norm_stream_kernel<3,")] or [0]
        assert sums == ((2, 1, 1, 0)[variant] if rides else 0), names    # (updated in place the bias's sum stands first, in a launch of its own)
        ref = run(E, lambda t: E.tensor(t, dtype=dt), variant)
        for i, (p, q) in enumerate(zip(got, ref)):
            check(ctx, E, p, q, tol, (variant, i))


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("reduce", ["mean", "amax"])
@pytest.mark.parametrize("rows,cols", [(2, 8), (64, 256), (257, 512), (8193, 520)])
def test_other_reductions_of_the_same_program(ctx, rows, cols, reduce, dt):  # noqa: F811
    """A column's mean and its largest value of dy * xhat next to the input gradient."""
    E, data = Eager(), operands(rows, cols, dt)

    def prog(B):
        x, dy, w, b = (B.tensor(t, dtype=dt) for t in data)
        y, mu, rs = B.layer_norm(x, w, b, eps=1e-5)
        xhat = B.mul(B.sub(x, B.reshape(mu, (rows, 1))), B.reshape(rs, (rows, 1)))
        return B.layer_norm_grad(dy, x, w, mu, rs), getattr(B, reduce)(B.mul(dy, xhat), axis=0), B.sum(dy, axis=0)
    for i, (p, q) in enumerate(zip(prog(ctx), prog(E))):
        check(ctx, E, p, q, 2e-2 if dt == "bf16" else 2e-5 * max(1.0, rows ** 0.5 / 8), (reduce, i))
