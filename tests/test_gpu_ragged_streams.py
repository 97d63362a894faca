"""GPU parity (-m gpu) of the streamed kernels on sizes that are no multiple of what a lane, a wave or a
workgroup takes at once, against the CPU oracle.  Tolerances as in test_gpu_parity.py: 1e-5 norm-wise
for fp32, sums of N(0,1) terms scaled by the square root of their number (they cancel)."""
import numpy as np
import pytest

from oracle.numeric import Eager
from workloads import programs
from test_gpu_parity import TOL32, check, ctx, rng  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(5, 64), (7, 67), (3, 513), (2049, 130), (4099, 127), (70, 128), (4099, 255), (1025, 1023), (1024, 1028), (33, 4097), (2, 8199), (130, 1777)])
def test_row_reductions_of_any_length(ctx, rows, cols):  # noqa: F811
    """A quarter and half a wave, one, two and four waves per row, two and four vectors per trip, rows that end inside a vector and
    rows that start off a 16-byte boundary; a window as operand; values that must not leak in from
    the next row (the maximum of negative numbers, minus infinity)."""
    E, g = Eager(), rng(rows * 10000 + cols)
    x, y = (g.standard_normal((rows, cols), dtype=np.float32) for _ in range(2))
    x[0, -1] = -np.inf
    b = g.standard_normal(cols, dtype=np.float32)
    w = g.standard_normal((rows + 1, cols), dtype=np.float32)

    def prog(B, x, y, b, w):
        return (B.sum(B.mul(y, y), axis=1), B.amax(B.neg(B.abs(x)), axis=1), B.mean(B.tanh(B.add(B.mul(y, y), b)), axis=1),
                B.sum(B.mul(B.exp(B.neg(B.abs(x))), B.add(y, b)), axis=1), B.sum(B.square(B.narrow(w, 0, 1, rows)), axis=1))
    got = prog(ctx, *(ctx.tensor(t) for t in (x, y, b, w)))
    ref = prog(E, *(E.tensor(t) for t in (x, y, b, w)))
    for i, (gt, rt) in enumerate(zip(got, ref)):
        check(ctx, E, gt, rt, 2e-6 * cols ** 0.5 + TOL32, i)


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1025, 8193, 32770, 669706, 4194305])
def test_global_reductions_of_any_length(ctx, n):  # noqa: F811
    """No whole trip, whole trips and a rest, a rest of one to three elements; the bare operand, a lone
    square or abs, a program with one and with two inputs; sum, maximum and mean."""
    E, g = Eager(), rng(n)
    x, y = (g.standard_normal(n, dtype=np.float32) for _ in range(2))

    def prog(B, x, y):
        return (B.sum(B.square(x)), B.amax(B.neg(B.abs(x))), B.amax(x), B.mean(B.mul(B.mul(x, y), B.mul(x, y))), B.sum(B.exp(B.neg(B.square(y)))))
    got, ref = prog(ctx, ctx.tensor(x), ctx.tensor(y)), prog(E, E.tensor(x), E.tensor(y))
    for i, (gt, rt) in enumerate(zip(got, ref)):
        check(ctx, E, gt, rt, TOL32, i)


@pytest.mark.parametrize("n", [15, 17, 18, 1023, 1025, 2047, 2050, 3073, 100003, 669706, 16777217])
def test_elementwise_of_any_length_in_place(ctx, n):  # noqa: F811
    """An optimiser update in place twice over element counts that are no multiple of four: below and above
    the shortest one that is streamed, a last element alone in its tile, beyond the last-level cache."""
    E, g = Eager(), rng(n)
    p, gr, m = (g.standard_normal(n, dtype=np.float32) for _ in range(3))
    v = np.abs(g.standard_normal(n, dtype=np.float32)) + 0.1

    def run(B, mk):
        ts = [mk(t) for t in (p, gr, m, v)]
        for t in (1, 2):
            programs.c4_step(B, *ts, lr=1e-2, beta1=0.9, beta2=0.999, eps=1e-8, t=t, max_norm=1.0)
            if B is ctx:
                info = ctx.barrier(True)
                assert info.n_regions == (1 if n <= 65536 else 2)     # (up to there the update is the finaliser of the norm)
        return ts
    got, ref = run(ctx, lambda a: ctx.tensor(a, donatable=True)), run(E, E.tensor)
    for gt, rt in zip(got, ref):
        check(ctx, E, gt, rt, TOL32)


@pytest.mark.parametrize("n", [4, 2048, 2049, 2052, 5001, 65536])
def test_finaliser_in_and_behind_the_reduction(ctx, n):  # noqa: F811
    """What consumes the reduced value element by element: in the reduction's own launch, or in one behind
    it; the reduced value itself and a scalar made of it are results as well."""
    E, x = Eager(), rng(n).standard_normal(n, dtype=np.float32)

    def prog(B, x):
        s = B.amax(B.abs(x))
        r = B.sqrt(s)
        return B.div(x, s), s, r, B.mul(B.add(x, r), 2.0)
    got = prog(ctx, ctx.tensor(x))
    ref = prog(E, E.tensor(x))
    for i, (gt, rt) in enumerate(zip(got, ref)):
        check(ctx, E, gt, rt, TOL32, i)
    assert float(np.max(np.abs(ctx.fetch(got[0])))) == 1.0
