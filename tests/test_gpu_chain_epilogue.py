"""GPU parity (-m gpu) of contractions whose post program is evaluated as a chain, and of neighbours that are not
one, at sizes around tiles, 16-byte chunks and what a lane takes per trip, against the CPU oracle."""
import numpy as np
import pytest

from oracle.numeric import Eager, round_to_bf16
from test_gpu_parity import check, ctx, rng  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu


def programs(B, p, t):
    """name -> results of the product `p`; t: bias, bias2 [n]; x, y [m, n].  quotient and the last three are
    no chains: a divisor that is computed, an earlier value read again, a third full input, more steps than a chain has."""
    u = B.add(p, t["bias"])
    long = p
    for i in range(9):
        long = B.add(long, t["bias"] if i % 2 else t["x"])
    return {"plain": [p], "bias": [u], "bias_gelu_both": [u, B.gelu(u)], "product_and_relu": [p, B.relu(u)], "gelu_grad": [B.gelu_grad(p, t["x"])],
            "gelu_grad_of": [B.gelu_grad(t["x"], p)], "relu_grad": [B.relu_grad(p, t["x"])], "relu_grad_of": [B.relu_grad(t["x"], p)],
            "residual": [B.add(t["x"], B.gelu(u))], "two_full_two_row": [B.add(B.mul(B.sub(t["y"], B.add(u, t["x"])), t["bias2"]), 0.25)],
            "scaled": [B.add(t["x"], p, alpha=0.3)], "scales": [B.add(B.mul(p, 0.7), t["x"], alpha=-0.6)], "quotients": [B.div(t["x"], B.add(B.square(p), 2.0))],
            "quotient": [B.div(p, B.add(B.abs(t["x"]), 1.0))], "limits": [B.maximum(B.minimum(p, t["x"]), t["bias"])], "roots": [B.sqrt(B.add(B.abs(p), 1.0))],
            "again": [B.add(B.mul(u, t["x"]), p)], "three": [B.add(B.add(B.add(p, t["x"]), t["y"]), t["z"])], "long": [long]}


NAMES = ["plain", "bias", "bias_gelu_both", "product_and_relu", "gelu_grad", "gelu_grad_of", "relu_grad", "relu_grad_of", "residual", "two_full_two_row", "scaled",
         "scales", "quotients", "quotient", "limits", "roots", "again", "three", "long"]


# no chains; and, with the roundings of bf16, a program long enough for a launch of its own behind the product
NO_CHAIN = {"f32": {"quotient", "again", "three", "long"}, "bf16": {"quotient", "again", "three", "long", "two_full_two_row"}}


def contractions(ctx):  # noqa: F811
    """Kernels of the pending step, which is run."""
    ctx.set_profiling(True)
    ctx.barrier()
    names = [r["kernel"] for r in ctx.last_launches()]
    ctx.set_profiling(False)
    return names


def expect_one(names, dt, halves, name=""):
    """One launch, of the LDS-staged kernel, with so many halves to a workgroup."""
    assert len(names) == 1 and names[0].startswith("lt_gemm_bf16_kernel" if dt == "bf16" else "lt_gemm_kernel") and names[0].endswith(f",{halves}>"), (name, names)


@pytest.mark.parametrize("dt,m,n,k,halves", [("bf16", 1, 8, 40, 1), ("bf16", 130, 136, 72, 1), ("bf16", 257, 200, 96, 1), ("bf16", 129, 264, 33, 1), ("bf16", 512, 768, 64, 1),
                                             ("bf16", 600, 600, 520, 2), ("bf16", 129, 1544, 521, 2), ("bf16", 3100, 64, 600, 2), ("bf16", 300, 60, 1088, 0),
                                             ("f32", 1100, 1036, 120, 1), ("f32", 1100, 1036, 123, 1), ("f32", 1990, 2052, 72, 1), ("f32", 1001, 1004, 136, 2),
                                             ("f32", 1001, 1004, 139, 2), ("f32", 1, 8, 40, 0), ("f32", 130, 136, 72, 0), ("f32", 257, 200, 96, 0), ("f32", 300, 60, 1088, 0),
                                             ("f32", 129, 264, 33, 0), ("f32", 512, 768, 64, 0)])
def test_post_programs(ctx, dt, m, n, k, halves):  # noqa: F811
    """Bar: bf16 2e-2 of the result's largest value (one rounding of it, and of what the product is combined with);
    fp32 1e-5, and 1e-6 times the square root of k for its sum.  Halves 1 and 2: one launch of the LDS-staged kernel, which runs a
    chain as such.  (fp32 in tiles of 64 x 64 and 128 x 128; products of few tiles of 16 x 16 times k have kernels of their
    own, which do not, and neither does a second launch over several partial products: halves 0.)"""
    E, g = Eager(), rng(m * 7 + n * 11 + k)
    rnd = round_to_bf16 if dt == "bf16" else (lambda t: t)
    mk = lambda *s: rnd(g.standard_normal(s, dtype=np.float32))                               # noqa: E731
    a, b = mk(m, k), rnd((g.standard_normal((k, n), dtype=np.float32) / np.float32(k ** 0.5)))
    t = {"bias": mk(n), "bias2": mk(n), "x": mk(m, n), "y": mk(m, n), "z": mk(m, n)}
    for name in NAMES:
        got = programs(ctx, ctx.matmul(ctx.tensor(a, dtype=dt), ctx.tensor(b, dtype=dt)), {q: ctx.tensor(v, dtype=dt) for q, v in t.items()})[name]
        names = contractions(ctx)
        if halves and name not in NO_CHAIN[dt]:
            expect_one(names, dt, halves, name)
        ref = programs(E, E.matmul(E.tensor(a, dtype=dt), E.tensor(b, dtype=dt)), {q: E.tensor(v, dtype=dt) for q, v in t.items()})[name]
        for i, (x, y) in enumerate(zip(got, ref)):
            check(ctx, E, x, y, 2e-2 if dt == "bf16" else max(1e-5, 1e-6 * k ** 0.5), f"{name} {i}")


@pytest.mark.parametrize("dt,m,n,k,halves", [("bf16", 300, 264, 440, 1), ("bf16", 600, 600, 520, 2), ("bf16", 300, 264, 1100, 0), ("f32", 1100, 1036, 120, 1),
                                             ("f32", 1001, 1004, 136, 2), ("f32", 300, 264, 1100, 0)])
def test_update_in_place(ctx, dt, m, n, k, halves):  # noqa: F811
    """The full input of a chain is also what it overwrites (halves as above)."""
    E, g = Eager(), rng(5)
    rnd = round_to_bf16 if dt == "bf16" else (lambda t: t)
    a, b, w = (rnd(g.standard_normal(s, dtype=np.float32)) for s in ((m, k), (k, n), (m, n)))
    out = []
    for B in (ctx, E):
        W = B.tensor(w, dtype=dt, donatable=True) if B is ctx else B.tensor(w, dtype=dt)
        B.assign(W, B.sub(W, B.mul(B.matmul(B.tensor(a, dtype=dt), B.tensor(b, dtype=dt)), 0.01)))
        out.append(W)
    names = contractions(ctx)
    if halves:
        expect_one(names, dt, halves)
    check(ctx, E, out[0], out[1], 2e-2 if dt == "bf16" else 4e-5, "w")
