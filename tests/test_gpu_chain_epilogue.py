"""GPU parity (-m gpu) of contractions whose post program is evaluated as a chain, and of neighbours that are not
one, at sizes around tiles, 16-byte chunks and what a lane takes per trip, against the CPU oracle."""
import numpy as np
import pytest

from oracle.numeric import Eager, round_to_bf16
from test_gpu_parity import check, ctx, rng  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu


def programs(B, p, t):
    """name -> results of the product `p`; t: bias, bias2 [n]; x, y [m, n].  The last three are no chains: an earlier
    value read again, a third full input, more steps than a chain has."""
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


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("m,n,k", [(1, 8, 40), (130, 136, 72), (257, 200, 96), (300, 60, 1088), (129, 264, 33), (512, 768, 64)])
def test_post_programs(ctx, m, n, k, dt):  # noqa: F811
    """Bar: bf16 2e-2 of the result's largest value (one rounding of it, and of what the product is combined with);
    fp32 1e-5, and 1e-6 times the square root of k for its sum.  (k: more than 1024 or 512 x 768 columns leave the
    one-launch kernels for small fp32 products.)"""
    E, g = Eager(), rng(m * 7 + n * 11 + k)
    rnd = round_to_bf16 if dt == "bf16" else (lambda t: t)
    mk = lambda *s: rnd(g.standard_normal(s, dtype=np.float32))                               # noqa: E731
    a, b = mk(m, k), rnd((g.standard_normal((k, n), dtype=np.float32) / np.float32(k ** 0.5)))
    t = {"bias": mk(n), "bias2": mk(n), "x": mk(m, n), "y": mk(m, n), "z": mk(m, n)}
    for name in NAMES:
        got, ref = (programs(B, B.matmul(B.tensor(a, dtype=dt), B.tensor(b, dtype=dt)), {q: B.tensor(v, dtype=dt) for q, v in t.items()})[name] for B in (ctx, E))
        for i, (x, y) in enumerate(zip(got, ref)):
            check(ctx, E, x, y, 2e-2 if dt == "bf16" else max(1e-5, 1e-6 * k ** 0.5), f"{name} {i}")


@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_update_in_place(ctx, dt):  # noqa: F811
    """The full input of a chain is also what it overwrites."""
    E, g = Eager(), rng(5)
    rnd = round_to_bf16 if dt == "bf16" else (lambda t: t)
    a, b, w = (rnd(g.standard_normal(s, dtype=np.float32)) for s in ((300, 1100), (1100, 264), (300, 264)))
    out = []
    for B in (ctx, E):
        W = B.tensor(w, dtype=dt, donatable=True) if B is ctx else B.tensor(w, dtype=dt)
        B.assign(W, B.sub(W, B.mul(B.matmul(B.tensor(a, dtype=dt), B.tensor(b, dtype=dt)), 0.01)))
        out.append(W)
    check(ctx, E, out[0], out[1], 2e-2 if dt == "bf16" else 4e-5, "w")
