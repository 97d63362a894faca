"""GPU parity (-m gpu) of contractions whose rows, columns and depth are no multiple of a tile, a slice
or a 16-byte chunk, against the CPU oracle; operands are the middle part of larger buffers whose other
elements are NaN, so that a value from past an edge shows."""
import numpy as np
import pytest

from oracle.numeric import Eager, round_to_bf16
from test_gpu_parity import check, ctx, rng  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (3, 5, 7), (9, 65, 33), (127, 129, 31), (129, 63, 32), (130, 200, 64), (200, 64, 200), (201, 203, 97), (64, 72, 136), (136, 257, 264),
          (300, 10, 160), (256, 130, 1000), (77, 128, 4101), (5, 64, 1100), (40, 192, 2052), (16, 64, 1025), (700, 1030, 70)]


def window(B, full, rows):
    return B.narrow(full, 0, 1, rows)


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_ragged(ctx, m, n, k, ta, tb, dt):  # noqa: F811
    """Bar: bf16 2e-2 of the result's largest value (one bf16 rounding of it, and of the inputs of the sum
    with a bias; the products themselves are exact in fp32); fp32 1e-5, and 6e-8 of the terms'
    magnitudes adding up like a random walk where k is long."""
    E, g = Eager(), rng(m * 7 + n * 11 + k)
    rnd = round_to_bf16 if dt == "bf16" else (lambda t: t)
    tol = 2e-2 if dt == "bf16" else max(1e-5, 1e-6 * k ** 0.5)

    def operand(rows, cols):
        t = np.full((rows + 2, cols), np.nan, np.float32)
        t[1:-1] = rnd(g.standard_normal((rows, cols), dtype=np.float32))
        return t
    a, b = operand(*((k, m) if ta else (m, k))), operand(*((n, k) if tb else (k, n)))
    bias, res = (rnd(g.standard_normal(s, dtype=np.float32)) for s in ((n,), (m, n)))

    def prog(B, a, b, bias, res):
        p = B.matmul(window(B, a, a.shape[0] - 2), window(B, b, b.shape[0] - 2), trans_a=ta, trans_b=tb)
        q = B.matmul(window(B, a, a.shape[0] - 2), window(B, b, b.shape[0] - 2), trans_a=ta, trans_b=tb)
        return p, B.add(B.relu(B.add(q, bias)), res)
    got = prog(ctx, *(ctx.tensor(t, dtype=dt) for t in (a, b, bias, res)))
    ref = prog(E, *(E.tensor(t, dtype=dt) for t in (a, b, bias, res)))
    for i, (x, y) in enumerate(zip(got, ref)):
        check(ctx, E, x, y, tol, i)


@pytest.mark.parametrize("s,h,d", [(200, 3, 64), (201, 2, 32), (33, 4, 128), (259, 2, 64), (16, 5, 32)])
def test_ragged_attention_products(ctx, s, h, d):  # noqa: F811
    """The five products of an attention layer over heads that are split and merged by views."""
    E, g = Eager(), rng(s * 100 + h * 10 + d)
    q, k, v, dc = (round_to_bf16(g.standard_normal((2 * s, h * d), dtype=np.float32)) for _ in range(4))

    def prog(B, q, k, v, dc):
        split = lambda t: B.permute(B.reshape(t, (2, s, h, d)), (0, 2, 1, 3))                  # noqa: E731
        merge = lambda t: B.reshape(B.permute(t, (0, 2, 1, 3)), (2 * s, h * d))                # noqa: E731
        qh, kh, vh, dh = (split(t) for t in (q, k, v, dc))
        p = B.softmax(B.mul(B.matmul(qh, kh, trans_b=True), 0.125))
        ds = B.softmax_grad(B.matmul(dh, vh, trans_b=True), p)
        return merge(B.matmul(p, vh)), merge(B.matmul(ds, kh)), merge(B.matmul(ds, qh, trans_a=True)), merge(B.matmul(p, dh, trans_a=True))
    got = prog(ctx, *(ctx.tensor(t, dtype="bf16") for t in (q, k, v, dc)))
    ref = prog(E, *(E.tensor(t, dtype="bf16") for t in (q, k, v, dc)))
    for i, (x, y) in enumerate(zip(got, ref)):
        check(ctx, E, x, y, 2e-2, i)


# second: several partial products are left, and a launch that adds them up
@pytest.mark.parametrize("dt,m,n,k,second", [("bf16", 600, 600, 500, False), ("bf16", 1000, 1000, 2100, True), ("bf16", 129, 1544, 583, False),
                                             ("bf16", 3100, 64, 600, False), ("bf16", 257, 1096, 545, False), ("bf16", 600, 600, 549, False),
                                             ("f32", 1000, 1000, 136, False), ("f32", 1000, 1000, 163, False), ("f32", 1000, 1000, 240, False),
                                             ("f32", 500, 1000, 2050, True), ("f32", 997, 1000, 137, False), ("f32", 960, 968, 203, False),
                                             ("f32", 1000, 1024, 257, False), ("f32", 1400, 257, 512, True)])
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False), (True, True)])
def test_halves_of_a_workgroup(ctx, dt, m, n, k, second, ta, tb):  # noqa: F811
    """Shapes whose workgroups are two halves that share k: odd numbers of slices, a rest of k, tiles over both edges, rows that start off a
    16-byte boundary, narrow tiles; as it is, with bias and GELU, and added to a residual.  Bars as above."""
    E, g = Eager(), rng(m * 7 + n * 11 + k)
    rnd = round_to_bf16 if dt == "bf16" else (lambda t: t)

    def operand(rows, cols, std=1.0):
        t = np.full((rows + 2, cols), np.nan, np.float32)
        t[1:-1] = rnd(g.standard_normal((rows, cols), dtype=np.float32) * np.float32(std))
        return t
    a, b = operand(*((k, m) if ta else (m, k))), operand(*((n, k) if tb else (k, n)), std=k ** -0.5)
    bias, res = (rnd(g.standard_normal(s, dtype=np.float32)) for s in ((n,), (m, n)))

    def prog(B, post):
        a_, b_, bias_, res_ = (B.tensor(t, dtype=dt) for t in (a, b, bias, res))
        p = B.matmul(window(B, a_, a.shape[0] - 2), window(B, b_, b.shape[0] - 2), trans_a=ta, trans_b=tb)
        return p if post == "plain" else B.gelu(B.add(p, bias_)) if post == "gelu" else B.add(res_, p, alpha=0.5)
    for post in ("plain", "gelu", "residual"):
        got = prog(ctx, post)
        ctx.set_profiling(True)
        ctx.barrier()
        names = [r["kernel"] for r in ctx.last_launches()]
        ctx.set_profiling(False)
        assert names[0].startswith("lt_gemm") and names[0].rstrip(">").endswith(",2") and len(names) == (2 if second else 1), names
        check(ctx, E, got, prog(E, post), 2e-2 if dt == "bf16" else max(1e-5, 1e-6 * k ** 0.5), post)


@pytest.mark.parametrize("m,n,k,post,halves", [(100, 256, 520, "plain", 2), (100, 256, 520, "gelu", 1), (500, 704, 520, "gelu", 2), (600, 704, 800, "plain", 2),
                                               (600, 704, 800, "gelu", 1), (800, 904, 800, "gelu", 2), (1280, 1280, 800, "moments", 1), (1280, 1280, 800, "plain", 2),
                                               (1024, 1024, 1400, "plain", 2), (1024, 1024, 1400, "moments", 1), (512, 768, 4200, "plain", 2), (512, 3072, 4200, "plain", 1)])
def test_where_halves_are_taken(ctx, m, n, k, post, halves):  # noqa: F811
    """bf16: few tiles with a program in the epilogue, an odd number of partial products of which fp32 results come or whose
    k is long, keep a workgroup for each.  Bar: 2e-2 of the largest value, also of fp32 results, as the oracle rounds the product that
    the launch combines them with as it is."""
    E, g = Eager(), rng(m + n + k)
    mk = lambda *s: round_to_bf16(g.standard_normal(s, dtype=np.float32))                     # noqa: E731
    a, b, bias = mk(m, k), round_to_bf16(g.standard_normal((k, n), dtype=np.float32) * np.float32(k ** -0.5)), mk(n)
    m0, v0 = (g.standard_normal((m, n), dtype=np.float32) for _ in range(2))

    def prog(B):
        p = B.matmul(B.tensor(a, dtype="bf16"), B.tensor(b, dtype="bf16"))
        if post == "plain":
            return [p]
        if post == "gelu":
            u = B.add(p, B.tensor(bias, dtype="bf16"))
            return [u, B.gelu(u)]
        m1, v1 = B.add(B.mul(B.tensor(m0), 0.9), p, alpha=0.1), B.add(B.mul(B.abs(B.tensor(v0)), 0.99), B.square(p), alpha=0.01)
        return [m1, v1, B.div(m1, B.add(B.sqrt(v1), 0.5))]
    got = prog(ctx)
    ctx.set_profiling(True)
    ctx.barrier()
    names = [r["kernel"] for r in ctx.last_launches()]
    ctx.set_profiling(False)
    assert names[0].endswith(f",{halves}>"), names
    for i, (x, y) in enumerate(zip(got, prog(E))):
        check(ctx, E, x, y, 2e-2, (post, i))


@pytest.mark.parametrize("m,n,k,share", [(70, 1000, 2000, 2), (33, 1300, 1100, 3), (33, 1000, 2000, 4), (33, 800, 2000, 5), (33, 650, 2000, 6), (20, 1000, 2100, 8),
                                         (100, 1024, 1300, 2), (70, 1024, 1300, 3), (40, 1088, 1300, 5), (20, 1024, 2000, 8)])
def test_shared_tiles(ctx, m, n, k, share):  # noqa: F811
    """Workgroups that share a tile (two to eight of them; tiles of 32 x 32, 64 x 32 and 16 x 64) and add up one another's
    partial products, in fp32.  Bar as above."""
    E, g = Eager(), rng(m + n + k)
    a, b, bias, res = (g.standard_normal(s, dtype=np.float32) for s in ((m, k), (k, n), (n,), (m, n)))

    def prog(B):
        return B.add(B.relu(B.add(B.matmul(B.tensor(a), B.tensor(b)), B.tensor(bias))), B.tensor(res))
    got = prog(ctx)
    ctx.set_profiling(True)
    ctx.barrier()
    names = [r["kernel"] for r in ctx.last_launches()]
    ctx.set_profiling(False)
    assert len(names) == 1 and names[0].startswith("lt_gemm_small_kernel"), names
    check(ctx, E, got, prog(E), max(1e-5, 1e-6 * k ** 0.5), share)
