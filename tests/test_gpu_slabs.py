"""GPU (-m gpu): bf16 products whose workgroups' halves share slabs of 64 k, where the last slab has only its first half (an odd
number of slices) and where a rest of k follows, in all layouts, tiles whole and over the edge.  Small whole numbers: every product and
partial sum is exact in fp32, and results below 256 in bf16 (compared bit for bit); both operands end with their last row's end."""
import numpy as np
import pytest

from test_gpu_parity import ctx, rng  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [512, 544, 576, 600, 608, 640, 680])
@pytest.mark.parametrize("trans", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("m,n", [(512, 1024), (450, 1000), (504, 72)])
def test_odd_slabs(ctx, m, n, k, trans):  # noqa: F811
    g = rng(m * 13 + n * 7 + k)
    # (few entries are not zero: sums stay below 256)
    a, b = ((g.integers(-2, 3, s) * (g.random(s) < 0.15)).astype(np.float32) for s in ((k, m) if trans[0] else (m, k), (n, k) if trans[1] else (k, n)))
    c = ctx.matmul(ctx.tensor(a, dtype="bf16"), ctx.tensor(b, dtype="bf16"), trans_a=trans[0], trans_b=trans[1])
    ctx.set_profiling(True)
    ctx.barrier()
    names = [r["kernel"] for r in ctx.last_launches()]
    ctx.set_profiling(False)
    assert names[0].rstrip(">").endswith(",2"), names
    exact = (a.T if trans[0] else a).astype(np.float64) @ (b.T if trans[1] else b).astype(np.float64)
    assert np.abs(exact).max() < 256
    assert np.array_equal(ctx.fetch(c), exact.astype(np.float32))
