"""GPU (-m gpu): global reductions around the sizes where their workgroups' share changes, where tiles of the rest run out and where the
last vector is not whole; prologues that are applied in place and interpreted ones.  Against 64 bits: fp32 sums whose terms are added in
runs of at most a few hundred, 2e-6 of the sum of magnitudes; maxima are exact."""
import numpy as np
import pytest

from test_gpu_parity import ctx, rng  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 1024, 4097, 8191, 262147, 786432, 786433, 1000003, 1049600, 3145728, 3145731, 4194309])
@pytest.mark.parametrize("form", ["square", "abs", "plain", "chain", "max abs"])
def test_rest_of_a_global_reduction(ctx, n, form):  # noqa: F811
    x = rng(n).standard_normal(n).astype(np.float32)
    x[-1] = 50.0                      # (the last element counts)
    t = ctx.tensor(x)
    e = x.astype(np.float64)
    if form == "square":
        got, exact, mass = ctx.sum(ctx.square(t)), (e * e).sum(), (e * e).sum()
    elif form == "abs":
        got, exact, mass = ctx.sum(ctx.abs(t)), np.abs(e).sum(), np.abs(e).sum()
    elif form == "plain":
        got, exact, mass = ctx.sum(t), e.sum(), np.abs(e).sum()
    elif form == "chain":
        got = ctx.mean(ctx.add(ctx.mul(t, 0.5), 1.0))
        exact, mass = (0.5 * e + 1).mean(), np.abs(0.5 * e + 1).mean()
    else:
        got, exact, mass = ctx.amax(ctx.abs(t)), np.abs(e).max(), 0.0
    ctx.barrier()
    assert abs(float(ctx.fetch(got)) - exact) <= 2e-6 * mass
