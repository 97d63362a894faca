"""A step that would fit its workspace with every region in a launch of its own fits it: what lowering merges
and regroups may want memory earlier, and is undone when there is none.  Null device, then (-m gpu) values."""
import numpy as np
import pytest

from paper_2102_13267_amd import Context
from paper_2102_13267_amd.lt import LtError


def scaled(B, x):
    """x / max|x|: a finaliser of 4096 elements runs behind its reduction and reads the maximum from memory."""
    return [B.div(x, B.amax(B.abs(x)))]


def norm(B, x, dy, g, b):
    """A norm, its input's gradient and both parameters': the bias gradient's sum rides along in the launch of the weight gradient."""
    rows = x.shape[0]
    y, mu, rs = B.layer_norm(x, g, b, eps=1e-5)
    xhat = B.mul(B.sub(x, B.reshape(mu, (rows, 1))), B.reshape(rs, (rows, 1)))
    return [y, B.layer_norm_grad(dy, x, g, mu, rs), B.sum(B.mul(dy, xhat), axis=0), B.sum(dy, axis=0)]


# program, shapes of its inputs, bytes that its parts need at once (granules of 256), launches with room and without
CASES = [(scaled, [(4096,)], 4096 * 4, 2, 1),
         # (the statistics of 100 rows are read for the last time by the weight gradient: the bias gradient takes their place)
         (norm, [(100, 128), (100, 128), (128,), (128,)], 2 * 100 * 128 * 4 + 512 + 2 * 512, 3, 4)]


def library_bytes():
    c = Context(workspace_bytes=64 << 20)
    n = c.stats().arena_bytes_in_use
    c.close()
    return n


@pytest.mark.parametrize("prog,shapes,need,merged,apart", CASES)
def test_fits_where_its_parts_fit(prog, shapes, need, merged, apart):
    for spare, n in ((64 << 20, merged), (0, apart), (-256, None)):
        c = Context(workspace_bytes=library_bytes() + need + spare)
        keep = prog(c, *(c.tensor(np.zeros(s, np.float32)) for s in shapes))
        if n is None:
            with pytest.raises(LtError):
                c.barrier()
        else:
            assert c.barrier().n_launches == n
        del keep
        c.close()


@pytest.mark.gpu
@pytest.mark.parametrize("prog,shapes,need,merged,apart", CASES)
def test_values(prog, shapes, need, merged, apart):
    """The same step twice in the least memory, by the spare plan: 1e-5 (2e-5 for sums that cancel) of the largest value."""
    from oracle.numeric import Eager
    g, E = np.random.Generator(np.random.PCG64(9)), Eager()
    data = [g.standard_normal(s).astype(np.float32) for s in shapes]
    c = Context(device=0, workspace_bytes=16 << 20)
    left = (16 << 20) - c.stats().arena_bytes_in_use - need
    rest = c.neg(c.tensor(np.zeros(left // 4, np.float32)))          # (takes what the step does not need)
    c.barrier()
    ref = [E.fetch(t) for t in prog(E, *(E.tensor(t) for t in data))]
    tensors = [c.tensor(t) for t in data]
    for _ in range(2):
        out = prog(c, *tensors)
        assert c.barrier().n_launches == apart
        for a, b in zip(out, ref):
            assert np.max(np.abs(c.fetch(a) - b)) <= 2e-5 * np.max(np.abs(b))
        del out, a
    del rest
    c.close()
