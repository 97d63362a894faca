"""GPU parity (-m gpu) of a weight gradient whose optimiser update runs in a second launch over a workspace
that the plan can do without: with it, without it because the library's static scratch is used, and
without it because the caller's workspace is too small (8 MiB, half of them taken by the library's scratch,
against 4.2 MiB and more of product) -- the same bits, and the oracle's values."""
import numpy as np
import pytest

from oracle.numeric import Eager, round_to_bf16
from test_gpu_parity import rel_err, rng

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt,m,n,k", [("bf16", 512, 512, 200), ("bf16", 1028, 1040, 200), ("bf16", 100, 70, 130), ("bf16", 130, 1028, 33), ("f32", 1100, 1030, 70), ("f32", 1028, 1024, 64)])
def test_update_in_a_second_launch_or_in_the_contraction(dt, m, n, k):
    from paper_2102_13267_amd import Context
    g, rnd = rng(m + n + k), (round_to_bf16 if dt == "bf16" else (lambda t: t))
    x, dy, w = (rnd(g.standard_normal(s, dtype=np.float32)) for s in ((k, m), (k, n), (m, n)))
    m0, v0 = g.standard_normal((m, n), dtype=np.float32), np.abs(g.standard_normal((m, n), dtype=np.float32)) + 0.5

    def run(B, mk):
        tx, tdy, tw = (mk(t, dt) for t in (x, dy, w))
        tm, tv = mk(m0, "f32"), mk(v0, "f32")
        for t in (3, 4):
            gr = B.matmul(tx, tdy, trans_a=True)
            m1 = B.add(B.mul(tm, 0.9), gr, alpha=0.1)
            v1 = B.add(B.mul(tv, 0.999), B.square(gr), alpha=0.001)
            step = B.div(B.mul(B.div(m1, 1.0 - 0.9 ** t), 0.1), B.add(B.sqrt(B.div(v1, 1.0 - 0.999 ** t)), 1e-8))
            p1 = B.sub(tw, step)
            B.assign(tw, B.cast(p1, "bf16") if dt == "bf16" else p1)
            B.assign(tm, m1)
            B.assign(tv, v1)
            del gr, m1, v1, step, p1
            yield B
        yield [tw, tm, tv]
    results = []
    for size, static in ((256 << 20, False), (256 << 20, True), (8 << 20, False)):
        c = Context(device=0, workspace_bytes=size)
        it = run(c, lambda a, d, c=c: c.tensor(a.copy(), dtype=d, donatable=True))
        for _ in range(2):
            next(it)
            info = c.barrier_static() if static else c.barrier()
            assert info.n_launches == 2
        results.append([c.fetch(t).copy() for t in next(it)])
        c.close()
    for other in results[1:]:
        for a, b in zip(results[0], other):
            assert np.array_equal(a, b)
    E = Eager()
    it = run(E, lambda a, d: E.tensor(a.copy(), dtype=d))
    next(it)
    next(it)
    for a, r in zip(results[0], next(it)):
        assert rel_err(a, E.fetch(r)) <= (2e-2 if dt == "bf16" else 2e-5)


def adam_steps(c, n_steps, data):
    """Adam on a 1028 x 1040 weight whose gradient is a contraction in bf16; results after n_steps."""
    x, dy, w, m0, v0 = data
    tx, tdy, tw = (c.tensor(t, dtype="bf16", donatable=True) for t in (x, dy, w))
    tm, tv = (c.tensor(t.copy(), donatable=True) for t in (m0, v0))
    for _ in range(n_steps):
        gr = c.matmul(tx, tdy, trans_a=True)
        m1 = c.add(c.mul(tm, 0.9), gr, alpha=0.1)
        v1 = c.add(c.mul(tv, 0.999), c.square(gr), alpha=0.001)
        p1 = c.sub(tw, c.div(c.mul(m1, 0.1), c.add(c.sqrt(v1), 1e-8)))
        c.assign(tw, c.cast(p1, "bf16"))
        c.assign(tm, m1)
        c.assign(tv, v1)
        del gr, m1, v1, p1
        c.barrier()
    return [c.fetch(t).copy() for t in (tw, tm, tv)]


def adam_data():
    g = rng(11)
    x, dy, w = (round_to_bf16(g.standard_normal(s, dtype=np.float32)) for s in ((200, 1028), (200, 1040), (1028, 1040)))
    return x, dy, w, g.standard_normal((1028, 1040), dtype=np.float32), np.abs(g.standard_normal((1028, 1040), dtype=np.float32)) + 0.5


def test_a_step_short_of_the_optional_workspace_keeps_its_graphs():
    """8 MiB hold everything the step needs but the product's workspace: it runs without that, and as one
    HIP graph from the third repetition on, like the step with all its memory; the same bits."""
    from paper_2102_13267_amd import Context
    results = []
    for size in (256 << 20, 8 << 20):
        c = Context(device=0, workspace_bytes=size)
        c.set_graphs(True)
        results.append(adam_steps(c, 6, adam_data()))
        assert c.stats().graph_launches > 0, size
        c.close()
    for a, b in zip(*results):
        assert np.array_equal(a, b)


def test_a_launch_left_out_is_not_reported():
    """Without its workspace the step is one launch: one record with a time of its own, one launch counted."""
    from paper_2102_13267_amd import Context
    for size, n in ((256 << 20, 2), (8 << 20, 1)):
        c = Context(device=0, workspace_bytes=size)
        c.set_profiling(True)
        adam_steps(c, 3, adam_data())
        records = c.last_launches()
        assert len(records) == n and c.stats().kernels_launched == 3 * n
        assert all(r["ms"] > 0 for r in records) and "gemm" in records[0]["kernel"]
        c.close()


def test_streams_without_the_optional_workspaces():
    """A transformer layer step on four streams, with all its memory, then 8 MiB short of that: the optimiser
    updates' workspaces are left out, and with them launches that others are ordered behind; the same bits."""
    from paper_2102_13267_amd import Context
    from test_gpu_parity import spread
    from workloads import programs
    from workloads.inputs import c3_inputs
    bsz, seq, d, ffn, heads = 2, 100, 1024, 4096, 16
    inp, keys, results, counts, size = c3_inputs(bsz, seq, d, ffn), programs.C3_WEIGHTS + programs.C3_VECTORS, [], [], 1 << 30
    for n_streams in (4, 4, 1):
        c = Context(device=0, workspace_bytes=size)
        c.set_streams(n_streams)
        P = {k: c.tensor(round_to_bf16(inp[k]), dtype="bf16", donatable=True) for k in keys}
        M, V = ({k: c.tensor(np.zeros_like(inp[k]), donatable=True) for k in keys} for _ in range(2))
        xt, dyt = c.tensor(round_to_bf16(inp["x"]), dtype="bf16"), c.tensor(round_to_bf16(inp["dy"]), dtype="bf16")
        for step in range(3):
            y, dx = programs.c3_step(c, xt, dyt, P, M, V, heads, t=step + 1)
            assert spread(c, c.barrier())
        counts.append(c.stats().kernels_launched)
        if size == 1 << 30:
            size = c.stats().arena_bytes_peak - (8 << 20)
        results.append([c.fetch(t) for t in [y, dx] + [D[k] for D in (P, M, V) for k in keys]])
        c.close()
    assert counts[0] > counts[1] == counts[2]
    for other in results[1:]:
        for a, b in zip(results[0], other):
            assert np.array_equal(np.asarray(a).view(np.uint8), np.asarray(b).view(np.uint8))
