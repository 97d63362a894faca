"""GPU (-m gpu): a context that was never told how many streams to use decides by the plan whether it spreads; results are bit-identical
to one stream and to four, whatever it decides (few edges and long launches, many edges and short ones)."""
import numpy as np
import pytest

from test_gpu_parity import _stream_case, rng

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,schedule,default", [(64, 256, 1, 1), (1024, 512, 1, 1),              # nothing leaves the caller's stream
                                                        (4096, 512, 4, 1), (8192, 256, 4, 1),            # declined
                                                        (2048, 1024, 4, 4), (8192, 1024, 4, 4)])         # spread
def test_default_streams_do_not_change_results(rows, cols, schedule, default):
    from paper_2102_13267_amd import Context
    g = rng(rows + cols)
    data = [g.standard_normal(s).astype(np.float32) * f for s, f in (((rows, cols), 1.0), ((cols, cols // 2), 0.03), ((cols, cols), 0.03), ((rows, cols), 1.0))]
    results = []
    for n_streams in (None, 1, 4):
        c = Context(device=0, workspace_bytes=2 << 30)
        if n_streams:
            c.set_streams(n_streams)
        steps = []
        for _ in range(2):
            outs = _stream_case(c, *data)
            c.barrier(False)
            steps.append([c.fetch(t).copy() for t in outs])
        assert c.plan_streams() == {None: default, 1: 1, 4: schedule}[n_streams]
        results.append(steps)
        c.close()
    for other in results[1:]:
        for a_step, b_step in zip(results[0], other):
            for a, b in zip(a_step, b_step):
                assert np.array_equal(a, b)
