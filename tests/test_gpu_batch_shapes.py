"""The separate batched kernels (work list, push, field update) at every kind of launch
shape, in graphed and direct rounds and one step per call: a batch that expects more
slots than fused steps take, in FP64 and FP32-bulk, against its tubes stepped alone."""
import numpy as np
import pytest

from gpu_common import say
from paper_1011_6330_amd import synth

pytestmark = pytest.mark.gpu

N = 700


def _cfg(**over):
    return dict(synth.preset("c2"), q_over_m=synth.q_over_m_for(60.0), sort_every=8, ppc=4000.0, capacity=3 << 20, **over)


def _state(t):
    d = t.diagnostics(n_bins=16, fields=True, j=True)
    x, u = t.read_particles()
    k = np.lexsort((u, x))
    return dict(d, x=x[k], u=u[k])


@pytest.mark.parametrize("precision", [0, 1])
def test_batch_past_the_fused_size(precision):
    from paper_1011_6330_amd import Batch, Tube
    cfgs = [dict(_cfg(precision=precision, gamma_fp64=8.0), n_cells=n, warm=8 * n + 5) for n in (N, 513, 1100)]
    loads = [synth.warm_start(c, seed=k) for k, c in enumerate(cfgs)]
    want = []
    for c, (x, u) in zip(cfgs, loads):
        t = Tube(synth.tube_params(c))
        t.inject(x, u)
        for _ in range(20):
            t.step(1)
        want.append(_state(t))
        t.close()
    shapes = [(256, 4), (64, 4), (512, 4)] if precision else [(256, 2), (64, 4), (512, 2), (128, 2)]
    for block, per in shapes:
        for graph in (True, False):
            for calls in ((20,), (1,) * 20):
                say("batch", precision, block, per, graph, len(calls))
                b = Batch([synth.tube_params(c) for c in cfgs])
                b.set_config(block, per, graph=graph)
                for t, (x, u) in zip(b.tubes, loads):
                    t.inject(x, u)
                for m in calls:
                    b.step(m)
                for k, t in enumerate(b.tubes):
                    got = _state(t)
                    for q, v in want[k].items():
                        assert np.array_equal(v, got[q], equal_nan=True), f"tube {k}, {block}x{per}: {q} differs"
                b.close()
