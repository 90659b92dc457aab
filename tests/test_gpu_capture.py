"""pic_step captured into a caller's graph.  A capture of an even number of steps (in one
call or two), over whole sort rounds where the tube sorts, starts and ends with the
same buffers, so each replay advances the tube by that many steps, also with eager
steps between the replays; every replay is compared, bit for bit, with a tube stepped
eagerly.  A capture that is never replayed leaves the tube as it was."""
import numpy as np
import pytest

from gpu_common import say
from paper_1011_6330_amd import synth

pytestmark = pytest.mark.gpu

SCALARS = ("n_alive", "n_slots", "n_injected", "n_exit", "n_absorb", "last_n_inj", "w0", "status", "e_surf",
           "exit_sum_lo", "exit_sum_hi", "step")


def _state(t):
    d = t.diagnostics(n_bins=16, fields=True, j=True, raise_on_status=False)
    x, u = t.read_particles()
    k = np.lexsort((u, x))
    return dict({q: d[q] for q in SCALARS + ("ez", "er", "b_phi", "j_last", "prof_count", "prof_sum_lo")}, x=x[k], u=u[k])


def _make(precision, sort_every, batch):
    from paper_1011_6330_amd import Batch, Tube
    p = synth.tube_params(dict(synth.preset("c1"), precision=precision, sort_every=sort_every, gamma_fp64=8.0))
    b = Batch([p, dict(p, n_cells=700, length=7.0)]) if batch else Tube(p)
    tubes = b.tubes if batch else [b]
    for t in tubes:
        t.inject(*synth.random_particles(t.N, 900, seed=5))
    b.step(0)
    b.sync()
    return b, tubes


def _capture(b, calls):
    import torch
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=b.stream):
        for m in calls:
            b.step(m)
    return g


def _same(ta, tb, what):
    for k, (a, b) in enumerate(zip(ta, tb)):
        sa, sb = _state(a), _state(b)
        for q in sa:
            assert np.array_equal(sa[q], sb[q], equal_nan=True), f"{what}, tube {k}: {q} differs"


CALLS = [(2,), (4,), (6,), (8,), (10,), (12,), (16,), (64,), (1, 1), (3, 3), (5, 1), (7, 9)]


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("calls,sort_every", [(c, 0) for c in CALLS] + [((16,), 8), ((32,), 16), ((24,), 4), ((8,), 1)])
def test_replays_equal_eager_steps(calls, sort_every, precision, batch):
    import torch
    say("capture", calls, "sort", sort_every, "precision", precision, "batch", batch)
    a, ta = _make(precision, sort_every, batch)
    b, tb = _make(precision, sort_every, batch)
    g = _capture(b, calls)
    between = 2 * sort_every if sort_every else 4
    for r in range(4):
        with torch.cuda.stream(b.stream):
            g.replay()
        torch.cuda.synchronize()
        a.step(sum(calls))
        a.sync()
        _same(ta, tb, f"replay {r}")
        a.step(between)                    # eager work between the replays
        b.step(between)
        _same(ta, tb, f"eager steps after replay {r}")
    a.close()
    b.close()


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("precision", [0, 1])
def test_capture_never_replayed(precision, batch):
    """The first steps of a tube captured over two sort rounds and the graph dropped: the
    eager steps that follow sort as if it had never been."""
    a, ta = _make(precision, 8, batch)
    b, tb = _make(precision, 8, batch)
    g = _capture(b, (16,))
    del g
    for _ in range(3):
        a.step(16)
        b.step(16)
        _same(ta, tb, "after a dropped capture")
    a.close()
    b.close()
