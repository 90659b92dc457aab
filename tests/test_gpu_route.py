"""A tube or batch that moves from fused steps to separate kernels, and back, as particles
are loaded and leave: the same bits as one stepped one step per call (separate kernels
throughout), graphs of both kinds replayed."""
import numpy as np
import pytest

from gpu_common import say
from paper_1011_6330_amd import synth

pytestmark = pytest.mark.gpu

N = 700


def _state(t):
    d = t.diagnostics(n_bins=16, fields=True, j=True, raise_on_status=False)
    x, u = t.read_particles()
    k = np.lexsort((u, x))
    return dict(d, x=x[k], u=u[k])


def _same(ta, tb, what):
    for k, (a, b) in enumerate(zip(ta, tb)):
        sa, sb = _state(a), _state(b)
        for q, v in sa.items():
            assert np.array_equal(v, sb[q], equal_nan=True), f"{what}, tube {k}: {q} differs"


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("sort_every", [0, 8])
def test_route_changes_keep_the_bits(precision, sort_every, batch):
    from paper_1011_6330_amd import Batch, Tube
    n = 4300000 if batch else (2200000 if precision else 1700000)
    p = synth.tube_params(dict(synth.preset("c1"), n_cells=N, length=7.0, ppc=4.0, capacity=n + 100000,
                               precision=precision, gamma_fp64=8.0, sort_every=sort_every, q_over_m=-1e-6))
    x, u = synth.random_particles(N, n, seed=3, u_lo=-0.5, u_hi=20.0)
    order = np.argsort(x)
    x, u = x[order], u[order]
    hs = [Batch([p, dict(p, n_cells=300, length=3.0, capacity=4096)]) if batch else Tube(p) for _ in range(2)]
    tubes = [h.tubes if batch else [h] for h in hs]

    def step(m):
        hs[0].step(m)
        for _ in range(m):
            hs[1].step(1)

    def load(k):
        for t in tubes:
            t[0].inject(x[k], u[k])

    say("route", precision, sort_every, batch)
    load(slice(0, n, 1000))
    step(40)                               # fused
    load(slice(0, n - 10000))              # past the limit: separate
    step(37)
    _same(*tubes, "after the load")
    step(900)                              # most leave; the read-outs tell the host
    for t in tubes:
        t[0].diagnostics(fields=False, raise_on_status=False)   # (clipped injections latch a status)
    step(43)                               # fused again where a sort has dropped the removed slots
    _same(*tubes, "at the end")
    for h in hs:
        h.close()


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("sort_every", [0, 8])
def test_scattered_slots_keep_the_bits(precision, sort_every, batch):
    """Shuffled slots over many cells take separate kernels until a sort, a load of an ordered
    beam goes on fused, a saved state is judged by its slots."""
    from paper_1011_6330_amd import Batch, Tube
    cells, n = 40000, 70000 if batch else 9000
    p = synth.tube_params(dict(synth.preset("c1"), n_cells=cells, length=400.0, ppc=4.0, capacity=400000, flags=1,
                               precision=precision, gamma_fp64=8.0, sort_every=sort_every))
    x, u = synth.random_particles(cells, n, seed=4)
    y, v = synth.random_particles(cells, 3000, seed=5)
    order = np.argsort(y)
    hs = [Batch([p, dict(p, n_cells=300, length=3.0)]) if batch else Tube(p) for _ in range(2)]
    tubes = [h.tubes if batch else [h] for h in hs]
    for t in tubes:
        t[0].inject(x, u)
    for m in (20, 7, 13):
        hs[0].step(m)
        for _ in range(m):
            hs[1].step(1)
        _same(*tubes, f"after {m} steps")
        for t in tubes:
            t[0].inject(y[order], v[order])
    if not batch:
        state = hs[0].save()
        hs[0].load(state)
        c = Tube(p)
        c.load(state)
        for _ in range(24):
            hs[1].step(1)
        hs[0].step(24)
        c.step(24)
        _same(*tubes, "after loading its own state")
        _same([c], [hs[1]], "loaded into another tube")
        c.close()
    for h in hs:
        h.close()
