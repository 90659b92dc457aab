"""Fused steps (one kernel per step) against single steps (push, then field update):
a tube stepped M at a time and one stepped M times once hold the same bits, in FP64
and FP32-bulk, for runs of 2, 3 and 4 steps (the three ways the current buffers can
end) and more, at the edges of the blocks (512 faces, 256 and 512 slots), with
particles spread past the 64-face window, injected particles that stay, return to
the star or are clipped at the capacity, frozen fields, replayed injections and
sorts."""
import numpy as np
import pytest

from gpu_common import assert_state_equal, make_pair
from paper_1011_6330_amd import synth

pytestmark = pytest.mark.gpu


def _state(t):
    d = t.diagnostics(n_bins=16, fields=True, j=True, raise_on_status=False)
    x, u = t.read_particles()
    k = np.lexsort((u, x))
    return dict(d, x=x[k], u=u[k])


def _same(a, b, what):
    for k, v in a.items():
        assert np.array_equal(v, b[k], equal_nan=True), f"{what}: {k} differs"


CASES = {
    "cold": dict(cfg=dict(), n=0),
    "n2": dict(cfg=dict(n_cells=2, length=0.02), n=3),
    "n511": dict(cfg=dict(n_cells=511), n=255),
    "n512": dict(cfg=dict(n_cells=512), n=256),
    "n513_sorted": dict(cfg=dict(n_cells=513, sort_every=4), n=257),
    "spread": dict(cfg=dict(n_cells=5000, length=40.0), n=1025),
    "dense_sorted": dict(cfg=dict(n_cells=700, ppc=60.0, sort_every=8), n=40000),
    "returning": dict(cfg=dict(q_over_m=+30.0), n=500),
    "clipped": dict(cfg=dict(capacity=600), n=100),
    "roomy": dict(cfg=dict(n_cells=2000, capacity=5 << 20), n=40000),   # more slots than twice the expected ones
    "frozen": dict(cfg=dict(flags=2), n=500),
    "no_injection": dict(cfg=dict(flags=1), n=500),
}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("case", sorted(CASES))
def test_runs_equal_single_steps(case, precision):
    from paper_1011_6330_amd import Tube
    cfg = dict(synth.preset("c1"), precision=precision, gamma_fp64=8.0, **CASES[case]["cfg"])
    ts = [Tube(synth.tube_params(cfg)) for _ in range(2)]
    for t in ts:
        if CASES[case]["n"]:
            t.inject(*synth.random_particles(int(cfg["n_cells"]), CASES[case]["n"], seed=5))
    for M in (2, 3, 4, 1, 7, 64, 40):
        ts[0].step(M)
        for _ in range(M):
            ts[1].step(1)
        _same(_state(ts[1]), _state(ts[0]), f"{case} after a run of {M}")
    for t in ts:
        t.close()


def test_runs_match_oracle_with_schedule():
    cfg = dict(synth.preset("c1"), n_cells=777)
    g, o = make_pair(cfg)
    counts = (np.arange(60) * 7) % 11
    g.set_injection_schedule(counts, first_step=3)
    g.step(3)
    o.step(3)
    assert_state_equal(g, o, what="before the schedule")
    g.step(29)
    inj = g.diagnostics(fields=False)["n_injected"] - o.counters["n_injected"]
    assert inj == counts[:29].sum()
    h, _ = make_pair(cfg)
    h.set_injection_schedule(counts, first_step=3)
    for _ in range(32):
        h.step(1)
    _same(_state(h), _state(g), "schedule")
    g.close()
    h.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("sort_every", [0, 8])
def test_batch_runs_equal_single_steps(precision, sort_every):
    from paper_1011_6330_amd import Batch
    base = dict(synth.preset("c1"), precision=precision, sort_every=sort_every, gamma_fp64=8.0)
    sizes = [(2, 3), (513, 700), (1024, 0), (2100, 5000)]
    cfgs = [dict(base, n_cells=N, length=0.01 * N, capacity=2 * n + 3000) for N, n in sizes]
    bs = [Batch([synth.tube_params(c) for c in cfgs]) for _ in range(2)]
    for b in bs:
        for t, (N, n) in zip(b.tubes, sizes):
            if n:
                t.inject(*synth.random_particles(N, n, seed=N))
    for M in (2, 3, 4, 1, 14, 16):
        bs[0].step(M)
        for _ in range(M):
            bs[1].step(1)
        for k in range(len(sizes)):
            _same(_state(bs[1].tubes[k]), _state(bs[0].tubes[k]), f"tube {k} after a run of {M}")
    for b in bs:
        b.close()
