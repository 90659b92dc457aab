"""The separate push kernel of a tube (one step per call, lapse tubes) at every launch
shape, nontemporal and plain, in both tile orders, with a partial last tile: FP64 and
the lapse bit-identical to the oracle, FP32-bulk to fused steps."""
import numpy as np
import pytest

from gpu_common import assert_state_equal, make_pair
from paper_1011_6330_amd import synth

pytestmark = pytest.mark.gpu

N = 700
SHAPES = [(b, p, nt) for b in (64, 128, 256, 512) for p in (2, 4, 8) for nt in (False, True)
          if not (p == 4 and b == 512) and not (p == 8 and b > 128)]
SHAPES32 = [(b, 4, nt) for b in (64, 128, 256, 512) for nt in (False, True)]


def _cfg(**over):
    return dict(synth.preset("c2"), n_cells=N, q_over_m=synth.q_over_m_for(60.0), ppc=12.0, warm=12 * N + 77,
                capacity=30 * N, sort_every=8, **over)


def _state(t):
    d = t.diagnostics(n_bins=16, fields=True, j=True)
    x, u = t.read_particles()
    k = np.lexsort((u, x))
    return dict(d, x=x[k], u=u[k])


@pytest.mark.parametrize("shape", SHAPES)
def test_f64_single_steps_match_oracle(shape):
    cfg = _cfg()
    x, u = synth.warm_start(cfg)
    g, o = make_pair(cfg, x, u)
    g.set_push_config(*shape)
    for s in range(20):                    # both tile orders, two sorts
        g.step(1)
        o.step(1)
    assert_state_equal(g, o, ordered=False, what=f"shape {shape}")
    g.close()


@pytest.mark.parametrize("nt", [False, True])
@pytest.mark.parametrize("rounds", [False, True])
def test_lapse_matches_oracle(nt, rounds):
    """Lapse tubes never take fused steps: single steps and replayed rounds."""
    cfg = _cfg(flags=8, rg_over_rstar=0.4)
    x, u = synth.warm_start(cfg)
    g, o = make_pair(cfg, x, u)
    g.set_push_config(128, 2, nt)
    for _ in range(1 if rounds else 20):
        g.step(20 if rounds else 1)
    o.step(20)
    assert_state_equal(g, o, ordered=False, what=f"lapse nt {nt}")
    g.close()


@pytest.mark.parametrize("gamma", [1e6, 8.0])
def test_f32_single_steps_equal_at_every_shape(gamma):
    """All particles in the low stream, and most in the high one."""
    from paper_1011_6330_amd import Tube
    cfg = _cfg(precision=1, gamma_fp64=gamma)
    x, u = synth.warm_start(cfg)
    want = None
    for shape in [None] + SHAPES32:
        t = Tube(synth.tube_params(cfg))
        t.inject(x, u)
        if shape:
            t.set_push_config(*shape)
        for _ in range(20 if shape else 1):
            t.step(1 if shape else 20)     # the first: fused steps
        got = _state(t)
        want = want or got
        for k, v in want.items():
            assert np.array_equal(v, got[k], equal_nan=True), f"shape {shape}: {k} differs"
        t.close()
