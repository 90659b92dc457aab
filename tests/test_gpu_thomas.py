"""The tridiagonal solve where its chunks of 512 rows, its eight rows per lane and
its pipeline end: the Poisson start bit-identical to the oracle with and without
the lapse, and its transpose through one reverse step."""
import numpy as np
import pytest

from gpu_common import make_pair, say
from paper_1011_6330_amd import synth

pytestmark = pytest.mark.gpu

SIZES = [2, 3, 8, 9, 511, 512, 513, 1023, 1025, 2049, 3072, 5121]


@pytest.mark.parametrize("lapse", [False, True])
@pytest.mark.parametrize("N", SIZES)
def test_poisson_chunk_edges_bit_identical(N, lapse):
    cfg = dict(synth.preset("c1"), n_cells=N, length=0.01 * N, rho_kind=synth.RHO_FRAME_DRAG, kappa=0.15, r_star=3.0,
               flags=9 if lapse else 1, rg_over_rstar=0.4 if lapse else 0.0, capacity=20000)
    g, o = make_pair(cfg, *synth.random_particles(N, 5000, seed=N))
    d = g.diagnostics()
    assert np.array_equal(d["ez"], o.ez) and np.array_equal(d["er"], o.er)
    g.close()


# one reverse step, as test_adjoint_few_steps_tight (its bound: 1e-12 of the largest)
@pytest.mark.parametrize("N", [3, 511, 512, 513, 1025, 2049])
def test_transposed_solve_chunk_edges(N):
    cfg = dict(n_cells=N, length=0.05 * N, radius=1.0, dt_over_dz=0.5, q_over_m=synth.q_over_m_for(12.0), ppc=30.0,
               rho_kind=2, rho_amp=1.0, kappa=0.15, r_star=10.0, knots=np.ones(9), capacity=20000, warm=0, sort_every=0)
    cfg["macro_charge"] = -(1.0 - cfg["kappa"]) * 0.05 / cfg["ppc"]
    rng = np.random.default_rng(N)
    x = np.concatenate([N - rng.uniform(0.0, 0.4, 200), rng.uniform(0.0, N, 3000)])
    x = np.minimum(x, np.nextafter(float(N), 0.0))
    u = np.concatenate([rng.uniform(2.0, 30.0, 200), rng.uniform(-5.0, 30.0, 3000)])
    g, o = make_pair(cfg, x, u)
    r = g.run_adjoint(1, 1)
    loss, nex, g_rho, _ = o.adjoint(1)
    assert r["loss"] == loss and r["n_exit"] == nex > 0
    err = np.abs(r["g_rho"] - g_rho).max() / np.abs(g_rho).max()
    say("transposed solve", N, err)
    assert err <= 1e-12
    g.close()
