"""The full-GR step at the edges of its short forms, bit-identical to the oracle: cell
counts around the field update's four faces per thread and its blocks, cells small
against the star (the midpoint's reciprocal from the one at the start of the step, up
to cells of 2^-9 R_*) and large, heights past the short forms' range, and particles that return, cross the tube's ends or
start at x = 0."""
import numpy as np
import pytest

from gpu_common import assert_state_equal, make_pair
from paper_1011_6330_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [8, 8 | 1, 8 | 2])
@pytest.mark.parametrize("N,r_star", [(2, 10.0), (3, 0.3), (4, 10.0), (5, 5.12), (6, 5.11), (7, 10.0), (255, 3.0),
                                      (1023, 5.12), (1024, 5.11), (1025, 10.0), (2050, 0.5), (260, 1e-60)])
def test_gr_step_edges(N, r_star, flags):
    cfg = dict(synth.preset("c1"), n_cells=N, length=0.01 * N, kappa=0.15, r_star=r_star, rg_over_rstar=0.4, flags=flags,
               ppc=10.0, capacity=40 * N + 20000)
    x, u = synth.random_particles(N, 2 * N + 7, seed=N)
    x[0] = 0.0
    g, o = make_pair(cfg, x, u)
    for m in (1, 2, 30):
        g.step(m)
        o.step(m)
        assert_state_equal(g, o, what=f"{N} cells, star of {r_star}, flags {flags}, after {m} more steps")
    g.close()
