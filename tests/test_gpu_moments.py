"""The particle pass of the diagnostics (signed-gamma profile and node weights in
one read) at the sizes where its blocks, its LDS windows and its accumulators
end: against an evaluation of the same integer sums in NumPy from the particles
the tube holds.  Every result is an integer or one of the values, so it is exact."""
import numpy as np
import pytest

from paper_1011_6330_amd import synth

pytestmark = pytest.mark.gpu


def _expected(x, u, N, nb, bits):
    g = np.sqrt(1.0 + u * u)
    g = np.where(u < 0.0, -g, g)
    b = np.clip(np.floor((x * float(nb)) / float(N)).astype(np.int64), 0, nb - 1)
    fl = np.floor(g)
    fr = np.rint((g - fl) * 4294967296.0)
    cnt = np.bincount(b, minlength=nb)
    lo, hi = np.zeros(nb, np.uint64), np.zeros(nb, np.int64)
    mn, mx = np.full(nb, np.inf), np.full(nb, -np.inf)
    np.minimum.at(mn, b, g)
    np.maximum.at(mx, b, g)
    for k in np.unique(b):
        s = b == k
        t = (sum(int(v) for v in fl[s]) << 32) + sum(int(v) for v in fr[s])
        lo[k], hi[k] = t & (2 ** 64 - 1), t >> 64
    cell = np.floor(x)
    F = np.rint((x - cell) * 2.0 ** bits).astype(np.int64)
    w = np.zeros(N + 1, np.int64)
    np.add.at(w, cell.astype(np.int64), 2 ** bits - F)
    np.add.at(w, cell.astype(np.int64) + 1, F)
    return cnt, lo, hi, mn, mx, w


# particles around a block's 1024 slots and a wave's 256; bins within, at and past the window's 256; cells past
# its 1024 nodes; order: sorted, shuffled, or all in one cell; gammas past 2^31 (summed one by one) and returning
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N,n,nb,load", [(2, 1, 1, "sorted"), (100, 255, 37, "sorted"), (1500, 1023, 256, "shuffled"),
                                         (5000, 1025, 257, "sorted"), (40000, 30001, 1000, "shuffled"),
                                         (300, 50000, 64, "sorted"), (64, 9000, 200, "one cell"),
                                         (700, 4097, 300, "fast")])
def test_profile_and_weights_exact(precision, N, n, nb, load):
    from paper_1011_6330_amd import Tube
    cfg = dict(synth.preset("c2"), n_cells=N, q_over_m=-1.0, ppc=max(n / N, 1.0), capacity=n + 5000, sort_every=0,
               precision=precision, gamma_fp64=20.0, max_bins=1024, flags=1)
    t = Tube(synth.tube_params(cfg))
    x, u = synth.random_particles(N, n, seed=n)
    if load == "one cell":
        x = 7.0 + (x - np.floor(x))
    elif load != "shuffled":
        x = np.sort(x)
    if load == "fast":
        u = u * np.where(np.arange(n) % 3 == 0, 1e9, 1.0)
    t.inject(x, u)
    d = t.diagnostics(n_bins=nb, weights=True, gauss=True)
    cnt, lo, hi, mn, mx, w = _expected(*t.read_particles(), N, nb, 32)
    for k, v in (("prof_count", cnt), ("prof_sum_lo", lo), ("prof_sum_hi", hi), ("prof_min", mn), ("prof_max", mx),
                 ("weights", w)):
        assert np.array_equal(d[k], v), k
    only = t.diagnostics(n_bins=nb)
    assert np.array_equal(only["prof_sum_lo"], lo) and np.array_equal(t.diagnostics(weights=True)["weights"], w)
    t.close()


# read-outs through the page-locked buffer (from a handle's second on) and array by array (its first, and what is
# past the buffer's 4 MiB): the same values
@pytest.mark.parametrize("N", [3, 1001, 120001, 600001])
def test_repeated_readouts_equal_the_first(N):
    from paper_1011_6330_amd import Tube
    n = 5000
    cfg = dict(synth.preset("c2"), n_cells=N, q_over_m=-1.0, ppc=max(n / N, 1e-3), capacity=n + 5000, sort_every=0, flags=1)
    t = Tube(synth.tube_params(cfg))
    t.inject(*synth.random_particles(N, n, seed=3))
    ask = dict(n_bins=77, fields=True, gauss=True, j=True, weights=True, rho=True)
    first, again = t.diagnostics(**ask), t.diagnostics(**ask)
    other = Tube(synth.tube_params(cfg))
    for d in (again, t.diagnostics(**ask)):
        assert d.keys() == first.keys()
        for k, v in first.items():
            assert np.array_equal(d[k], v), k
    other.close()
    t.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_bins_are_clear_for_each_readout(precision):
    """Read-outs of any number of bins after one another (each leaves the bins clear),
    with steps, weights and fields between them."""
    from paper_1011_6330_amd import Tube
    N, n = 900, 3000
    cfg = dict(synth.preset("c2"), n_cells=N, q_over_m=-1e-9, ppc=4.0, capacity=n + 100, sort_every=4,
               precision=precision, gamma_fp64=20.0, max_bins=1000, flags=3)
    t = Tube(synth.tube_params(cfg))
    t.inject(*synth.random_particles(N, n, seed=1))
    for nb, more in ((64, {}), (64, {}), (1000, {}), (1, dict(weights=True)), (0, {}), (37, dict(fields=False)), (999, {}),
                     (0, dict(gauss=True)), (64, dict(fields=False)), (1000, dict(gauss=True))):
        d = t.diagnostics(n_bins=nb, **more)
        if nb:
            exp = _expected(*t.read_particles(), N, nb, 32)
            for k, v in zip(("prof_count", "prof_sum_lo", "prof_sum_hi", "prof_min", "prof_max"), exp):
                assert np.array_equal(d[k], v), (nb, k)
        t.step(3)
    t.close()
