"""Knot gradients from the node gradient (the hat weights' sums in node order) at the
edges of the runs of 2048 nodes that the kernel takes and for few and many knots: the
same bits as the sum in NumPy, node by node.  And gradients of runs whose last segments
the tape holds: one segment, two, three, a short last one, a second sweep."""
import numpy as np
import pytest

from paper_1011_6330_amd import synth

pytestmark = pytest.mark.gpu


def _tube(N, K, n=3000):
    from paper_1011_6330_amd import Tube
    cfg = dict(n_cells=N, length=10.0, radius=1.0, dt_over_dz=0.5, q_over_m=synth.q_over_m_for(0.9 * N / 10.0),
               ppc=n / N, rho_kind=2, rho_amp=1.0, kappa=0.15, r_star=10.0, knots=1.0 + 0.1 * np.arange(K) / K,
               capacity=3 * n + 4096, warm=n, sort_every=0)
    cfg["macro_charge"] = -(1.0 - cfg["kappa"]) * (cfg["length"] / N) / cfg["ppc"]
    x, u = synth.warm_start(cfg, seed=0)
    t = Tube(synth.tube_params(cfg))
    t.inject(x, u)
    return t, cfg


@pytest.mark.parametrize("N", [37, 2046, 2047, 2048, 4100])
@pytest.mark.parametrize("K", [2, 3, 64, 300])
def test_knot_sums_are_in_node_order(N, K):
    t, cfg = _tube(N, K)
    r = t.run_adjoint(12, 5)
    dz = cfg["length"] / N
    out = np.zeros(K)
    for i in range(N + 1):
        z = i * dz
        s = (z * float(K - 1)) / cfg["length"]
        kk = min(max(int(np.floor(s)), 0), K - 2)
        g = s - kk
        eta = 1.0 + z / cfg["r_star"]
        fd = 1.0 - cfg["kappa"] / (eta * eta * eta)
        out[kk] += r["g_rho"][i] * (-(1.0 - g) * fd)
        out[kk + 1] += r["g_rho"][i] * (-g * fd)
    assert np.abs(out).max() > 0
    assert np.array_equal(out, r["g_knots"])
    t.close()


@pytest.mark.parametrize("T,ckpt", [(6, 6), (6, 10), (12, 6), (13, 6), (18, 6), (40, 7), (5, 1), (1, 1), (2, 1)])
def test_held_segments_give_the_recomputed_gradient(T, ckpt):
    t, _ = _tube(128, 5)
    t.adjoint_forward(T, ckpt)
    a = t.backward()
    b = t.backward()
    whole, _ = _tube(128, 5)
    c = whole.run_adjoint(T, T)          # one segment
    for k in ("loss", "g_rate", "g_kappa"):
        assert a[k] == b[k] == c[k], k
    for k in ("g_rho", "g_knots"):
        assert np.array_equal(a[k], b[k]) and np.array_equal(a[k], c[k]), k
    # and the tube is where plain steps leave it
    plain, _ = _tube(128, 5)
    plain.step(T)
    t.step(3)
    plain.step(3)
    da, dp = t.diagnostics(j=True), plain.diagnostics(j=True)
    for k in ("ez", "er", "b_phi", "j_last", "n_alive", "n_injected"):
        assert np.array_equal(da[k], dp[k]), k
    for q in (t, whole, plain):
        q.close()
