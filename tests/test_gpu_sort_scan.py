"""The scan of the sort keys in its three forms -- the counts before a block summed by
the block itself (up to 8 blocks of 1024 keys), block totals summed (up to 8192
blocks), block totals scanned -- at the edges between them: a tube that sorts holds
the same particles and fields, bit for bit, as one that never sorts, in the order of
its keys, over several sorts (each leaves the key counts clear for the next)."""
import numpy as np
import pytest

from paper_1011_6330_amd import synth

pytestmark = pytest.mark.gpu

FROZEN = 3   # no injection, frozen fields


def _particles(N, n, seed):
    """Momenta a good way from the stream threshold and next to no kick (q_over_m below),
    so that no particle changes its stream, which would round its momentum."""
    z, u = synth.random_particles(N, n, seed=seed)
    keep = np.abs(np.abs(u) - np.sqrt(63.0)) > 0.5
    return z[keep], u[keep]


def _state(t):
    d = t.diagnostics(n_bins=16, fields=True, j=True, raise_on_status=False)
    x, u = t.read_particles()
    k = np.lexsort((u, x))
    return dict(d, x=x[k], u=u[k]), x, u


def _ordered(x, u, f32, gamma, what):
    g = np.sqrt(1.0 + u * u) >= gamma if f32 else np.zeros(x.size, bool)
    n_lo = int(x.size - g.sum())
    assert not g[:n_lo].any(), f"{what}: streams mixed"
    for part in (x[:n_lo], x[n_lo:]):
        assert (np.diff(np.floor(part)) >= 0).all(), f"{what}: not in key order"


def _check(sorted_tubes, plain_tubes, step, f32, gamma):
    for M in (4, 4, 1, 3, 8):
        step(M)
        for k, (a, b) in enumerate(zip(sorted_tubes, plain_tubes)):
            sa, x, u = _state(a)
            sb, _, _ = _state(b)
            for key, v in sb.items():
                if key == "n_slots":      # a sort drops the removed slots
                    assert M == 1 or sa[key] == x.size
                    continue
                if key == "n_slots_high":
                    assert M == 1 or sa[key] == (f32 and (np.sqrt(1.0 + u * u) >= gamma).sum())
                    continue
                assert np.array_equal(v, sa[key], equal_nan=True), f"tube {k} after {M} steps: {key} differs"
            if M != 1:
                _ordered(x, u, f32, gamma, f"tube {k} after {M} steps")


def _cfg(N, n, precision, sort_every):
    return dict(synth.preset("c1"), n_cells=N, length=0.01 * N, precision=precision, gamma_fp64=8.0, flags=FROZEN,
                q_over_m=-1e-9, ppc=4.0, capacity=n + 4096, sort_every=sort_every)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("blocks", [1, 8, 8192])
@pytest.mark.parametrize("over", [0, 1])
def test_sorts_of_one_tube(precision, blocks, over):
    from paper_1011_6330_amd import Tube
    keys = 1024 * blocks + over
    N = keys if precision == 0 else (keys + 1) // 2 - 1
    n = 5000
    ts = [Tube(synth.tube_params(_cfg(N, n, precision, s))) for s in (4, 0)]
    for t in ts:
        t.inject(*_particles(N, n, blocks))
    _check(ts[:1], ts[1:], lambda M: [t.step(M) for t in ts], precision == 1, 8.0)
    for t in ts:
        t.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("sizes", [(2, 1024, 8192), (1025, 8193, 700, 40000), (8193 * 1024, 5, 9000)])
def test_sorts_of_a_batch(precision, sizes):
    from paper_1011_6330_amd import Batch
    bs = [Batch([synth.tube_params(_cfg(N, 3000, precision, s)) for N in sizes]) for s in (4, 0)]
    for b in bs:
        for t, N in zip(b.tubes, sizes):
            t.inject(*_particles(N, 3000, N))
    _check(bs[0].tubes, bs[1].tubes, lambda M: [b.step(M) for b in bs], precision == 1, 8.0)
    for b in bs:
        b.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_cells,capacity", [(8192, 100), (8193, 1024), (70001, 1025), (300000, 900)])
def test_more_keys_than_the_slots_blocks_clear(n_cells, capacity, precision):
    """Tubes of many keys and few slots, whose scatter has blocks that only clear counts: alone
    and in a batch, against a tube that never sorts."""
    from paper_1011_6330_amd import Batch, Tube
    cfg = dict(synth.preset("c1"), n_cells=n_cells, length=1e-3 * n_cells, ppc=1e-3, capacity=capacity, flags=1,
               precision=precision, gamma_fp64=8.0)
    x, u = synth.random_particles(n_cells, min(capacity, 80), seed=9)
    plain, alone = Tube(synth.tube_params(cfg)), Tube(synth.tube_params(dict(cfg, sort_every=2)))
    b = Batch([synth.tube_params(dict(cfg, sort_every=2)), synth.tube_params(dict(cfg, sort_every=2, n_cells=50))])
    for t in (plain, alone, b.tubes[0]):
        t.inject(x, u)
    for h in (plain, alone, b):
        h.step(9)

    def state(t):
        d = t.diagnostics(n_bins=8, fields=True, j=True)
        px, pu = t.read_particles()
        k = np.lexsort((pu, px))
        return [d["ez"], d["er"], d["b_phi"], d["j_last"], d["prof_count"], px[k], pu[k]]

    want = state(plain)
    for t in (alone, b.tubes[0]):
        for a, c in zip(want, state(t)):
            assert np.array_equal(a, c)
    for h in (plain, alone, b):
        h.close()
