"""The autotuner's choices and cache, on a stand-in for the tube (whose push time depends
on the access and the size of its streams, as the card's does)."""
import json

import pytest

from paper_1011_6330_amd import GR_ALPHA, autotune


class FakeTube:
    def __init__(self, capacity, flags=0, precision=0, n=1000000):
        self.cfg = dict(capacity=capacity, flags=flags, precision=precision)
        self.n, self.tried, self.shape = n, [], None

    def diagnostics(self, fields=False):
        return dict(n_alive=self.n)

    def set_push_config(self, b, p, nt):
        self.shape = (b, p, nt)

    def step_timed(self, steps):
        self.tried.append(self.shape)
        b, p, nt = self.shape
        cached = 32 << 20 < self.cfg["capacity"] * (12 if self.cfg["precision"] else 16) <= 1 << 30
        return dict(push_ms=steps * (1.0 + (nt == cached) + abs(b - 128) / 1000 + p / 100), push_launches=steps)


@pytest.fixture
def cache(tmp_path):
    return str(tmp_path / "sub" / "tune.json")


def test_entry_of_an_older_version_is_not_read(cache, tmp_path):
    (tmp_path / "sub").mkdir()
    old = f"tube/{autotune._device_key()}/f64/{autotune._bucket(1000000)}"
    with open(cache, "w") as f:
        json.dump({old: [256, 2, True]}, f)
    t = FakeTube(30 << 20)
    assert autotune.tune_tube(t, cache_path=cache)[:3] == (128, 2, False) and t.tried
    again = FakeTube(30 << 20)
    assert autotune.tune_tube(again, cache_path=cache)[:3] == (128, 2, False) and not again.tried
    assert again.shape == (128, 2, False)


def test_access_kept_per_size_of_the_streams(cache):
    """The same particle count in tubes of three capacities: an entry each."""
    picks = [autotune.tune_tube(FakeTube(c), cache_path=cache)[2] for c in (1 << 20, 30 << 20, 100 << 20)]
    assert picks == [True, False, True]
    for c, nt in zip((1 << 20, 30 << 20, 100 << 20), picks):
        t = FakeTube(c)
        assert autotune.tune_tube(t, cache_path=cache)[2] is nt and not t.tried


def test_lapse_tubes_try_their_own_kernels_and_keep_their_own_entry(cache):
    t = FakeTube(30 << 20, flags=GR_ALPHA)
    autotune.tune_tube(t, cache_path=cache)
    assert sorted(t.tried) == [(128, 2, False), (128, 2, True)]
    flat = FakeTube(30 << 20)
    autotune.tune_tube(flat, cache_path=cache)
    assert len(flat.tried) == len(autotune.TUBE_SHAPES)
