"""The pool of tube and batch streams: its bookkeeping, on stand-ins for torch's streams
(32 underlying ones handed out in turn)."""
import itertools
import threading

import pytest

from paper_1011_6330_amd import _binding


class FakeStream:
    def __init__(self, handle):
        self.cuda_stream = handle


@pytest.fixture
def pool():
    """(pool, make): torch's rotation over 32 handles."""
    turn = itertools.count()
    return _binding._StreamPool(), lambda: FakeStream(1000 + next(turn) % 32)


def test_reused_last_first_and_once(pool):
    p, make = pool
    ka, a = p.take(0, make)
    kb, b = p.take(0, make)
    assert a.cuda_stream != b.cuda_stream
    p.release(ka)
    p.release(kb)
    assert p.take(0, make)[1] is b and p.take(0, make)[1] is a
    assert p.take(0, make)[1].cuda_stream not in (a.cuda_stream, b.cuda_stream)


def test_stream_in_use_by_another_is_not_handed_out(pool):
    """b works on a's stream; a closes; c must not get it, nor anyone after b (it is the caller's now)."""
    p, make = pool
    ka, a = p.take(0, make)
    kb, b = p.use(0, a)
    p.release(ka)
    kc, c = p.take(0, make)
    assert c.cuda_stream != a.cuda_stream
    p.release(kb)
    assert all(p.take(0, make)[1].cuda_stream != a.cuda_stream for _ in range(30))


def test_given_stream_equal_to_an_idle_one(pool):
    p, make = pool
    ka, a = p.take(0, make)
    p.release(ka)
    own = FakeStream(a.cuda_stream)
    kb, _ = p.use(0, own)
    assert p.take(0, make)[1].cuda_stream != own.cuda_stream
    p.release(kb)
    assert p.take(0, make)[1].cuda_stream != own.cuda_stream


def test_new_streams_avoid_those_in_use(pool):
    """torch's rotation comes round to a stream that is still open: the next one is taken."""
    p, make = pool
    held = p.use(0, FakeStream(1005))[0]
    got = [p.take(0, make)[1].cuda_stream for _ in range(31)]
    assert len(set(got)) == 31 and 1005 not in got
    p.release(held)


def test_more_than_32_open_closed_interleaved(pool):
    """70 open tubes share 32 streams; whatever the order of closing, each stream is idle at
    most once, and 32 tubes opened afterwards have 32 streams."""
    p, make = pool
    keys = [p.take(0, make)[0] for _ in range(70)]
    for k in keys[::3] + keys[1::3] + keys[2::3]:
        p.release(k)
    assert len({p.take(0, make)[1].cuda_stream for _ in range(32)}) == 32


def test_devices_apart(pool):
    p, make = pool
    k0, s0 = p.take(0, make)
    p.release(k0)
    k1, s1 = p.take(1, make)
    assert s1 is not s0
    assert p.take(0, make)[1] is s0


def test_threads(pool):
    """Eight threads open and close; no two open tubes ever share a stream."""
    p, make = pool
    lock, live, bad = threading.Lock(), set(), []

    def work():
        for _ in range(300):
            key, s = p.take(0, make)
            with lock:
                if s.cuda_stream in live:
                    bad.append(s.cuda_stream)
                live.add(s.cuda_stream)
            with lock:
                live.discard(s.cuda_stream)
            p.release(key)

    ts = [threading.Thread(target=work) for _ in range(8)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
