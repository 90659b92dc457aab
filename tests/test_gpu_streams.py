"""Streams of tubes and batches: an open one has its own, a closed one's serves the next,
a caller's stays the caller's; the results do not depend on which."""
import numpy as np
import pytest

from paper_1011_6330_amd import synth

pytestmark = pytest.mark.gpu


def test_streams_are_reused_after_close():
    import torch
    from paper_1011_6330_amd import Batch, Tube
    p = synth.tube_params(dict(synth.preset("c1"), sort_every=8))

    def run(**kw):
        t = Tube(p, **kw)
        t.step(100)
        d = t.diagnostics(j=True)
        return t, d

    a, da = run()
    b, db = run()
    assert a.stream.cuda_stream != b.stream.cuda_stream
    first = a.stream.cuda_stream
    a.close()
    a.close()                                  # once only
    own = torch.cuda.Stream()
    c, dc = run(stream=own)
    assert c.stream is own
    c.close()
    e, de = run()
    assert e.stream.cuda_stream == first
    f = Batch([p, p])
    assert f.stream.cuda_stream not in (first, b.stream.cuda_stream, own.cuda_stream)
    f.step(100)
    df = f.tubes[1].diagnostics(j=True)
    for d in (db, dc, de, df):
        for k in ("ez", "er", "b_phi", "j_last"):
            assert np.array_equal(d[k], da[k]), k
    for t in (b, e, f):
        t.close()
