"""State that outlives a chunk of known tokens: captured chains after buffers have moved."""
import dataclasses

import numpy as np
import pytest

import synth
from tests.nc_util import gpu_available

pytestmark = pytest.mark.gpu
T = synth.TINY


def _ctx(vocab=T.vocab, **kw):
    import paper_2602_19626_amd as nc
    shape = dataclasses.replace(T, vocab=vocab)
    return nc.Context(nc.make_config(shape, **kw),
                      synth.flat_weights(shape, synth.make_weights(shape, 5)))


def _streams(lens, vocab=T.vocab):
    return [synth.make_stream(n, vocab, seed=i, span=(4, 32)) if n else np.zeros(0, np.int32)
            for i, n in enumerate(lens)]


def test_captured_chains_follow_their_buffers():
    """A shape's chain is captured at its second use.  Between uses every chunk buffer grows, or only
    some do (a stream with an invalid distribution beside empty ones is coded step by step, which
    grows the logits alone: an infinite mixer rate makes the position after the first mixed one
    invalid): the bytes stay those of a fresh context."""
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    kw = dict(max_streams=40, warmup=60, skip="none", mix_eta=float("inf"))
    ctx = _ctx(**kw)
    small, wide, wider = _streams([33]), _streams([33] * 3), _streams([60] * 7)
    ref = [_ctx(**kw).encode_stream(s)[0] for s in (small, wide, wider)]
    with pytest.raises(nc.NacrithError) as e:
        ctx.encode_stream(_streams([70] + [0] * 39))
    assert e.value.status == 6
    for k in (0, 0, 0, 1, 0, 0, 2, 0, 0, 1, 1, 1, 0, 2, 2):
        assert ctx.encode_stream((small, wide, wider)[k])[0] == ref[k], k
    back = ctx.decode_stream(ref[2], [60] * 7)
    assert all(np.array_equal(a, b) for a, b in zip(back, wider))
