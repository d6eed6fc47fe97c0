"""Device memory that runs out: the call reports it, and the context can be used again."""
import dataclasses

import numpy as np
import pytest

import synth
from tests.nc_util import gpu_available

pytestmark = pytest.mark.gpu
T = synth.TINY


def test_a_reset_that_does_not_fit():
    """Key and value caches of 40,000 streams (over 400 GB in one allocation, which no card holds): the
    reset fails, no stream can be used until the next one, and that gives the same results as before."""
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    shape = dataclasses.replace(T, head_dim=64, n_heads=8, n_kv_heads=8, ctx_len=2048, slide=512)
    ctx = nc.Context(nc.make_config(shape, max_streams=40_000),
                     synth.flat_weights(shape, synth.make_weights(shape, 5)))
    toks = synth.make_stream(150, shape.vocab, seed=1, span=(4, 32))
    ref = ctx.encode_stream([toks])
    ctx.reset(1, 200)
    p = ctx.probs_for_context(0, toks[:40])
    with pytest.raises(nc.NacrithError) as e:
        ctx.reset(40_000, 4)
    assert e.value.status == 3
    with pytest.raises(nc.NacrithError) as e:
        ctx.probs_for_context(0, toks[:40])
    assert e.value.status == 6
    ctx.reset(1, 200)
    assert np.array_equal(ctx.probs_for_context(0, toks[:40]), p)
    assert ctx.encode_stream([toks]) == ref
    assert np.array_equal(ctx.decode_stream(ref[0], [150])[0], toks)
