"""Device memory that runs out: the call reports it, and the context can be used again; or the call
does without."""
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


def test_a_prompt_whose_second_chunk_does_not_fit():
    """Chunks of 32 positions, whose buffers (2.1 MB of logits and n-gram distributions and 0.1 MB
    beside them a set) are limited to one set: the first chunk's tokens are in the models when the
    second finds no room.  The prompt's results are those of the same tokens one by one, and so are
    those of the tokens after it, of a prompt of one chunk and of one without any buffer."""
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    shape = dataclasses.replace(T, vocab=8200)
    ctx = nc.Context(nc.make_config(shape, warmup=20, max_streams=2),
                     synth.flat_weights(shape, synth.make_weights(shape, 5)))
    toks = synth.make_stream(150, shape.vocab, seed=3, span=(4, 32))
    ctx.chunk_bytes(3_000_000)
    ctx.reset(2, 200)
    done = 0
    for cut, memory in ((20, 0), (100, 1), (101, 1), (125, 1), (150, 2), (150, 2)):
        if cut == 150:
            ctx.chunk_bytes(1000)
        got, g = ctx.probs_for_context(0, toks[:cut], probe=True)
        for t in toks[done:cut]:
            ctx.mix_update(1, t)
        done = cut
        ref, r = ctx.probs_for_context(1, toks[:cut], probe=True)
        assert np.array_equal(got, ref), cut
        for k in ("mode", "mix_w", "entropy_bits", "pmax"):
            assert g[k] == r[k], (cut, k)
        assert ctx.fallbacks() == {"invalid": 0, "expired": 0, "memory": memory}, cut


@pytest.mark.parametrize("limit", [0, 1_000_000, 8_000_000])
def test_encode_whose_chunks_do_not_fit(limit):
    """No room for a chunk, none for its n-gram side, none for the second set (three streams of 150
    tokens take 6.6 MB a set): the same bytes, which decode, and chunks again once there is room."""
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    shape = dataclasses.replace(T, vocab=8200)
    ctx = nc.Context(nc.make_config(shape, warmup=20, max_streams=3),
                     synth.flat_weights(shape, synth.make_weights(shape, 5)))
    toks = [synth.make_stream(n, shape.vocab, seed=n, span=(4, 32)) for n in (150, 33, 70)]
    ref = ctx.encode_stream(toks)
    ctx.chunk_bytes(limit)
    assert ctx.encode_stream(toks) == ref
    assert ctx.fallbacks() == {"invalid": 0, "expired": 0, "memory": 1}
    back = ctx.decode_stream(ref[0], [150, 33, 70])
    assert all(np.array_equal(a, b) for a, b in zip(back, toks))
    ctx.chunk_bytes(1 << 40)
    assert ctx.encode_stream(toks) == ref
    assert ctx.fallbacks()["memory"] == 1


def test_a_calibration_that_does_not_fit():
    """Bfloat16 caches of 16,000 streams (2 x 84 GB) and then float32 ones beside them, which no card
    holds: the calibration fails, and a context calibrated before codes as it did."""
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    shape = dataclasses.replace(T, head_dim=64, n_heads=8, n_kv_heads=8, ctx_len=2048, slide=512)
    ctx = nc.Context(nc.make_config(shape, precision="fp8", use_ngram=False, skip="none",
                                    use_mixer=False, max_streams=16_000),
                     synth.flat_weights(shape, synth.make_weights(shape, 5)))
    toks = synth.make_stream(150, shape.vocab, seed=1, span=(4, 32))
    ctx.calibrate_fp8(toks)
    ref = ctx.encode_stream([toks])
    ctx.reset(16_000, 4)
    with pytest.raises(nc.NacrithError) as e:
        ctx.calibrate_fp8(toks[:100])
    assert e.value.status == 3
    assert ctx.encode_stream([toks]) == ref
    assert np.array_equal(ctx.decode_stream(ref[0], [150])[0], toks)
