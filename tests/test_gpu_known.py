"""Chunks of known tokens (encode, committed prompts) against the step path (one coding step per
committed token): the same bits."""
import dataclasses

import numpy as np
import pytest

import synth
from tests.nc_util import gpu_available

pytestmark = pytest.mark.gpu
T = synth.TINY


@pytest.mark.parametrize("vocab,order,skip,prec", [(512, 1, "pmax", "fp32"), (512, 3, "none", "bf16"),
                                                   (4100, 4, "entropy", "fp32"),
                                                   (8192, 2, "entropy", "bf16")])
def test_prompt_in_pieces_equals_token_by_token(vocab, order, skip, prec):
    """A prompt committed in pieces that end inside, at and past the slide, the four-position runs of
    the dense n-gram kernel and single tokens, and the same tokens committed one at a time: equal
    distributions, diagnostics and mixer weights; full contexts evict alike (64 slots)."""
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    shape = dataclasses.replace(T, vocab=vocab)
    w = synth.flat_weights(shape, synth.make_weights(shape, 5))
    cfg = nc.make_config(shape, ngram_order=order, skip=skip, precision=prec, warmup=20,
                         max_streams=2)
    ctx = nc.Context(cfg, w)
    n = T.ctx_len + T.slide + 60
    toks = synth.make_stream(n, vocab, seed=7, span=(4, 32))
    toks[40:40 + 2 * 70:2] = 3                      # context (3,) meets over 64 continuations
    toks[41:41 + 2 * 70:2] = 100 + np.arange(70)
    ctx.reset(2, n + 2)
    done = 0
    for cut in (1, 5, 6, 31, 32, 33, 36, 68, 101, n):
        got, g = ctx.probs_for_context(0, toks[:cut], probe=True)
        for t in toks[done:cut]:
            ctx.mix_update(1, t)
        done = cut
        ref, r = ctx.probs_for_context(1, toks[:cut], probe=True)
        assert np.array_equal(got, ref), cut
        assert g["mode"] == r["mode"] and g["mix_w"] == r["mix_w"], cut
        assert g["entropy_bits"] == r["entropy_bits"] and g["pmax"] == r["pmax"], cut
        for k in ("logits", "ptilde", "p_ngram", "cdf"):
            if r["llm_ran"] or k in ("p_ngram", "cdf"):
                assert np.array_equal(g[k], r[k]), (cut, k)


def test_invalid_distributions_are_refused_like_step_by_step():
    """NaN weights: every distribution is invalid, the chunk path hands over to single steps, and
    encode refuses the stream."""
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    w = synth.flat_weights(T, synth.make_weights(T, 5))
    w[:T.d_model] = np.nan
    ctx = nc.Context(nc.make_config(T), w)
    with pytest.raises(nc.NacrithError) as e:
        ctx.encode_stream([synth.make_stream(50, T.vocab, seed=1)])
    assert e.value.status == 6


@pytest.mark.parametrize("vocab,streams,prec", [(8200, 1, "bf16"), (4100, 7, "fp32"),
                                                (12292, 40, "bf16"), (16385 * 4, 40, "fp32")])
def test_one_launch_chains_equal_streams_alone(vocab, streams, prec):
    """Chains of 1 to 17 segments a row, rows that end inside a chunk, and row counts on both sides of
    the one-launch rule (40 rows of 17 segments are past it): the bytes of each stream alone, whose
    tokens decode (a step per token) gives back."""
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    shape = dataclasses.replace(T, vocab=vocab)
    w = synth.flat_weights(shape, synth.make_weights(shape, 5))
    toks = [synth.make_stream(1 + (37 * i + 70) % 150, vocab, seed=i, span=(4, 32))
            for i in range(streams)]
    ctx = nc.Context(nc.make_config(shape, precision=prec, warmup=20, max_streams=streams), w)
    data, _ = ctx.encode_stream(toks)
    back = ctx.decode_stream(data, [len(t) for t in toks])
    assert all(np.array_equal(a, b) for a, b in zip(back, toks))
    one = nc.Context(nc.make_config(shape, precision=prec, warmup=20), w)
    for i in range(0, streams, 6):
        assert one.encode_stream([toks[i]])[0][0] == data[i], i


def test_two_contexts_at_once():
    """Chains of two contexts, each near the one-launch limit, run at the same time from two threads:
    the bytes of either alone."""
    if not gpu_available():
        pytest.skip("no GPU")
    import threading

    import paper_2602_19626_amd as nc
    shape = dataclasses.replace(T, vocab=49152)
    w = synth.flat_weights(shape, synth.make_weights(shape, 5))
    toks = [synth.make_stream(200 + i, shape.vocab, seed=i, span=(4, 32)) for i in range(21)]
    ctxs = [nc.Context(nc.make_config(shape, max_streams=len(toks)), w) for _ in range(2)]
    ref = ctxs[0].encode_stream(toks)[0]
    out = [None, None]

    def code(k):
        out[k] = [ctxs[k].encode_stream(toks)[0] for _ in range(3)]

    threads = [threading.Thread(target=code, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in range(2):
        assert all(r == ref for r in out[k]), k
