"""State that outlives a chunk of known tokens (captured chains after buffers have moved), and the way
back to single steps where a call's chunks cannot be used: counted, and with the step path's bits."""
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


def test_captured_decode_passes_follow_their_buffers():
    """Decode passes are captured with the addresses and the layer stride of the caches, which move when
    a later call has more streams or longer ones: the tokens stay those of direct launches."""
    if not gpu_available():
        pytest.skip("no GPU")
    sets = [_streams(lens) for lens in ([40], [40, 25], [90], [40] * 7, [300, 40], [40], [40, 25])]
    ref = _ctx(max_streams=7, warmup=20)
    ctx = _ctx(max_streams=7, warmup=20, decode_graphs=True)
    for toks in sets:
        data, _ = ref.encode_stream(toks)
        for _ in range(2):
            back = ctx.decode_stream(data, [len(t) for t in toks])
            assert all(np.array_equal(a, b) for a, b in zip(back, toks))
    assert ctx.stats()["graph_replays"] > 0


NONE = {"invalid": 0, "expired": 0}


def _counts(ctx):
    f = ctx.fallbacks()
    return {k: f[k] for k in NONE}


def _same_as_steps(ctx, toks, cuts, mark=lambda cut: None):
    """Stream 0 takes toks in the pieces that end at cuts, stream 1 token by token: equal
    distributions and diagnostics at every cut (NaN where both are)."""
    done = 0
    for cut in cuts:
        mark(cut)
        got, g = ctx.probs_for_context(0, toks[:cut], probe=True)
        for t in toks[done:cut]:
            ctx.mix_update(1, t)
        done = cut
        ref, r = ctx.probs_for_context(1, toks[:cut], probe=True)
        np.testing.assert_array_equal(got, ref, err_msg=str(cut))
        for k in ("mode", "mix_w", "entropy_bits", "pmax", "p_ngram", "cdf"):
            np.testing.assert_array_equal(g[k], r[k], err_msg=f"{cut} {k}")


def test_valid_calls_stay_with_chunks():
    """Chains in one launch (1 and 3 segments), chains of a launch per position (40 rows of 17
    segments) and prompts in pieces: no call goes back to steps."""
    if not gpu_available():
        pytest.skip("no GPU")
    for vocab, lens in ((512, [150]), (8200, [150, 33, 70]), (16385 * 4, [20 + k for k in range(40)])):
        ctx = _ctx(vocab, warmup=20, max_streams=len(lens))
        toks = _streams(lens, vocab)
        data, _ = ctx.encode_stream(toks)
        back = ctx.decode_stream(data, lens)
        assert all(np.array_equal(a, b) for a, b in zip(back, toks))
        assert _counts(ctx) == NONE, vocab
    ctx = _ctx(8200, warmup=20, max_streams=2)
    ctx.reset(2, 200)
    _same_as_steps(ctx, _streams([160], 8200)[0], (1, 40, 150, 160))
    assert _counts(ctx) == NONE


def test_two_contexts_at_once_stay_with_chunks():
    """Two contexts, each near the largest chain in one launch, at work from two threads."""
    if not gpu_available():
        pytest.skip("no GPU")
    import threading
    toks = _streams([200 + i for i in range(21)], 49152)
    ctxs = [_ctx(49152, max_streams=len(toks)) for _ in range(2)]
    ref = ctxs[0].encode_stream(toks)[0]
    out = [None, None]

    def code(k):
        out[k] = [ctxs[k].encode_stream(toks)[0] for _ in range(3)]

    threads = [threading.Thread(target=code, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(r == ref for k in range(2) for r in out[k])
    assert [_counts(c) for c in ctxs] == [NONE, NONE]


def test_waits_that_give_up():
    """No polls: a word that is not there at the first look ends its wait.  Encode and prompts (the
    second after a committed prefix, which is committed again) give the step path's results."""
    if not gpu_available():
        pytest.skip("no GPU")
    toks = _streams([150, 33, 70], 8200)
    ctx = _ctx(8200, warmup=20, max_streams=3)
    ref = ctx.encode_stream(toks)[0]
    assert _counts(ctx) == NONE
    ctx.chunk_polls(0)
    assert ctx.encode_stream(toks)[0] == ref
    assert _counts(ctx) == {"invalid": 0, "expired": 1}
    ctx.chunk_polls(1 << 31)   # (at most the default)
    assert ctx.encode_stream(toks)[0] == ref
    assert _counts(ctx) == {"invalid": 0, "expired": 1}
    ctx.reset(2, 200)
    _same_as_steps(ctx, toks[0], (40, 150), lambda cut: ctx.chunk_polls(0 if cut == 150 else 1 << 18))
    assert _counts(ctx) == {"invalid": 0, "expired": 2}


def test_an_invalid_distribution_after_a_committed_prefix():
    """The mixer starts at position 60 with an infinite rate, so position 61 and those after it have
    no distribution: pieces before, at and past it against token by token, then encode, which refuses
    the stream and takes a shorter one."""
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    toks = _streams([110])[0]
    ctx = _ctx(max_streams=2, warmup=60, skip="none", mix_eta=float("inf"))
    ctx.reset(2, 200)
    _same_as_steps(ctx, toks, (33, 60, 61))
    assert _counts(ctx) == NONE
    ctx.reset(2, 200)
    _same_as_steps(ctx, toks, (33, 80, 110))
    assert _counts(ctx)["invalid"] == 2 and _counts(ctx)["expired"] == 0
    with pytest.raises(nc.NacrithError) as e:
        ctx.encode_stream([toks])
    assert e.value.status == 6 and _counts(ctx)["invalid"] == 3
    data, _ = ctx.encode_stream([toks[:60]])
    assert np.array_equal(ctx.decode_stream(data, [60])[0], toks[:60])
    assert _counts(ctx) == {"invalid": 3, "expired": 0}


def test_nan_weights_are_counted_as_invalid():
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    w = synth.flat_weights(T, synth.make_weights(T, 5))
    w[:T.d_model] = np.nan
    for toks in (_streams([50])[0], np.zeros(1, np.int32)):
        ctx = nc.Context(nc.make_config(T), w)
        with pytest.raises(nc.NacrithError) as e:
            ctx.encode_stream([toks])
        assert e.value.status == 6 and _counts(ctx) == {"invalid": 1, "expired": 0}
