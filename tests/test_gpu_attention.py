"""Attention over groups of items: rows of a pass whose (query, head) columns fill one item, end
inside one, fill a group of four and run past it, at every head dimension, over windows that cross
chunks, quads and the ring's end.  Every kernel folds an item's chunks in the same order, so a
stream of many rows a pass must give the distributions of the same stream, one row a pass."""
import dataclasses

import numpy as np
import pytest

import synth
from tests.nc_util import gpu_available

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,heads,kv,prec", [(16, 4, 2, "bf16"), (32, 3, 1, "fp32"),
                                              (32, 2, 2, "bf16"), (64, 6, 2, "fp32"),
                                              (64, 9, 3, "bf16"), (64, 8, 1, "fp8")])
@pytest.mark.parametrize("ctx_len,slide", [(128, 32), (768, 256)])
def test_passes_of_many_rows_equal_single_rows(hd, heads, kv, prec, ctx_len, slide):
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    shape = dataclasses.replace(synth.TINY, head_dim=hd, n_heads=heads, n_kv_heads=kv,
                                ctx_len=ctx_len, slide=slide)
    ctx = nc.Context(nc.make_config(shape, precision=prec, skip="none", max_streams=2),
                     synth.flat_weights(shape, synth.make_weights(shape, 3)))
    n = ctx_len + 2 * slide + 75
    toks = synth.make_stream(n, shape.vocab, seed=9, span=(4, 32))
    if prec == "fp8":
        ctx.calibrate_fp8(toks)
    ctx.reset(2, n + 2)
    cuts = sorted({1, 6, 17, 22, 64, 65, 129, ctx_len - 1, ctx_len + slide + 5, n})
    done = 0
    for cut in cuts:
        got, g = ctx.probs_for_context(0, toks[:cut], probe=True)
        for t in toks[done:cut]:
            ctx.mix_update(1, t)
        done = cut
        ref, r = ctx.probs_for_context(1, toks[:cut], probe=True)
        assert np.array_equal(g["logits"], r["logits"]), cut
        assert np.array_equal(got, ref), cut


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_many_streams_of_uneven_rows(prec):
    """Enough items for one wave each (over 1,024) with groups of 1 to 4, beside the streams alone."""
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    shape = dataclasses.replace(synth.TINY, head_dim=64, n_heads=6, n_kv_heads=2, slide=64)
    w = synth.flat_weights(shape, synth.make_weights(shape, 3))
    streams = [synth.make_stream(3 + 5 * i, shape.vocab, seed=i, span=(4, 32)) for i in range(60)]
    ctx = nc.Context(nc.make_config(shape, precision=prec, max_streams=len(streams)), w)
    data, _ = ctx.encode_stream(streams)
    one = nc.Context(nc.make_config(shape, precision=prec), w)
    for i in (0, 1, 4, 9, 13, 30, 59):
        assert one.encode_stream([streams[i]])[0][0] == data[i], i
    back = ctx.decode_stream(data, [len(s) for s in streams])
    assert all(np.array_equal(a, b) for a, b in zip(back, streams))


@pytest.mark.parametrize("ctx_len,slide,heads", [(8, 8, 8), (12, 4, 8), (16, 16, 4), (32, 16, 4),
                                                 (24, 24, 8), (32, 32, 4)])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_contexts_shorter_than_a_chunk(ctx_len, slide, heads, prec):
    """Contexts whose ctx_len + slide is below the 64 keys of an attention chunk, or just there: streams
    of several items a group, one stream alone, one row a pass and the decoder agree, and the
    distributions are the oracle's (float32 against float64: 1e-5; BF16 passes only among themselves)."""
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    from oracle import pipeline as op
    shape = dataclasses.replace(synth.TINY, ctx_len=ctx_len, slide=slide, n_heads=heads)
    w = synth.make_weights(shape, 3)
    flat = synth.flat_weights(shape, w)
    n_streams = 9   # 36 items in 18 groups a pass (16 rows or 8, 2 or 4 query heads a kv head)
    toks = [synth.make_stream(5 * (ctx_len + slide) + 3 * i, shape.vocab, seed=i, span=(4, 32))
            for i in range(n_streams)]
    kw = dict(ngram_order=3, precision=prec, skip="none", mix_init="uniform", warmup=20)
    ctx = nc.Context(nc.make_config(shape, max_streams=n_streams, **kw), flat)
    data, _ = ctx.encode_stream(toks)
    back = ctx.decode_stream(data, [len(t) for t in toks])
    assert all(np.array_equal(a, b) for a, b in zip(back, toks))
    one = nc.Context(nc.make_config(shape, **kw), flat)
    assert [one.encode_stream([t])[0][0] for t in toks] == data
    t = toks[-1]
    pos = [0, 1, ctx_len - 1, ctx_len, ctx_len + slide + 1, len(t) - 1]
    ref = op.encode(op.Settings(vocab=shape.vocab, ngram_order=3, mix_init="uniform",
                                skip="none", use_skip=False, warmup=20), shape, w,
                    t, record=pos, block=1)
    one.reset(1, len(t) + 1)
    for i in sorted(pos):
        p = one.probs_for_context(0, t[:i])
        if prec == "fp32":
            assert np.max(np.abs(p - ref.records[i]["p"])) < 1e-5, i
