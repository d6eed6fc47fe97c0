"""Edges of the LDS-staged GEMM tiles: rows and columns past the last tile, K that ends inside a
64-wide part, odd and even part counts, every head dimension.  Every launch shape adds the same
per-part chains in the same order, so forcing each shape must leave the logits bit-identical to the
split kernel's."""
import dataclasses

import numpy as np
import pytest

import synth
from tests.nc_util import gpu_available

pytestmark = pytest.mark.gpu
GEMMS = ("qkv", "oproj", "gateup", "down", "lmhead")
BUCKETS = (1, 2, 4, 8, 16, 32, 48, 64, 96, 128, 192, 256)


@pytest.mark.parametrize("hd,heads,kv,d,ffn,prec", [
    (16, 4, 2, 64, 176, "fp32"),     # K = 64 and 176 (a part ends after 48 entries)
    (32, 3, 1, 80, 208, "bf16"),     # K = 80, 96, 208; N = 160
    (64, 3, 1, 144, 272, "fp32"),    # K = 144, 192, 272
    (64, 2, 2, 128, 320, "bf16"),    # K = 128 (2 parts), 320 (5 parts)
    (32, 4, 2, 192, 64, "fp8"),      # K = 192 (3 parts), 128, 64 (1 part)
])
def test_tile_edges_match_the_split_kernel(hd, heads, kv, d, ffn, prec):
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2602_19626_amd as nc
    shape = dataclasses.replace(synth.TINY, head_dim=hd, n_heads=heads, n_kv_heads=kv, d_model=d,
                                d_ffn=ffn, vocab=516)
    ctx = nc.Context(nc.make_config(shape, precision=prec),
                     synth.flat_weights(shape, synth.make_weights(shape, 11)))
    toks = synth.make_stream(150, shape.vocab, seed=4, span=(4, 32))
    if prec == "fp8":
        ctx.calibrate_fp8(toks)
    kinds = ["split", "tile_small", "tile_64"] + (
        ["wide_128"] if prec != "fp32" and hd > 16 else [])
    ref = None
    for kind in kinds:
        ctx.tiles_set([{"gemm": g, "max_rows": b, "kind": kind, "mb": 1, "waves": 3}
                       for g in GEMMS for b in BUCKETS])
        out = [np.frombuffer(ctx.encode_stream([toks])[0][0], dtype=np.uint8).astype(np.float32)]
        ctx.reset(1, 200)
        for n in (1, 33, 97, 128, 150):      # passes of 2, 32, 64, 31 and 22 rows
            p, pr = ctx.probs_for_context(0, toks[:n], probe=True)
            out += [p, pr["logits"]]
        out = np.concatenate(out)
        ref = out if ref is None else ref
        assert np.array_equal(out, ref), kind
