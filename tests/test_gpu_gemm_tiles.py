"""The GEMM's tile shapes: every shape the dispatch can pick (which launches
take which is checked on the host by test_gemm_tile_rule.py) gives a row the
same bits as any other shape does, and the oracle's logits."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import OracleLM
from synth import SHAPES, make_weights
from tests.parity import compare

pytestmark = pytest.mark.gpu

# d 512 and d_ff 1024 are whole stages of every tile shape; d_ff 688 (11
# panels of 64) only of the shapes with one panel per stage
SHAPE = dataclasses.replace(SHAPES["tiny"], name="tiles", n_layers=2, d_model=512, n_heads=8,
                            n_kv_heads=2, d_ff=1024, vocab=640)
LENS = [1, 16, 7, 40, 64, 100, 33, 128]
ALLOWED = np.array([3, 77, 400, 639], np.int32)


TOKENS = [1, 15, 16, 17, 64, 65, 129, 513, 1025, 2049, 4100, 8200, 16384]
MODELS = [("int4_g32", 1024), ("int4_g32", 688), ("fp8_e4m3", 1024)]
# widths and token counts whose launches take the shapes that SHAPE's do not
OTHER = [("int4_g32", (320, 4, 2, 64, 256), 1), ("int4_g32", (320, 4, 2, 64, 256), 33),
         ("int4_g32", (256, 8, 2, 128, 688), 100), ("fp8_e4m3", (320, 32, 8, 128, 688), 2049),
         ("fp8_e4m3", (256, 8, 8, 128, 256), 1300), ("fp8_e4m3", (256, 4, 2, 64, 14336), 513),
         ("fp8_e4m3", (3072, 4, 2, 64, 256), 1300), ("fp8_e4m3", (3072, 4, 2, 64, 256), 4100)]
ALONE = 23  # rows that also get a pass each


def _other(widths):
    d, heads, kv, hd, d_ff = widths
    return dataclasses.replace(SHAPE, d_model=d, n_heads=heads, n_kv_heads=kv, head_dim=hd,
                               d_ff=d_ff)


def _rows(tokens):
    """Row lengths that make one pass of exactly `tokens` tokens."""
    out, left, i = [], tokens, 0
    while left > 0:
        n = min(LENS[i % len(LENS)], left)
        out.append(n)
        left -= n
        i += 1
    return out


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_31808_amd import lmop
    return lmop


@pytest.fixture(scope="module", params=MODELS, ids=["int4", "int4-688", "fp8"])
def model(request, L):
    fmt, d_ff = request.param
    shape = dataclasses.replace(SHAPE, d_ff=d_ff)
    w = make_weights(shape, seed=31, fmt=fmt)
    ctx = L.Context(shape, device=0)
    ctx.load_weights(w)
    return w, shape, ctx


@pytest.mark.parametrize("tokens", TOKENS)
def test_tile_shapes_agree(model, L, tokens):
    _check(L, *model, tokens)


@pytest.mark.parametrize("fmt,widths,tokens", OTHER)
def test_other_widths_agree(L, fmt, widths, tokens):
    shape = _other(widths)
    w = make_weights(shape, seed=33, fmt=fmt)
    ctx = L.Context(shape, device=0)
    ctx.load_weights(w)
    _check(L, w, shape, ctx, tokens)
    ctx.close()


def _check(L, w, shape, ctx, tokens):
    rng = np.random.default_rng([5, tokens])
    lens = _rows(tokens)
    offs = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    toks = rng.integers(0, shape.vocab, size=tokens).astype(np.int32)

    def run(o, t, budget):
        print("tile shapes:", tokens, "tokens, budget", budget, flush=True)
        return ctx.eval_rows(t, o, L.LMOP_ENUM, ALLOWED, no_dedup=True, max_batch_tokens=budget,
                             debug_logits=len(o) <= 24)

    whole, logits = run(offs, toks, 1 << 15)  # one pass (2,048 rows at most)
    few = min(len(lens), ALONE)
    alone, _ = run(offs[:few + 1], toks[:offs[few]], 1)  # one pass per row
    for f in ("value", "logprob", "logprob_full"):
        assert np.array_equal(whole[f][:few], alone[f]), f
    if logits is not None:
        ref = OracleLM(w, shape).eval_rows(None, [toks[offs[i]:offs[i + 1]] for i in range(few)],
                                           1, ALLOWED, keep_logits=True)
        compare(ref, whole, logits, f"{tokens} tokens")


@pytest.mark.parametrize("fmt", ["int4_g32", "fp8_e4m3"])
@pytest.mark.parametrize("tokens", [1, 9, 16, 17, 40])
def test_few_tokens_long_k(L, fmt, tokens):
    """Few tokens over a K loop longer than every ring (128 panels of the down
    projection): the loaders, converters and consumers of the split kernel
    wrap their rings, and a row's bits are those of a large batch."""
    shape = dataclasses.replace(SHAPE, d_model=1024, d_ff=8192, vocab=512)
    w = make_weights(shape, seed=32, fmt=fmt)
    ctx = L.Context(shape, device=0)
    ctx.load_weights(w)
    rng = np.random.default_rng([6, tokens])
    toks = rng.integers(0, shape.vocab, size=tokens + 300).astype(np.int32)
    allowed = np.array([3, 77, 400, 511], np.int32)
    print("long K:", fmt, tokens, "tokens", flush=True)
    few, logits = ctx.eval_rows(toks[:tokens], np.array([0, tokens]), L.LMOP_ENUM, allowed,
                                debug_logits=True)
    ref = OracleLM(w, shape).eval_rows(None, [toks[:tokens]], 1, allowed, keep_logits=True)
    compare(ref, few, logits, f"{tokens} tokens")
    many, many_logits = ctx.eval_rows(toks, np.array([0, tokens, tokens + 300]), L.LMOP_ENUM,
                                      allowed, debug_logits=True)
    assert np.array_equal(logits[0], many_logits[0])
    assert few["logprob_full"][0] == many["logprob_full"][0]
    ctx.close()
