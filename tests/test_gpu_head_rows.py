"""The LM head by number of rows: the register-streaming kernel (up to 16, 32
and 64 rows; at most 32 for vocabularies below 65,536) and the LDS-ring kernel
give a row the same bits, and the oracle's logits, for widths that are not
whole prefetch rounds and a vocabulary that is not whole tiles."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import OracleLM
from synth import SHAPES, make_weights
from tests.parity import compare

pytestmark = pytest.mark.gpu
ALLOWED = np.array([0, 5, 640, 1000], np.int32)


@pytest.mark.parametrize("d_model,vocab", [(64, 1001), (320, 1155), (512, 2048), (64, 65665),
                                           (320, 66001)])
def test_head_kernels_agree(d_model, vocab):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_31808_amd import lmop as L
    shape = dataclasses.replace(SHAPES["tiny"], n_layers=0, d_model=d_model, vocab=vocab)
    w = make_weights(shape, seed=9, n_layers=0)
    ctx = L.Context(shape, device=0)
    ctx.load_weights(w)
    toks = np.random.default_rng(d_model).integers(0, vocab, size=130).astype(np.int32)
    ref = OracleLM(w, shape).eval_rows(None, [toks[i:i + 1] for i in range(130)], 1, ALLOWED,
                                       keep_logits=True)
    full, full_logits = ctx.eval_rows(toks, np.arange(131), L.LMOP_ENUM, ALLOWED, no_dedup=True,
                                      debug_logits=True)
    compare(ref, full, full_logits, "130 rows")
    for n in (1, 15, 16, 17, 31, 32, 33, 63, 64, 65):
        print("head:", d_model, vocab, n, "rows", flush=True)
        out, logits = ctx.eval_rows(toks[:n], np.arange(n + 1), L.LMOP_ENUM, ALLOWED, no_dedup=True,
                                    debug_logits=True)
        assert np.array_equal(logits, full_logits[:n])
        for f in ("value", "logprob", "logprob_full", "tokens"):
            assert np.array_equal(out[f], full[f][:n]), (n, f)


@pytest.mark.parametrize("vocab", [131072, 131073, 150001])
def test_large_vocabularies(vocab):
    """The head finish holds the partials of up to 1,024 chunks (V = 131,072)
    in registers and walks longer lists twice: both give the log-probability
    of the logits, for the register-streaming head and the ring."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_31808_amd import lmop as L
    shape = dataclasses.replace(SHAPES["tiny"], n_layers=0, d_model=64, vocab=vocab)
    ctx = L.Context(shape, device=0)
    w = make_weights(shape, seed=9, n_layers=0)
    ctx.load_weights(w)
    toks = np.random.default_rng(vocab).integers(0, vocab, size=70).astype(np.int32)
    allowed = np.array([0, 5, 131071, vocab - 1 if vocab > 131072 else 640], np.int32)
    ref = OracleLM(w, shape).eval_rows(None, [toks[i:i + 1] for i in range(70)], 1, allowed,
                                       keep_logits=True)
    for n in (3, 70):
        print("vocabulary:", vocab, n, "rows", flush=True)
        out, logits = ctx.eval_rows(toks[:n], np.arange(n + 1), L.LMOP_ENUM, allowed, no_dedup=True,
                                    debug_logits=True)
        if n == 70:
            compare(ref, out, logits, f"V = {vocab}")
        z = logits[:, 0, :].astype(np.float64)
        # the sum over 1,025 and more chunks in fp32: a wave's 64 lanes add 17
        # to 19 chunks each, then 6 steps; each add errs by 2^-24 of the sum
        m = z.max(1, keepdims=True)
        lse = np.log(np.exp(z - m).sum(1)) + m[:, 0]
        assert np.allclose(out["logprob_full"], z[:, allowed].max(1) - lse, atol=2e-5)
    ctx.close()
