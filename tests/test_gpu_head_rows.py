"""The LM head by number of rows: the register-streaming kernel (up to 16, 32
and 64 rows) and the LDS-ring kernel give a row the same bits, and the
oracle's logits, for widths that are not whole prefetch rounds and a
vocabulary that is not whole tiles."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import OracleLM
from synth import SHAPES, make_weights
from tests.parity import compare

pytestmark = pytest.mark.gpu
ALLOWED = np.array([0, 5, 640, 1000], np.int32)


@pytest.mark.parametrize("d_model,vocab", [(64, 1001), (320, 1155), (512, 2048)])
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
