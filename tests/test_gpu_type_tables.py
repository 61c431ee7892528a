"""The tables of an output type: the token index built on the device for every
size of the allowed list, and an automaton whose state masks are too large for
the staging slot."""
import dataclasses

import numpy as np
import pytest
import torch

from synth import SHAPES, make_weights, option_trie

pytestmark = pytest.mark.gpu
TINY = SHAPES["tiny"]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_31808_amd import lmop as L
    c = L.Context(TINY, device=0)
    c.load_weights(make_weights(TINY, seed=1234))
    return c


def _rows(n=6):
    rng = np.random.default_rng(3)
    lens = rng.integers(1, 20, size=n)
    offs = np.concatenate([[0], np.cumsum(lens)])
    return rng.integers(0, TINY.vocab, size=int(offs[-1])).astype(np.int32), offs


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 2048])
def test_allowed_list_sizes(ctx, n):
    toks, offs = _rows()
    allowed = np.random.default_rng(n).permutation(TINY.vocab)[:n].astype(np.int32)
    out, logits = ctx.eval_rows(toks, offs, 1, allowed, debug_logits=True)
    z = logits[:, 0, :].astype(np.float64)
    za = z[:, allowed]
    assert np.array_equal(out["value"], za.argmax(1))
    best = za.max(1)
    # fp32 log-sum-exp of at most 2,048 terms
    lse = lambda x: np.log(np.exp(x - x.max(1, keepdims=True)).sum(1)) + x.max(1)
    assert np.allclose(out["logprob"], best - lse(za), atol=1e-5)
    assert np.allclose(out["logprob_full"], best - lse(z), atol=1e-5)


@pytest.mark.parametrize("pad", [0, 60000])
def test_large_state_masks(ctx, pad):
    """60,000 states that no edge leads to (masks of 1.4 MB, not staged) change nothing."""
    rng = np.random.default_rng(8)
    ids = rng.permutation(TINY.vocab)[:24].tolist()
    options = [(ids[i % 8], ids[8 + i]) for i in range(16)]
    aut, _ = option_trie(options)
    big = dataclasses.replace(
        aut, n_states=aut.n_states + pad,
        edge_offset=np.concatenate([aut.edge_offset, np.full(pad, aut.edge_offset[-1], np.int32)]),
        accepting=np.concatenate([aut.accepting, np.ones(pad, np.uint8)]))
    toks, offs = _rows()
    a, _ = ctx.eval_rows(toks, offs, 3, aut, max_tokens=2)
    b, _ = ctx.eval_rows(toks, offs, 3, big, max_tokens=2)
    for f in ("value", "tokens", "logprob", "logprob_full"):
        assert np.array_equal(a[f], b[f]), f
