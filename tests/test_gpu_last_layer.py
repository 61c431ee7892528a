"""The last layer: a pass that computes Q and attention for the rows' last
tokens only gives every row the bits of a pass that computes them for all
tokens, and the oracle's logits; Q widths that are not whole 256-column tiles,
both head sizes and weight formats, rows without tokens, long own texts."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import OracleLM
from synth import SHAPES, make_weights
from tests.parity import compare

pytestmark = pytest.mark.gpu
ALLOWED = np.array([3, 77, 400, 639], np.int32)


@pytest.mark.parametrize("heads,kv_heads,head_dim,fmt", [
    (4, 2, 64, "int4_g32"), (5, 1, 64, "int4_g32"), (3, 3, 128, "fp8_e4m3"), (18, 1, 64, "int4_g32"),
    (8, 2, 128, "int4_g32")])
@pytest.mark.parametrize("lens", [(1, 200, 150, 31), (0, 300, 63, 64, 65, 2), (700,), (1, 1, 259)])
def test_last_tokens_only(heads, kv_heads, head_dim, fmt, lens):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_31808_amd import lmop as L
    shape = dataclasses.replace(SHAPES["tiny"], name="last", n_heads=heads, n_kv_heads=kv_heads,
                                head_dim=head_dim, d_ff=320, vocab=640)
    w = make_weights(shape, seed=heads, fmt=fmt)
    ctx = L.Context(shape, device=0)
    ctx.load_weights(w)
    rng = np.random.default_rng([heads, len(lens)])
    prefix = rng.integers(0, shape.vocab, size=33).astype(np.int32)
    # rows of a few tokens each beside them: the pass alone decides, not a row
    lens = list(lens) + [4] * 12
    rows = [rng.integers(0, shape.vocab, size=n).astype(np.int32) for n in lens]
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    pre = ctx.set_prefix(prefix)
    out = {}
    for budget in (4096, 1):  # one pass, which saves over 256 tokens; a pass per row
        print("last layer:", heads, kv_heads, head_dim, fmt, lens, budget, flush=True)
        out[budget] = ctx.eval_rows(np.concatenate(rows), offs, L.LMOP_ENUM, ALLOWED, prefix=pre,
                                    no_dedup=True, debug_logits=True, max_batch_tokens=budget)
    ref = OracleLM(w, shape).eval_rows(prefix, rows, 1, ALLOWED, keep_logits=True)
    compare(ref, *out[4096], "one pass")
    # short rows by themselves stay below the split; the long ones are split in both
    assert np.array_equal(out[4096][1], out[1][1])
    assert out[4096][0].tobytes() == out[1][0].tobytes()
    ctx.release_prefix(pre)
    ctx.close()


@pytest.mark.parametrize("d_ff,launches", [(64, 2), (128, 3)])
def test_narrow_mlp(d_ff, launches):
    """130 rows of 3 tokens save over 256 queries; with d_ff 64 the MLP's
    buffer cannot hold their 130 x 256 normalised values, so the pass takes the
    whole projection (one QKV launch per layer, no further one)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_31808_amd import lmop as L
    shape = dataclasses.replace(SHAPES["tiny"], name="narrow", n_layers=2, d_ff=d_ff, vocab=640)
    w = make_weights(shape, seed=d_ff)
    ctx = L.Context(shape, device=0)
    ctx.load_weights(w)
    rng = np.random.default_rng(d_ff)
    rows = [rng.integers(0, shape.vocab, size=3).astype(np.int32) for _ in range(130)]
    offs = np.arange(0, 391, 3).astype(np.int64)
    print("narrow MLP:", d_ff, flush=True)
    ctx.set_profiling(1)
    whole = ctx.eval_rows(np.concatenate(rows), offs, L.LMOP_ENUM, ALLOWED, no_dedup=True,
                          debug_logits=True)
    assert ctx.kernel_stats()["gemm_w4a16_qkv"]["launches"] == launches
    ctx.set_profiling(0)
    alone = ctx.eval_rows(np.concatenate(rows), offs, L.LMOP_ENUM, ALLOWED, no_dedup=True,
                          debug_logits=True, max_batch_tokens=1)
    assert np.array_equal(whole[1], alone[1])
    assert whole[0].tobytes() == alone[0].tobytes()
    ref = OracleLM(w, shape).eval_rows(None, rows, 1, ALLOWED, keep_logits=True)
    compare(ref, *whole, f"d_ff {d_ff}")
    ctx.close()
