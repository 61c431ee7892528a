"""Which tile shape each weight GEMM of a pass takes, from the dispatch rule
itself (csrc/gemm_tiles.h, compiled for the host)."""
import ctypes as C
import os
import subprocess

from paper_2606_31808_amd import build

EPILOGUES = ("qkv", "add", "swiglu")
QUERY_SPLIT_TOKENS = 256  # kQuerySplitTokens of lmop_api.cpp

SOURCE = """
#include "gemm_tiles.h"
extern "C" int pick(int fp8, int add, int M, int N, int K) {
  return lmop::pick_gemm_tile(fp8, add, M, N, K);
}
extern "C" int head_streams(int rows, int vocab) { return lmop::head_streams(rows, vocab); }
extern "C" int tiles() { return lmop::kNumGemmTiles; }
extern "C" int offered(int i, int fp8, int add) { return lmop::kGemmTiles[i].offered(fp8, add); }
"""


def load_rule(folder):
    src, so = os.path.join(folder, "tiles.cpp"), os.path.join(folder, "tiles.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", f"-I{build.CSRC}", src, "-o", so],
                   check=True)
    return C.CDLL(so)


def _up(x, m):
    return -(-x // m) * m


def launches(shape, tokens, rows):
    """(epilogue, M, N, K) of every GEMM of one pass of `rows` rows with
    `tokens` tokens in all, as `forward` launches them."""
    d, nq, nkv = shape.d_model, shape.n_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim
    f64, qkv = _up(shape.d_ff, 64), nq + 2 * nkv
    out = []
    for l in range(shape.n_layers):
        m = tokens
        if l == shape.n_layers - 1:
            m = rows
            if tokens - rows >= QUERY_SPLIT_TOKENS and rows * d <= tokens * f64:
                out.append(("qkv", tokens, _up(qkv, 256) - nq // 256 * 256, d))
                out.append(("qkv", rows, _up(nq, 256), d))
            else:
                out.append(("qkv", tokens, _up(qkv, 256), d))
        else:
            out.append(("qkv", m, _up(qkv, 256), d))
        out.append(("add", m, _up(d, 256), nq))
        out.append(("swiglu", m, _up(2 * _up(shape.d_ff, 32), 256), d))
        out.append(("add", m, _up(d, 256), f64))
    return out


def picked(rule, fp8, shape, passes):
    """{(epilogue, tile index)} over passes of (tokens, rows)"""
    return {(e, rule.pick(fp8, e == "add", M, N, K))
            for tokens, rows in passes for e, M, N, K in launches(shape, tokens, rows)}


def offered(rule, fp8):
    return {(e, i) for e in EPILOGUES for i in range(rule.tiles())
            if rule.offered(i, fp8, e == "add")}
