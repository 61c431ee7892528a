"""The dispatch rules on the host: the passes that the GPU tests run take every
tile shape that the GEMM's rule offers, in every epilogue and weight format;
the LM head's rule takes the faster kernel."""
import dataclasses
import shutil

import pytest

from tests import gemm_launches as G
from tests import test_gpu_gemm_tiles as gpu


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    return G.load_rule(str(tmp_path_factory.mktemp("rule")))


def _passes(tokens):
    lens = gpu._rows(tokens)
    return [(tokens, len(lens))] + [(n, 1) for n in lens[:gpu.ALONE]]


@pytest.mark.parametrize("fmt", ["int4_g32", "fp8_e4m3"])
def test_gpu_cases_take_every_shape(rule, fmt):
    fp8 = fmt == "fp8_e4m3"
    taken = set()
    for f, d_ff in gpu.MODELS:
        if f == fmt:
            shape = dataclasses.replace(gpu.SHAPE, d_ff=d_ff)
            for t in gpu.TOKENS:
                taken |= G.picked(rule, fp8, shape, _passes(t))
    for f, widths, tokens in gpu.OTHER:
        if f == fmt:
            taken |= G.picked(rule, fp8, gpu._other(widths), _passes(tokens))
    assert taken == G.offered(rule, fp8)


# us per launch, streaming and ring kernel: (d, V, [(rows, stream, ring)])
HEAD = [
    (2048, 2048, [(1, 38.8, 56.2), (32, 56.7, 61.2), (64, 91.7, 66.7)]),
    (2048, 16384, [(16, 52.3, 59.9), (24, 59.6, 62.6), (32, 62.6, 62.7), (64, 101.2, 68.0)]),
    (2048, 50304, [(16, 62.0, 63.5), (24, 63.6, 63.9), (32, 66.6, 64.5), (64, 104.1, 69.5)]),
    (2048, 66048, [(1, 55.6, 114.6), (32, 68.4, 123.5), (64, 105.1, 135.0)]),
    (2048, 128256, [(1, 83.4, 132.1), (32, 84.6, 137.1), (64, 114.7, 149.9)]),
    (4096, 2048, [(1, 78.6, 98.5), (17, 91.7, 102.6), (32, 104.5, 104.6), (64, 173.3, 110.1)]),
    (4096, 8192, [(16, 95.2, 103.1), (17, 98.4, 103.6), (32, 112.1, 106.0), (64, 186.6, 111.8)]),
    (4096, 32000, [(16, 100.1, 103.9), (17, 103.4, 105.0), (32, 116.5, 106.7), (64, 189.6, 112.8)]),
    (4096, 65024, [(1, 101.9, 106.5), (17, 111.8, 107.2), (32, 124.6, 110.1), (64, 195.8, 117.0)]),
    (4096, 66048, [(1, 102.4, 200.3), (32, 124.3, 210.4), (64, 195.3, 221.2)]),
    (4096, 128256, [(1, 160.1, 208.6), (32, 159.5, 219.3), (64, 211.7, 231.6)]),
    (4096, 262144, [(1, 322.7, 417.9), (32, 314.6, 432.5), (64, 370.3, 458.8)]),
]


@pytest.mark.parametrize("d,vocab,points", HEAD)
def test_head_takes_the_faster_kernel(rule, d, vocab, points):
    for rows, stream, ring in points:
        took = stream if rule.head_streams(rows, vocab) else ring
        assert took <= 1.05 * min(stream, ring), rows  # repeated runs differ by up to 4%
    assert not rule.head_streams(65, vocab)  # its rows do not fit a wave
