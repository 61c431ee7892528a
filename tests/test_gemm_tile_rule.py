"""The GEMM's dispatch rule on the host: the passes that the GPU tests run take
every tile shape that the rule offers, in every epilogue and weight format."""
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
