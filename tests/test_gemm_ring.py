"""The GEMM ring's load counts, checked on the host: the wait before a stage is
read leaves none of its loads in flight, for every ring depth, with and
without the residual prefetch in the last stages."""
import ctypes as C
import shutil
import subprocess

import pytest

from paper_2606_31808_amd import build


@pytest.fixture(scope="module")
def ring(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("ring")
    (d / "ring.cpp").write_text(
        '#include "gemm_ring.h"\n'
        'extern "C" bool all_carry(int newest, int fly, int kt_n, int pf) {\n'
        "  return lmop::all_carry_prefetch(newest, fly, kt_n, pf);\n}\n")
    so = str(d / "ring.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", f"-I{build.CSRC}", str(d / "ring.cpp"),
                    "-o", so], check=True)
    fn = C.CDLL(so).all_carry
    fn.restype = C.c_bool
    return fn


@pytest.mark.parametrize("stages", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("ahead", [0, 1])
def test_wait_covers_the_stage(ring, stages, ahead):
    fly, loads = stages - 2 - ahead, 9
    if fly < 0:
        pytest.skip("no such ring")
    for kt_n in range(1, 40):
        for pf in range(0, min(kt_n, 32) + 1):
            carried = [loads + (s >= kt_n - pf) for s in range(kt_n)]
            for kt in range(kt_n - stages + 1):
                newest = kt + stages - 1  # the last stage issued when the wait is reached
                after = sum(carried[kt + 2 + ahead:newest + 1])
                allowed = fly * (loads + 1 if ring(newest, fly, kt_n, pf) else loads)
                assert allowed <= after, (kt_n, pf, kt, allowed, after)
                if fly == 1:  # the shapes in use: exact, no wait for a later stage
                    assert allowed == after
