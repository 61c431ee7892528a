"""The profile summaries of bench.py: every GEMM, head and attention kernel of
the sources has a family, and the timed launches are the last ones of all W4A16
GEMM kernels, not of one of them."""
import argparse
import json
import os
import re

import pytest

import bench
from paper_2606_31808_amd import build

NS = "void lmop::(anonymous namespace)::"
ARG = "(lmop::GemmArgs)"
NAMES = {
    "gemm_kernel": {"gemm_kernel<8, 1, 2, 4, 4, 1, 1, 2>": "W4A16 GEMM, SwiGLU (gate/up)",
                    "gemm_kernel<1, 1, 1, 1, 4, 8, 8, 1>": "W4A16 GEMM, residual add (o, down)",
                    "gemm_kernel<4, 2, 4, 2, 4, 2, 2, 2>": "W8A16 GEMM (FP8 weights)"},
    "gemm_split_kernel": {"gemm_split_kernel<1, 1, 1, 8>": "W4A16 GEMM, residual add (o, down)",
                          "gemm_split_kernel<1, 4, 2, 4>": "W4A16 GEMM, QKV + RoPE (qkv)",
                          "gemm_split_kernel<2, 1, 1, 8>": "W8A16 GEMM (FP8 weights)"},
    "head2_kernel": {"head2_kernel<5, 4>": "LM head GEMM"},
    "head_few_kernel": {"head_few_kernel<1, 4>": "LM head GEMM"},
    "attn_kernel": {"attn_kernel<128>": "attention"},
}


def test_every_kernel_has_a_family():
    found = set()
    for f in ("gemm.hip", "attention.hip"):
        with open(os.path.join(build.CSRC, f)) as src:
            found |= set(re.findall(r"^__global__.*?\bvoid (\w+)\(", src.read(), flags=re.M))
    assert found == set(NAMES)
    for samples in NAMES.values():
        for name, family in samples.items():
            assert bench.kernel_family(NS + name + ARG) == family
            assert bench._is_w4_gemm(NS + name + ARG) == family.startswith("W4A16")
    assert bench.kernel_family(NS + "rmsnorm_wave_kernel<16>") is None


@pytest.mark.parametrize("few", [0, 3, 7])
def test_timed_rows_count_split_launches(few):
    """A prefix pass of 6 launches, then 10 timed ones, some of few tokens."""
    names = ["gemm_kernel<8, 1, 2, 4, 4, 1, 1, 2>"] * (16 - few) + \
        ["gemm_split_kernel<1, 1, 1, 8>"] * few
    rows = [{"Kernel_Name": NS + n + ARG, "Dispatch_Id": str(2 * i)} for i, n in enumerate(names)]
    rows += [{"Kernel_Name": "other", "Dispatch_Id": str(2 * i + 1)} for i in range(16)]
    got = [int(r["Dispatch_Id"]) for r in bench._timed_gemm_rows(rows[::-1], 10)]
    assert got == list(range(12, 32, 2))


@pytest.mark.parametrize("change,known", [
    ({}, True), ({"workload": "filter_1b"}, False), ({"rows": 100}, False), ({"limit": 5}, False),
    ({"cascade": True}, False), ({"batch_tokens": 4096}, False), ({"workspace_gb": 8.0}, False),
    ({"weights": "fp8_e4m3"}, False), ({"head_restricted": True}, True)])
def test_traffic_is_of_the_recorded_workload(tmp_path, change, known):
    """The counters' bytes per launch go with the run that they were taken on."""
    args = argparse.Namespace(workload="filter_8b", rows=None, batch_tokens=0, limit=0,
                              cascade=False, workspace_gb=0.0, weights="int4_g32",
                              head_restricted=False)
    vars(args).update(change)
    f = tmp_path / "t.json"
    f.write_text(json.dumps({"workload": "filter_8b", "bytes_per_launch": 7.0,
                             "gemm_src_sha256_16": bench._src_hash()}))
    got = bench.measured_traffic(str(f), bench.recorded_workload(args))
    assert got == (7.0 if known else None)
    f.write_text(json.dumps({"workload": "filter_8b", "bytes_per_launch": 7.0,
                             "gemm_src_sha256_16": "0"}))
    assert bench.measured_traffic(str(f), "filter_8b") is None
