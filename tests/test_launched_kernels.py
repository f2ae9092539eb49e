"""Which kernels a call launches, by the host's rules on sizes (tests/probes/launched_kernels, without a GPU, for 256 compute units)."""
import os
import re
import subprocess

import pytest

import paper_2411_07942_amd as tpq

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def launched(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("launched_kernels") / "launched_kernels")
    subprocess.run(["hipcc", "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2411_07942_amd", "csrc"),
                    os.path.join(ROOT, "tests", "probes", "launched_kernels.hip"), "-o", exe, "-rdynamic", "-ldl"],
                   check=True, capture_output=True, text=True)

    def run(calls):
        """calls: what and its numbers; returns each call's kernels, template arguments included (k_gemm_few<128, 1>)."""
        text = "".join(" ".join(map(str, c)) + "\n" for c in calls)
        r = subprocess.run([exe, tpq.LIB_PATH], input=text, check=True, capture_output=True, text=True, timeout=60)
        out = subprocess.run(["c++filt"], input=r.stdout, check=True, capture_output=True, text=True).stdout.splitlines()
        assert len(out) == len(calls)
        return [re.findall(r"\b(k_\w+(?:<[^>]*>)?)\(", line) for line in out]
    return run


@pytest.mark.parametrize("E", [8, 4096, 4104, 8192, 8200, 16384, 16392, 32768])
def test_finalize(launched, E):
    """The ranked list takes every feature's rank, and the ascending one follows from those; alone it is a selection in one
    workgroup, 1024 features a round."""
    alone, both, none = launched([("finalize", E, 1, 8, 0), ("finalize", E, 1, 8, 1), ("finalize", E, 0, 8, 1)])
    rounds = next(r for r in (4, 8, 16, 32) if E <= 1024 * r)
    assert alone == ["k_ranges", "k_top<%d>" % rounds]
    assert both == ["k_ranges", "k_rank", "k_select"]
    assert none == ["k_ranges"]
