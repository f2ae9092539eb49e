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


# Kernel times in us, weights in the memory-side cache: the tile that the rounds choose, then 16, 32 and 64 tokens a workgroup of
# k_gemm_few.
GEMM_TIMES = [
    # T, K, E, G
    ((13, 640, 5120, 128), (9.0, 6.0, 6.1)),
    ((16, 640, 5120, 256), (10.0, 9.5, 9.5)),
    ((16, 1728, 5120, 128), (15.1, 10.8, 10.8)),
    ((64, 1728, 5120, 128), (16.0, 9.3, 11.8)),
    ((400, 1728, 5120, 128), (17.8, 29.0, 22.8)),
    ((700, 640, 5120, 128), (11.2, 26.8, 21.5)),
    ((1, 640, 5120, 64), (9.0, 4.0, 4.2, 4.8)),
    ((160, 1728, 5120, 64), (16.4, 17.4, 13.6, 10.6)),
    ((64, 640, 5120, 32), (10.0, 7.5, 7.0, 6.3)),
    ((33, 3584, 8192, 64), (26.0, 18.2, 12.7, 16.2)),
    ((64, 3584, 8192, 64), (26.7, 19.9, 14.0, 19.4)),
    ((16, 3584, 8192, 256), (30.2, 37.6, 38.2)),
    ((256, 256, 8192, 32), (7.9, 25.9, 19.0, 15.3)),
    ((429, 11824, 2416, 64), (78.8, 183.8, 130.7, 121.4)),
    ((14, 2880, 4144, 256), (23.9, 29.8, 30.6)),
    ((3, 13312, 296, 256), (96.5, 121.3, 121.9)),
    ((756, 7536, 1168, 256), (85.2, 88.0, 101.7)),
    ((23, 6712, 2264, 256), (78.1, 93.7, 100.4)),
]


def test_gemm_takes_a_fast_form(launched):
    """Never a form slower than the tile, nor more than 10 % off the fastest."""
    kernels = launched([("gemm", E, E // 64, G, T, K) for (T, K, E, G), _ in GEMM_TIMES])
    for (size, times), (kernel,) in zip(GEMM_TIMES, kernels):
        m = re.match(r"k_gemm_few<%d, (\d)>" % size[3], kernel)
        taken = times[{1: 1, 2: 2, 4: 3}[int(m.group(1))]] if m else times[0]
        assert taken <= times[0] and taken <= 1.1 * min(times), (size, kernel, times)


def test_gemm_forms_of_the_tests(launched):
    """The cases of test_gpu_gemm_few's FORMS, and the tiles that test_gpu_gemm names, run the kernels they say."""
    from test_gpu_gemm_few import FORMS
    cases = [(name, case) for name, of in FORMS for case in of] + [
        ("k_gemm_few<128, 1>", (65, 72, 5120, 80, 128)), ("k_gemm_tile<64, 1, 4, 1>", (500, 104, 5128, 77, 64)),
        ("k_gemm_tile<32, 2, 2, 2>", (900, 40, 5128, 77, 32)), ("k_gemm_tile<256, 2, 2, 1>", (300, 328, 5120, 80, 256)),
        ("k_gemm_tile<128, 2, 2, 3>", (2040, 200, 5120, 80, 128)), ("k_gemm_tile<256, 2, 2, 3>", (2040, 200, 5120, 300, 256)),
        ("k_gemm_tile<64, 2, 2, 4>", (4090, 136, 8192, 341, 64)), ("k_gemm_tile<128, 1, 2, 1>", (300, 1728, 5120, 80, 128)),
        ("k_gemm_tile<256, 2, 2, 1>", (200, 1728, 5120, 80, 256)), ("k_gemm_tile<64, 1, 2, 1>", (200, 2400, 8192, 80, 64)),
        ("k_gemm_few<64, 4>", (100, 640, 5120, 80, 64)), ("k_gemm_few<64, 4>", (230, 752, 2248, 35, 64)),
        ("k_gemm_few<32, 4>", (100, 1728, 5120, 80, 32)), ("k_gemm_few<128, 1>", (16, 3584, 8192, 128, 128))]
    ran = launched([("gemm", E, k, G, T, K) for _, (T, K, E, k, G) in cases])
    assert [(n, c) for (n, c), r in zip(cases, ran) if r != [n]] == []


def test_static_forms_of_the_tests(launched):
    """The cases of test_gpu_static_rows: the bf16 chain of every one of FOUR_ROWS has 4 rows a wave, and so have fp32 sums of more than
    16 ranks; full sizes of up to 12 ranks have the steps in LDS."""
    from test_gpu_static_rows import FOUR_ROWS
    for T, E, N, k, bits in FOUR_ROWS:
        gen = "true" if bits != 4 else "false"
        fp32, fp32_out, bf16 = launched([("static", E, k, 128, bits, N, T, acc, out) for acc, out in ((0, 0), (0, 1), (1, 0))])
        assert bf16 == ["k_decode_static<1, 0, 4, %s>" % gen]
        if N > 16:
            assert fp32 == ["k_decode_static<0, 0, 4, %s>" % gen] and fp32_out == ["k_decode_static<0, 1, 4, %s>" % gen]
        else:
            assert fp32 == ["k_decode_static_lds<0, 0, 2, %s>" % gen]
    for acc in (0, 1):
        assert launched([("static", 5120, 80, 128, 4, 8, 2048, acc, 0), ("static", 520, 9, 128, 4, 12, 5003, acc, 0)]) == [
            ["k_decode_static_lds<%d, 0, 2, false>" % acc]] * 2
        assert launched([("static", 520, 9, 128, 4, 17, 5003, acc, 0), ("static", 5120, 80, 128, 4, 8, 64, acc, 0)]) == [
            ["k_decode_static<%d, 0, 1, false>" % acc]] * 2
