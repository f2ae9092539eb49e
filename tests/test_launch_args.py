"""What the decoder's kernels may read as selected features stays inside the caller's sections.

Every wave reads the selected features' values of 8 ranks at a time, whether or not it uses them: from pointers and at a
row pitch that the host hands over.  tests/probes/launch_args runs the host half without a GPU and prints both;
here the furthest byte of each is held against the section the pointer lies in.
"""
import os
import subprocess

import pytest

import paper_2411_07942_amd as tpq

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def launch_args(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("launch_args") / "launch_args")
    subprocess.run(["hipcc", "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2411_07942_amd", "csrc"),
                    os.path.join(ROOT, "tests", "probes", "launch_args.hip"), "-o", exe, "-rdynamic", "-ldl"],
                   check=True, capture_output=True, text=True)

    def run(E, k, G, bits, N, T, pitch_outl):
        r = subprocess.run([exe, tpq.LIB_PATH] + [str(v) for v in (E, k, G, bits, N, T, pitch_outl)],
                           check=True, capture_output=True, text=True, timeout=60)
        return [(int(w[0]), int(w[1]), [int(p, 16) for p in w[2:]]) for w in map(str.split, r.stdout.splitlines())]
    return run


@pytest.mark.parametrize("E,k,G,bits,N,T,pitch_outl", [
    (512, 0, 64, 4, 3, 7, 0), (512, 0, 64, 4, 3, 7, 16), (512, 0, 64, 4, 8, 7, 4096),   # no selected features, pitch raised
    (512, 0, 128, 6, 9, 7, 4096), (512, 0, 64, 4, 1, 2000000, 4096),                    # another width; four blocks of rows
    (512, 8, 64, 4, 9, 7, 16), (512, 8, 64, 3, 2, 7, 4096), (512, 511, 64, 4, 5, 1, 1024),
])
def test_selected_features_are_read_inside_a_section(launch_args, E, k, G, bits, N, T, pitch_outl):
    L = tpq.layout_init(E, k, G, bits)
    # the sections' addresses, as the program lays them out, and their ends
    sections = {}
    for i in range(N):
        sections[(1 + 4 * i) << 40] = T * L.pitch_codes
        sections[(4 + 4 * i) << 40] = T * pitch_outl
    launches = launch_args(E, k, G, bits, N, T, pitch_outl)
    assert sum(rows for rows, _, _ in launches) == T
    for rows, pitch, pointers in launches:
        assert len(pointers) == -(-N // 8) * 8
        for p in pointers:
            base = p >> 40 << 40
            last = 2 * (max(k, 1) - 1)
            assert p + (rows - 1) * pitch + last + 2 <= base + sections[base]
