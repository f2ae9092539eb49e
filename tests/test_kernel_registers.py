"""What the compiler reports about the kernels of the built library: registers that did not fit.

The decoder's kernels hold their ranks' pointers in scalar registers.  Where those of all batch sizes were loaded ahead of the
branch between them, 48 and 58 of them were written to vector lanes and read back one by one, four cycles each: with fp32 output
2048 x 5120 of 8 ranks took 25.2 us instead of 20.0.
"""
import os
import re
import struct
import subprocess

import pytest

import paper_2411_07942_amd as tpq

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")


def _code_objects(path):
    """The gfx950 code objects of a shared library built by hipcc (clang's offload bundles: a magic, the number of entries, and per
    entry offset, size and the target's name)."""
    data = open(path, "rb").read()
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        pos = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            offset, size, n = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + n]:
                yield data[at + offset:at + offset + size]
            pos += 24 + n
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> the figures of its metadata"""
    out = {}
    for i, code in enumerate(_code_objects(tpq.LIB_PATH)):
        f = tmp_path_factory.mktemp("code") / ("%d.co" % i)
        f.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(f)], check=True, capture_output=True, text=True).stdout
        for entry in re.split(r"\n  - \.", notes)[1:]:
            v = dict(re.findall(r"\.?(\w+):\s+(\S+)", entry))
            if "name" in v:
                out[v["name"]] = {k: int(v[k]) for k in ("sgpr_spill_count", "vgpr_spill_count", "private_segment_fixed_size")}
    names = subprocess.run(["c++filt"], input="\n".join(out), check=True, capture_output=True, text=True).stdout.splitlines()
    return {re.search(r"\b(k_\w+(?:<[^>]*>)?)\(", n).group(1): v for n, v in zip(names, out.values())}


def test_decoder_registers(kernels):
    decoder = {n: v for n, v in kernels.items() if n.startswith("k_decode_")}
    assert len(decoder) > 100
    for name, v in decoder.items():
        assert v["vgpr_spill_count"] == 0 and v["private_segment_fixed_size"] == 0, (name, v)
        assert v["sgpr_spill_count"] <= 24, (name, v)
