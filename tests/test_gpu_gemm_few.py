"""The linear layer with few tokens: a workgroup per group of features and 16, 32 or 64 tokens, whose waves share K.  FORMS holds cases for
every form of this kernel and for the tiles, sizes at which the rule takes it (test_launched_kernels holds the rule to that).  The first
two tests are sizes at the edges of the stages of 32 k and of the waves' shares of them (fewer stages than waves, one more, a ring that is
refilled), and last groups that are ragged, hold selected features or nothing else; nearly all of them take 16 tokens a workgroup.
The bars are those of test_gpu_gemm."""
import pytest

from test_gpu_gemm import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [32, 64, 128, 256])
@pytest.mark.parametrize("T,K", [(1, 8), (15, 24), (16, 40), (17, 256), (31, 264), (33, 288), (48, 1032), (64, 72), (65, 2056)])
def test_edges(T, K, G):
    _run(T, K, 1288, 37, G, seed=T + K + G, ld_pad=8 * (T % 2))


@pytest.mark.parametrize("G", [32, 128, 256])
@pytest.mark.parametrize("E,k", [(8, 0), (8, 8), (264, 264), (520, 261), (1024, 0), (776, 600)])
def test_selected_features(E, k, G):
    _run(21, 200, E, k, G, seed=E + k + G, integer=True)


@pytest.mark.parametrize("T,K,E,k,G", [
    (100, 640, 5120, 80, 64), (230, 752, 2248, 35, 64), (100, 1728, 5120, 80, 32),    # 64 tokens a workgroup, the last one ragged
    (16, 3584, 8192, 128, 128),   # 16; weights larger than the L2s
    (300, 1728, 5120, 80, 128),   # tiles of 128 x 64
    (200, 1728, 5120, 80, 256),   # tiles of 256 x 64
    (200, 2400, 8192, 80, 64),    # tiles of 128 x 64
])
def test_sizes_between(T, K, E, k, G):
    _run(T, K, E, k, G, seed=T + K, rows=sorted({0, 14, 15, min(16, T - 1), T // 2, T - 2, T - 1}))


# Kernel, and T, K, E, k, G at which it runs.  Of each form: one token past a workgroup's or tile's with a K of two stages and a quarter (in
# k_gemm_few fewer than there are waves); one token short of a full one, with last groups of nothing but selected features; of k_gemm_few a
# full one with a K whose stages refill the waves' rings where the form takes one that long, and no selected features.
FORMS = [
    ("k_gemm_few<32, 1>", [(1, 72, 264, 37, 32), (15, 264, 264, 53, 32), (16, 1096, 264, 0, 32)]),
    ("k_gemm_few<32, 2>", [(65, 72, 4104, 37, 32), (479, 264, 264, 53, 32), (320, 1096, 264, 0, 32)]),
    ("k_gemm_few<32, 4>", [(129, 72, 1800, 37, 32), (959, 264, 264, 53, 32), (960, 1096, 264, 0, 32)]),
    ("k_gemm_few<64, 1>", [(1, 72, 264, 37, 64), (15, 264, 264, 85, 64), (16, 1096, 264, 0, 64)]),
    ("k_gemm_few<64, 2>", [(33, 72, 6152, 37, 64), (831, 264, 264, 85, 64), (832, 1096, 264, 0, 64)]),
    ("k_gemm_few<64, 4>", [(897, 72, 520, 37, 64), (639, 264, 776, 85, 64), (640, 1096, 776, 0, 64)]),
    ("k_gemm_few<128, 1>", [(1, 72, 264, 37, 128), (15, 264, 264, 149, 128), (16, 1096, 264, 0, 128)]),
    ("k_gemm_few<128, 2>", [(833, 72, 520, 37, 128), (831, 264, 520, 149, 128), (1184, 1096, 264, 0, 128)]),
    ("k_gemm_few<256, 1>", [(1, 72, 264, 37, 256), (15, 72, 520, 277, 256), (16, 1096, 264, 0, 256)]),
    ("k_gemm_few<256, 2>", [(1025, 72, 776, 37, 256), (1375, 72, 520, 277, 256), (2080, 200, 264, 0, 256)]),
    ("k_gemm_tile<32, 1, 2, 1>", [(65, 72, 6152, 37, 32), (63, 104, 8200, 53, 32)]),          # 128 features x 64 tokens
    ("k_gemm_tile<64, 1, 2, 1>", [(385, 72, 2568, 37, 64), (1279, 104, 776, 85, 64)]),
    ("k_gemm_tile<128, 1, 2, 1>", [(897, 72, 1032, 37, 128), (1215, 104, 776, 149, 128)]),
    ("k_gemm_tile<32, 1, 4, 1>", [(641, 72, 3080, 37, 32), (1151, 104, 1800, 53, 32)]),       # 128 x 128
    ("k_gemm_tile<128, 1, 4, 1>", [(641, 72, 3080, 37, 128), (1151, 104, 1800, 149, 128)]),
    ("k_gemm_tile<256, 2, 2, 1>", [(1473, 72, 1032, 37, 256), (2239, 104, 520, 277, 256)]),   # 256 x 64
    ("k_gemm_tile<256, 2, 2, 2>", [(769, 72, 5128, 37, 256), (3327, 104, 1032, 277, 256)]),   # 256 x 128
    ("k_gemm_tile<256, 2, 2, 3>", [(961, 72, 8200, 37, 256), (3647, 104, 2056, 277, 256)]),   # 256 x 192
]


@pytest.mark.parametrize("integer", [False, True])
@pytest.mark.parametrize("case", [c for _, cases in FORMS for c in cases], ids=str)
def test_every_form(case, integer):
    T, K, E, k, G = case
    rows = sorted(t for t in {0, 15, 16, 31, 32, 63, 64, T // 2, T // 3, T - 64, T - 33, T - 17, T - 16, T - 2, T - 1} if 0 <= t < T)
    _run(T, K, E, k, G, seed=T + K + G, integer=integer, rows=rows)
