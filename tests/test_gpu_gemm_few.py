"""The linear layer with few tokens: a workgroup per group of features and 16, 32 or 64 tokens, whose waves share K.  Sizes at the edges
of a workgroup's tokens, of the stages of 32 k and of the waves' shares of them (fewer stages than waves, one more, a ring that
is refilled), last groups that are ragged, hold selected features or nothing else, and larger sizes where the tiles take over.
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
    (100, 640, 5120, 80, 64),     # 64 tokens a workgroup, the second one ragged
    (100, 1728, 5120, 80, 32),    # more workgroups than compute units
    (230, 752, 2248, 35, 64),
    (16, 3584, 8192, 128, 128),   # weights larger than the L2s
    (300, 1728, 5120, 80, 128),   # tiles of 128 x 128
    (200, 1728, 5120, 80, 256),   # tiles of 256 x 64
    (200, 2400, 8192, 80, 64),    # tiles of 128 x 64
])
def test_sizes_between(T, K, E, k, G):
    _run(T, K, E, k, G, seed=T + K, rows=sorted({0, 14, 15, min(16, T - 1), T // 2, T - 2, T - 1}))
