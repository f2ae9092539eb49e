"""The static decoder where there are many rows: 16 rows of a pass share a workgroup and the pass's steps in LDS.  Every batch of
ranks up to the form's limit and one past it, rows that are no multiple of a workgroup's, of a wave's or of a pair, a ragged last
pass, selected features that fill more than one wave, no selected features, another code width; and the waves of 4 rows that are left where there are
more ranks.  Sampled rows against the oracle, bit by bit."""
import numpy as np
import pytest
import torch

from test_gpu_static import _ranges_from, _static_case

pytestmark = pytest.mark.gpu


def _case(T, E, N, k, bits=4):
    rng = np.random.default_rng(T + E + N)
    idx = np.sort(rng.choice(E, k, replace=False)).astype(np.int32)
    g = torch.Generator(device="cuda")
    g.manual_seed(T + N)
    Ys = [(torch.randn((T, E), generator=g, device="cuda") * (0.5 + i)).to(torch.bfloat16) for i in range(N)]
    m, M = _ranges_from(Ys)
    rows = np.unique(np.concatenate([np.arange(0, 40), np.arange(T - 40, T), rng.integers(0, T, 60)]))
    _static_case(E, 128, Ys, idx, m, M, rows=rows, ld_out=E + 8, bits=bits)


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 12, 13, 16, 17])
def test_ranks(N):
    _case(5003, 520, N, 9)


@pytest.mark.parametrize("T,E,N,k,bits", [
    (10001, 512, 3, 0, 4),       # k = 0, one row past a workgroup
    (1682, 2304, 4, 80, 4),      # two waves of selected features, two rows in the last pair
    (10014, 72, 2, 72, 4),       # k = E: nothing but selected features
    (2521, 1160, 5, 37, 2), (2522, 1160, 6, 37, 3), (2523, 1160, 7, 37, 5), (2524, 1160, 8, 37, 6), (2525, 1160, 9, 37, 8),
])
def test_shapes(T, E, N, k, bits):
    _case(T, E, N, k, bits)


# T, E, N, k, bits at which k_decode_static takes 4 rows a wave: more ranks than the steps in LDS are for (12 in the bf16 chain, 16 in
# fp32); rows that are no multiple of 4.
FOUR_ROWS = [(8195, 520, 13, 9, 4), (8197, 520, 16, 9, 4), (8194, 520, 17, 9, 4), (8195, 520, 23, 9, 4), (5479, 520, 17, 70, 4), (16385, 512, 18, 0, 4),
             (8195, 520, 13, 9, 3), (8198, 520, 17, 9, 5), (8195, 520, 19, 9, 8)]


@pytest.mark.parametrize("T,E,N,k,bits", FOUR_ROWS)
def test_four_rows_a_wave(T, E, N, k, bits):
    _case(T, E, N, k, bits)
