"""The decoder at every number of ranks: batches of 1 to 8 ranks have code of their own, more than 8 ranks a loop and a
remainder, in each of the decoder's forms (few selected features, many, compacted rows for more than 8 ranks, other code widths,
epilogue, static mode).  Ranks differ in magnitude by up to 2^24, so that the literal bf16 chain rounds terms away, keeps them
and meets ties.  Codes, sections and sums against the oracle, bit by bit (the order of the additions is fixed)."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as wl
from test_gpu_bits import _case as bits_case
from test_gpu_fused import _case as fused_case
from test_gpu_parity import _codec_case
from test_gpu_static import _ranges_from, _static_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [9, 70])   # at most 16 selected columns a pass of 512, or a lane per column
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 23])
def test_rank_count(N, k):
    T, E, G = 3, 1048, 32
    rng = np.random.default_rng(100 * N + k)
    idx = np.sort(rng.choice(E, k, replace=False)).astype(np.int32)
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    Ys = [(torch.randn((T, E), generator=g, device="cuda") * 2.0 ** (6 * (i % 5) - 12)).to(torch.bfloat16) for i in range(N)]
    _codec_case(dataclasses.replace(wl.TINY, N=N, T=T, E=E, k=k, G=G), Ys, idx)
    bits_case(E, G, (5, 6, 8)[N % 3], Ys, idx)
    addend = torch.randn((T, E), generator=g, device="cuda").to(torch.bfloat16)
    fused_case(E, G, Ys, idx, addend, addend[0].contiguous())
    m, M = _ranges_from(Ys)
    _static_case(E, G, Ys, idx, m, M)
