"""tpq_calibrate_finalize's selection at the edges of its digits and rounds (digits of 11 bits from the first bit in which the
ranges differ, 1024 features a round of the workgroup), and tpq_calibrate's one-launch form at the rows of its variants.
Indices and state are compared with the oracle exactly."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import paper_2411_07942_amd as tpq
import workloads as wl
from test_gpu_parity import _calibrate_both, _finalize_both

pytestmark = pytest.mark.gpu


def _ranges(kind, E, rng):
    if kind == "equal":                    # no bit differs: ties alone decide
        return np.full(E, 2.5, np.float32)
    if kind == "neighbours":               # the low bits decide: one digit, a few values
        return (np.float32(1.5).view(np.uint32) + rng.integers(0, 5, E).astype(np.uint32)).view(np.float32)
    if kind == "three digits":             # every bit but the sign is open
        return rng.integers(1, 0x7F000000, E).astype(np.uint32).view(np.float32)
    if kind == "signs":                    # one-signed columns whose ranges are negative, and zeros
        return (rng.integers(-3, 4, E) * rng.choice([1.0, 1e-30, 1e30], E)).astype(np.float32)
    return np.where(rng.random(E) < 0.02, 1e4, 1.0).astype(np.float32) * rng.integers(1, 3, E).astype(np.float32)  # "few values"


@pytest.mark.parametrize("kind", ["equal", "neighbours", "three digits", "signs", "few values"])
@pytest.mark.parametrize("E", [8, 1024, 1032, 4096, 4104, 8192, 8200, 32768])
def test_selection(kind, E):
    rng = np.random.default_rng(E + len(kind))
    M = _ranges(kind, E, rng).reshape(1, E)
    m = -M
    for k in sorted({1, max(1, E // 64), E // 2, E - 1, E}):
        _finalize_both(torch.from_numpy(m).cuda(), torch.from_numpy(M).cuda(), m, M, k)


@pytest.mark.parametrize("kind", ["equal", "neighbours", "three digits", "signs", "few values"])
@pytest.mark.parametrize("E", [8, 1024, 1032, 4096, 4104, 8192, 8200, 12288, 16384, 16392, 32768])
def test_selection_without_the_ranked_list(kind, E):
    """The ascending list alone is another kernel's; its workspace stays as it is."""
    rng = np.random.default_rng(E + len(kind))
    M = _ranges(kind, E, rng).reshape(1, E)
    m = -M
    Rbar = torch.empty(E, device="cuda")
    ws = torch.full((tpq.calibrate_finalize_workspace_bytes(E),), 0xA5, dtype=torch.uint8, device="cuda")
    for k in sorted({1, max(1, E // 64), E // 2, E - 1, E}):
        idx = torch.full((k + 64,), -7, dtype=torch.int32, device="cuda")
        tpq.calibrate_finalize(torch.from_numpy(m).cuda(), torch.from_numpy(M).cuda(), k, Rbar, idx, None, ws)
        torch.cuda.synchronize()
        _, Rbar_ref, sorted_ref, _ = oracle.calibrate_finalize(m, M, k)
        assert np.array_equal(Rbar.cpu().numpy(), Rbar_ref)
        assert np.array_equal(idx[:k].cpu().numpy(), sorted_ref) and bool((idx[k:] == -7).all().item())
    assert bool((ws == 0xA5).all().item())


@pytest.mark.parametrize("E,k", [(512, 8), (5120, 80), (5120, 4000), (16384, 100)])
def test_unordered_ranges_without_the_ranked_list(E, k):
    """Ranges that are NaN: which indices come out is unspecified, but they are features, ascending, and no more than k."""
    M = torch.rand((2, E), device="cuda")
    M[:, ::3] = float("nan")
    Rbar = torch.empty(E, device="cuda")
    idx = torch.full((k + 1024,), -7, dtype=torch.int32, device="cuda")
    ws = torch.empty(tpq.calibrate_finalize_workspace_bytes(E), dtype=torch.uint8, device="cuda")
    tpq.calibrate_finalize(-M, M, k, Rbar, idx, None, ws)
    torch.cuda.synchronize()
    got = idx.cpu().numpy()
    assert np.all(got[k:] == -7) and np.all((got[:k] >= 0) & (got[:k] < E)) and np.all(np.diff(got[:k]) > 0)


@pytest.mark.parametrize("S", [127, 255, 256, 257, 511, 512, 513])
def test_calibrate_rows_of_a_step(S):
    """One step of 128, 256, 512 or 1024 rows."""
    _calibrate_both(dataclasses.replace(wl.TINY, E=264, k=4), 3, S, N=2)
