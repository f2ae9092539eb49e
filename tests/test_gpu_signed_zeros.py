"""The decoder on messages that the encoder never writes: scales that are -0 or negative, zero points of -0, steps of 0 with
any code.  A sum whose terms are all -0 is -0, in fp32 and in the literal bf16 chain (IEEE addition; any other sum of zeros is
+0).  And the chain's additions over pairs and triples of values picked from the whole range of bf16.  Against the oracle, bit by
bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2411_07942_amd as tpq
from gpu_common import gpu_decode, gpu_plan

pytestmark = pytest.mark.gpu


def _message(L, T, ref):
    """The oracle's dense message as the library's sections."""
    m = tpq.Message(L, T, "cuda", fill=0)
    for name, pitch in (("codes", L.pitch_codes), ("scale", L.pitch_meta), ("zero", L.pitch_meta), ("outl", L.pitch_outl)):
        a = np.ascontiguousarray(getattr(ref, name)).view(np.uint8).reshape(T, -1)
        if a.size:
            rows = np.zeros((T, pitch), np.uint8)
            rows[:, :a.shape[1]] = a
            getattr(m, name)[:T * pitch] = torch.from_numpy(rows.reshape(-1)).cuda()
    return m


@pytest.mark.parametrize("k", [9, 70])   # the two forms of the selected features
@pytest.mark.parametrize("bits", [4, 6])
@pytest.mark.parametrize("N", [1, 2, 3, 5, 8, 9, 12, 64])
def test_sums_of_negative_zeros(N, bits, k):
    T, E, G = 5, 1048, 32
    rng = np.random.default_rng(100 * N + 10 * bits + k)
    idx = np.sort(rng.choice(E, k, replace=False)).astype(np.int32)
    L = tpq.layout_init(E, k, G, bits)
    plan = gpu_plan(L, idx)
    every = rng.random((T, L.ng)) < 0.5           # groups where every rank has the sign
    few = rng.random((T, L.code_bytes)) < 0.4     # bytes in which every rank has codes of 0
    msgs = []
    for _ in range(N):
        sign = every | (rng.random((T, L.ng)) < 0.5)
        scale = np.where(sign, rng.choice(np.array([0x8000, 0xBF80, 0x8001], np.uint16), (T, L.ng)),
                         rng.choice(np.array([0, 0x3F80], np.uint16), (T, L.ng))).astype(np.uint16)
        zero = np.where(sign, 0x8000, rng.choice(np.array([0, 0x8000, 0x3F80], np.uint16), (T, L.ng))).astype(np.uint16)
        codes = np.where(few | (rng.random((T, L.code_bytes)) < 0.5), 0, rng.integers(0, 256, (T, L.code_bytes))).astype(np.uint8)
        outl = rng.choice(np.array([0x8000, 0x8000, 0, 0x3F80], np.uint16), (T, k))
        msgs.append(oracle.Message(outl, codes, scale, zero))
    sent = [_message(L, T, m) for m in msgs]
    zeros = 0
    for accum, out_fp32 in ((tpq.ACC_BF16, False), (tpq.ACC_BF16, True), (tpq.ACC_FP32, False)):
        want = oracle.decode_reduce(msgs, idx, E, G, accum, out_fp32=out_fp32, bits=bits)
        got, _ = gpu_decode(L, plan, sent, T, accum, out_fp32)
        u = np.uint32 if out_fp32 else np.uint16
        assert np.array_equal(got.view(u), want.view(u)), (accum, out_fp32)
        zeros += int(np.sum(want.view(u) == (0x80000000 if out_fp32 else 0x8000)))
    assert zeros > 0


def _range_of_bf16():
    """Signs x exponents at both ends, around 1 and its neighbourhood x significands at the ends, the halves and the ties."""
    exps = [0, 1, 2, 8, 9, 10, 100, 118, 119, 120, 125, 126, 127, 128, 134, 135, 136, 200, 253, 254]
    sigs = [0, 1, 2, 0x3F, 0x40, 0x41, 0x7E, 0x7F]
    v = np.array([(e << 7) | s for e in exps for s in sigs], np.uint16)
    return np.concatenate([v, v | 0x8000])


@pytest.mark.parametrize("scale", [0x0000, 0x8000])   # a term is then the zero point itself (0 x 0 + zero; with +0 a zero point of -0 is +0)
@pytest.mark.parametrize("N", [2, 3, 9])
def test_chain_over_the_range_of_bf16(N, scale):
    v = _range_of_bf16()
    E, G = 10240, 32
    ng = E // G                                    # a row: one value of the first rank's with every value of the second's
    assert ng == v.size
    T = v.size
    rng = np.random.default_rng(N)
    L = tpq.layout_init(E, 0, G)
    idx = np.zeros(0, np.int32)
    plan = gpu_plan(L, idx)
    zero = [np.repeat(v[:, None], ng, 1), np.repeat(v[None, :], T, 0)] + [rng.choice(v, (T, ng)) for _ in range(N - 2)]
    codes = np.zeros((T, L.code_bytes), np.uint8)
    msgs = [oracle.Message(np.zeros((T, 0), np.uint16), codes, np.full((T, ng), scale, np.uint16), z) for z in zero]
    want = oracle.decode_reduce(msgs, idx, E, G, tpq.ACC_BF16, threads=8)
    got, _ = gpu_decode(L, plan, [_message(L, T, m) for m in msgs], T, tpq.ACC_BF16, False)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("bits", [3, 8])
@pytest.mark.parametrize("T", [7, 5003])           # a wave per row; where 5003, a workgroup per 16 rows
def test_static_steps_of_zero(T, bits):
    """A code below 0 times a step of 0 is -0."""
    E, k, G, N = 520, 9, 32, 3
    rng = np.random.default_rng(T + bits)
    idx = np.sort(rng.choice(E, k, replace=False)).astype(np.int32)
    L = tpq.layout_init(E, k, G, bits)
    plan = gpu_plan(L, idx)
    M = torch.rand((N, E), device="cuda") + 0.5
    M[:, rng.random(E) < 0.6] = 0.0
    step, _ = tpq.static_params(L, plan, -M, M)
    step_ref, _ = oracle.static_params(-M.cpu().numpy(), M.cpu().numpy(), bits=bits)
    msgs = [oracle.StaticMessage(rng.integers(0, 0x7F00, (T, k)).astype(np.uint16),
                                 rng.integers(0, 256, (T, L.code_bytes)).astype(np.uint8)) for _ in range(N)]
    sent = []
    for m in msgs:
        sent.append(_message(L, T, oracle.Message(m.outl, m.codes, np.zeros((T, L.ng), np.uint16), np.zeros((T, L.ng), np.uint16))))
    for accum in (tpq.ACC_BF16, tpq.ACC_FP32):
        out = torch.empty((T, E), dtype=torch.float32, device="cuda")
        tpq.decode_reduce_static(L, plan, sent, step, out, accum)
        torch.cuda.synchronize()
        want = oracle.decode_reduce_static(msgs, idx, step_ref, accum, out_fp32=True, threads=8, bits=bits)
        assert np.sum(want.view(np.uint32) == 0x80000000) > 0
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), accum
