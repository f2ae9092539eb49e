"""What the codec is timed on: the work that a tensor-parallel inference program has it do.

A case is one pass of one of seven paths, at one size:

  reduce    every rank's partial sum compressed in one launch, then decoded and added: the
            whole exchange of a block with the ranks resident on one GPU
  device    one device's share of a block: its own partial sum compressed, then the N messages
            that the all-gather has delivered decoded, added to residual and bias
  linear    the same share with the row-parallel linear layer in front: the product is
            compressed in the GEMM's epilogue, then decode and add as above
  static    the paper's static symmetric quantiser, whole exchange
  ring      one step of a ring reduction for several devices side by side
  calibrate a block's calibration on one device: the stream of sequences, the selection of
            the bf16 features, the plan and the static step tables that follow from it
  decode    the per-token regime of `device` through calls that are marshalled once, as a
            serving loop with fixed buffers keeps them

Sizes are those of the repository's workloads (Tiny, Llama-2-13B-shaped prefill,
Gemma-2-27B-shaped decode and calibration, Large prefill) and odd ones between them.
"""
from __future__ import annotations

import math

import torch

import paper_2411_07942_amd as tpq

ACC = {"fp32": tpq.ACC_FP32, "bf16": tpq.ACC_BF16, "fast": tpq.ACC_FAST}
OUT = {"bf16": torch.bfloat16, "fp32": torch.float32}


def listed():
    return [
        # the smallest exchange: 16 tokens of 512 features, four ranks; launches and host time
        dict(name="tiny_reduce", path="reduce", N=4, T=16, E=512, k=8, G=128, bits=4, acc="bf16", out="bf16"),
        # a decode step of one transformer block: 64 sequences, eight devices, serving loop
        dict(name="decode_block", path="decode", N=8, T=64, E=4608, k=72, G=128, bits=4, acc="bf16", out="bf16"),
        # attention output projection of a decode step with a few sequences in the batch
        dict(name="linear_decode", path="linear", N=8, T=13, E=5120, K=640, k=80, G=128, bits=4, acc="fast", out="bf16"),
        # MLP down projection of a 2048-token prefill, one device of eight, with its exchange
        dict(name="linear_prefill", path="linear", N=8, T=2048, E=5120, K=1728, k=80, G=128, bits=4, acc="fast",
             out="bf16"),
        # one device of eight in the same prefill where the partial sum comes from elsewhere
        dict(name="device_prefill", path="device", N=8, T=2048, E=5120, k=80, G=128, bits=4, acc="bf16", out="bf16"),
        # the whole exchange of that prefill: the repository's headline workload
        dict(name="prefill_reduce", path="reduce", N=8, T=2048, E=5120, k=80, G=128, bits=4, acc="fast", out="bf16"),
        # the largest: sixteen ranks of 16384 tokens, more bf16 features, small groups, fp32 sums
        dict(name="large_reduce", path="reduce", N=16, T=16384, E=8192, k=341, G=64, bits=4, acc="fp32", out="fp32"),
        # sizes that fit nothing: odd ranks, tokens, features and another code width
        dict(name="ragged_6bit", path="reduce", N=5, T=1777, E=5000, k=77, G=64, bits=6, acc="fp32", out="bf16"),
        # the static quantiser (4.2 bits a value on the wire) at the prefill size
        dict(name="static_prefill", path="static", N=8, T=2048, E=5120, k=80, G=128, bits=4, acc="fp32", out="bf16"),
        # a ring all-reduce moves T / N rows a step: 256 rows on each of eight devices
        dict(name="ring_step", path="ring", N=8, T=256, E=5120, k=80, G=128, bits=4, acc="bf16", out="bf16"),
        # calibration with short sequences: many small calls, then selection and tables
        dict(name="calibrate_short", path="calibrate", N=8, T=256, E=5120, k=80, G=128, bits=4, seqs=16),
        # calibration streamed in chunks of 16384 tokens
        dict(name="calibrate_chunks", path="calibrate", N=8, T=16384, E=4608, k=72, G=128, bits=4, seqs=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["reduce", "reduce", "device", "decode", "linear", "linear", "static", "ring", "calibrate"])
    E = 8 * rng.randint(64, 1024)                                     # 512 .. 8192
    k = rng.choice([E // 64, rng.randint(0, E // 24), rng.randint(1, E // 64)])
    c = dict(path=path, N=rng.choice([2, 3, 4, 5, 7, 8, 8, 8, 12, 16]), T=_log(rng, 16, 4096), E=E, k=k,
             G=rng.choice([32, 64, 128, 128, 256]), bits=4)
    if path == "decode":
        c["T"] = _log(rng, 1, 128)
    if path == "linear":
        c["T"] = rng.choice([_log(rng, 1, 128), _log(rng, 128, 4096)])
        c["K"] = 8 * _log(rng, 16, 448)                               # 128 .. 3584
    if path == "ring":
        c["T"] = _log(rng, 16, 1024)
    if path == "calibrate":
        c["seqs"] = rng.randint(1, 16)
        c["T"] = _log(rng, 64, 16384)
        if c["T"] > 4096:
            c["seqs"] = min(c["seqs"], 4)
        return c
    if path == "reduce" and rng.random() < 0.4:
        c["bits"] = rng.choice([2, 3, 5, 6, 8])
    if path in ("reduce", "static") and rng.random() < 0.2:
        c["T"], c["N"] = _log(rng, 4096, 16384), min(c["N"], 8)
    c["acc"] = rng.choice(["fast", "fp32", "bf16"] if path != "ring" else ["fp32", "bf16"])
    c["out"] = "bf16" if path == "ring" or c["acc"] != "fp32" else rng.choice(["bf16", "bf16", "fp32"])
    return c


# ---- inputs ------------------------------------------------------------------------------

def _gen(seed, *more):
    g = torch.Generator(device="cuda")
    s = seed
    for v in more:
        s = s * 1_000_003 + v
    g.manual_seed(s % (1 << 62))
    return g


def _features(case, seed):
    """The block's features of enormous range (Fig. 1 of the paper) and the k that stay bf16:
    those first, then others as a calibration run fills up with."""
    perm = torch.randperm(case["E"], generator=_gen(seed, 1), device="cuda")
    wide = perm[: max(1, case["E"] // 150)]
    return wide, perm[: case["k"]].sort().values.to(torch.int32)


def _activations(case, T, wide, seed, rank):
    """bf16 [T, E]: unit-scale features with heavy tails, the wide ones 30 to 100 times larger."""
    g = _gen(seed, 2, rank)
    x = torch.randn((T, case["E"]), generator=g, device="cuda")
    tail = torch.randn((T, 1), generator=g, device="cuda").abs_().add_(0.3)
    x.mul_(tail)
    x[:, wide] *= torch.rand(wide.numel(), generator=g, device="cuda") * 70.0 + 30.0
    return x.to(torch.bfloat16)


class _Msgs:
    """The messages of n ranks, each section of all ranks in one buffer (as an all-gather
    delivers them); pad bytes start as zero."""

    def __init__(self, L, n, T):
        self.L, self.n, self.T = L, n, T
        self.sections = {}
        self.msgs = [tpq.Message(L, 0, "cuda") for _ in range(n)]
        for name, pitch in (("codes", L.pitch_codes), ("scale", L.pitch_meta), ("zero", L.pitch_meta),
                            ("outl", L.pitch_outl)):
            buf = torch.zeros((n, max(int(pitch) * T, 16)), dtype=torch.uint8, device="cuda")
            self.sections[name] = buf if name == "codes" else buf.view(torch.bfloat16)
            for i, m in enumerate(self.msgs):
                setattr(m, name, buf[i])
                m.T = T

    def outputs(self, rows=None):
        return {k: v[:rows] for k, v in self.sections.items()}


def prepare(case, seed):
    path, N, T, E, k = case["path"], case["N"], case["T"], case["E"], case["k"]
    L = tpq.layout_init(E, k, case["G"], case["bits"])
    wide, idx = _features(case, seed)
    s = dict(case=case, L=L)
    if path == "calibrate":
        s["seqs"] = [_activations(case, T, wide, seed, q) for q in range(case["seqs"])]
        # the other devices' calibration state, as gathered
        g = _gen(seed, 3)
        s["M"] = torch.randn((N, E), generator=g, device="cuda").abs_() + 2.0
        s["m"] = -(torch.randn((N, E), generator=g, device="cuda").abs_() + 2.0)
        s["ws"] = tpq.calibrate_workspace(T, E, "cuda")
        s["wsf"] = torch.empty(tpq.calibrate_finalize_workspace_bytes(E), dtype=torch.uint8, device="cuda")
        s["Rbar"] = torch.empty(E, device="cuda")
        s["idx"] = torch.zeros(max(k, 4), dtype=torch.int32, device="cuda")
        return s
    plan = tpq.plan_build(L, idx if k else torch.zeros(4, dtype=torch.int32, device="cuda"))
    s["plan"] = plan
    msgs = _Msgs(L, N, T)
    s["msgs"], s["m"] = msgs, msgs.msgs
    if path != "ring":
        s["out"] = torch.empty((T, E), dtype=OUT[case["out"]], device="cuda")
    if path in ("reduce", "static"):
        s["Y"] = [_activations(case, T, wide, seed, i) for i in range(N)]
    if path == "static":
        lo = torch.stack([y.amin(0).float() for y in s["Y"]])
        hi = torch.stack([y.amax(0).float() for y in s["Y"]])
        s["step"], s["inv"] = tpq.static_params(L, plan, 0.8 * lo, 0.8 * hi)  # (ranges of another sample)
    if path in ("device", "decode", "linear"):
        # rank 0 is this device; the others' messages are what the all-gather has brought
        for i in range(1, N):
            tpq.encode(L, plan, [_activations(case, T, wide, seed, i)], [s["m"][i]])
        s["residual"] = torch.randn((T, E), generator=_gen(seed, 4), device="cuda").to(torch.bfloat16)
        s["bias"] = torch.randn(E, generator=_gen(seed, 5), device="cuda").to(torch.bfloat16)
    if path in ("device", "decode"):
        s["Y"] = [_activations(case, T, wide, seed, 0)]
    if path == "decode":
        s["enc"] = tpq.encode_call(L, plan, s["Y"], s["m"][:1])
        s["dec"] = tpq.decode_reduce_call(L, plan, s["m"], s["out"], ACC[case["acc"]])
    if path == "linear":
        g = _gen(seed, 6)
        s["X"] = torch.randn((T, case["K"]), generator=g, device="cuda").to(torch.bfloat16)
        W = torch.randn((E, case["K"]), generator=g, device="cuda") / math.sqrt(case["K"])
        W[wide] *= 30.0
        s["Wp"] = tpq.gemm_weights(L, plan, W.to(torch.bfloat16))
    if path == "ring":
        s["Y"] = [_activations(case, T, wide, seed, i) for i in range(N)]
        s["received"] = _Msgs(L, N, T)
        tpq.encode(L, plan, s["Y"][1:] + s["Y"][:1], s["received"].msgs)
    return s


# ---- one pass ------------------------------------------------------------------------------

def run(s):
    case, L = s["case"], s["L"]
    path = case["path"]
    if path == "calibrate":
        for q, y in enumerate(s["seqs"]):
            tpq.calibrate(y, 0, case["N"], q, 0.01, s["m"], s["M"], s["ws"])
        tpq.calibrate_finalize(s["m"], s["M"], case["k"], s["Rbar"], s["idx"], None, s["wsf"])
        plan = tpq.plan_build(L, s["idx"])
        step, inv = tpq.static_params(L, plan, s["m"], s["M"])
        return [s["m"], s["M"], s["Rbar"], s["idx"], step, inv]
    if path == "decode":
        s["enc"]()
        s["dec"]()
        return [s["msgs"].outputs(1), s["out"]]
    plan, acc = s["plan"], ACC[case["acc"]]
    if path == "reduce":
        tpq.encode(L, plan, s["Y"], s["m"])
        tpq.decode_reduce(L, plan, s["m"], s["out"], acc)
        return [s["msgs"].outputs(), s["out"]]
    if path == "static":
        tpq.encode_static(L, plan, s["Y"], s["inv"], s["m"])
        tpq.decode_reduce_static(L, plan, s["m"], s["step"], s["out"], acc)
        return [s["msgs"].outputs(), s["out"]]
    if path == "ring":
        tpq.hop(L, plan, s["Y"], s["received"].msgs, s["m"], acc)
        return [s["msgs"].outputs()]
    if path == "device":
        tpq.encode(L, plan, s["Y"], s["m"][:1])
    else:
        tpq.gemm_encode(L, s["X"], s["Wp"], s["m"][0])
    tpq.decode_reduce_fused(L, plan, s["m"], s["out"], s["residual"], s["bias"], acc)
    return [s["msgs"].outputs(1), s["out"]]


# ---- what a pass cannot do without ---------------------------------------------------------

def work(case):
    path, N, T, E, k = case["path"], case["N"], case["T"], case["E"], case["k"]
    L = tpq.layout_init(E, k, case["G"], case["bits"])
    W = L.code_bytes + 2 * k if path == "static" else L.wire_bytes_per_row   # bytes a row of a message
    ob = 4 if case.get("out") == "fp32" else 2
    y = 2 * T * E                                                            # a bf16 [T, E]
    if path == "calibrate":
        r8 = 8 * N * (E - k)                                                 # step and inv
        return {"bytes": case["seqs"] * y + 8 * N * E + 8 * E + 4 * E + 4 * k + r8, "flops": case["seqs"] * 2 * T * E}
    decode = T * (N * W + ob * E)
    ops = 3 * N * T * E
    if path in ("reduce", "static"):
        return {"bytes": N * (y + T * W) + decode, "flops": ops + 4 * N * T * E}
    if path == "ring":
        return {"bytes": N * (y + 2 * T * W), "flops": 7 * N * T * E}
    extra = 0 if path == "decode" else y + 2 * E                             # residual and bias
    if path == "linear":
        K = case["K"]
        return {"bytes": 2 * T * K + 2 * E * K + T * W + decode + extra, "flops": 2 * T * E * K + ops + 4 * T * E}
    return {"bytes": y + T * W + decode + extra, "flops": ops + 4 * T * E}


def tolerance(case):
    """Codes, scales, zeros and sums are fixed to the bit (the order of the additions is part of
    the interface), except behind the linear layer: its fp32 sum over K may be taken in any
    order, which moves a bf16 product by one unit in the last place where it lies next to a
    rounding boundary, and with it a code, or a group's range and all its codes.  Against the
    product summed in float64: rel 1.3e-4 at most (over the four sections and the sums; one
    flipped minimum among few groups is more), max 0.034 (a code step), 2.7e-5 of the code bytes
    (a single byte is 2e-3 of the smallest message)."""
    if case["path"] == "linear":
        return {"rel": 2e-3, "max": 0.15, "differ": 4e-3}
    return "exact"
