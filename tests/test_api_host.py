"""Host-side logic of the C ABI: exports, layout arithmetic, argument validation.

No compute call is made here: every call below either fails its argument check
(detected before anything is enqueued) or has nothing to do (T = 0), so the fake
pointers are never dereferenced and the tests run without a GPU.
"""
import collections
import ctypes
import gc
import os
import re
import subprocess
import sys
import weakref

import pytest
import torch

import paper_2411_07942_amd as tpq
from refmath import payload_bits, wire_bytes_per_row

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "tpq.h")).read()
    declared = set(re.findall(r"\b(tpq_[a-z_]+)\s*\(", header))
    assert declared == set(tpq.EXPORTS)
    lib = tpq._load()
    for name in declared:
        assert hasattr(lib, name), name


@pytest.mark.parametrize("E,k,G,W,pb,wb", [
    (512, 8, 128, 284, 4.1875, 4.4375),
    (5120, 80, 128, 2840, 4.1875, 4.4375),
    (4608, 72, 128, 2556, 4.1875, 4.4375),
    (8192, 128, 128, 4540, 4.1875, 4.43359375),
    (8192, 128, 64, 4792, 4.1875, 4.6796875),
    (8192, 341, 128, 4856, None, 4.7421875),
    (8192, 341, 64, 5100, None, 4.98046875),
])
def test_layout_closed_forms(E, k, G, W, pb, wb):
    """Bits per value: 4 + 12k/E (paper abstract / Sec. 4); wire adds scale + zero."""
    L = tpq.layout_init(E, k, G)
    assert (L.r, L.ng, L.code_bytes) == (E - k, -(-(E - k) // G), (E - k + 1) // 2)
    assert L.wire_bytes_per_row == W == wire_bytes_per_row(E, k, G)
    assert tpq.payload_bits(L) == payload_bits(E, k) == 4 + 12 * k / E
    if pb is not None:
        assert tpq.payload_bits(L) == pb < 4.2
    assert tpq.wire_bits(L) == wb == 8 * W / E
    for p in (L.pitch_codes, L.pitch_meta, L.pitch_outl):
        assert p % 16 == 0
    assert L.pitch_codes >= L.code_bytes and L.pitch_meta >= 2 * L.ng and L.pitch_outl >= 2 * k
    assert tpq.plan_bytes(L) >= 64 + 4 * k + 2 * (E - k)


@pytest.mark.parametrize("b", [2, 3, 4, 5, 6, 8])
@pytest.mark.parametrize("E,k,G", [(512, 8, 128), (5120, 80, 128), (1032, 1, 64), (64, 64, 32)])
def test_layout_other_widths(E, k, G, b):
    """b bits for the quantised features (Sec. 4, Fig. 3): b + (16 - b) k / E per value."""
    L = tpq.layout_init(E, k, G, b)
    r = E - k
    assert (L.bits, L.r, L.ng, L.code_bytes) == (b, r, -(-r // G), (r * b + 7) // 8)
    assert tpq.payload_bits(L) == b + (16 - b) * k / E
    assert L.wire_bytes_per_row == 2 * k + L.code_bytes + 4 * L.ng
    assert L.pitch_codes % 16 == 0 and L.pitch_codes >= L.code_bytes
    if b != 4 and r > 0:     # whole chunks are stored, 8 bytes are read from the start of each
        assert L.pitch_codes >= -(-r // 8) * b + 8


def test_k_floor_E_over_64_is_under_4p2_bits():
    for E in (512, 4096, 4608, 5120, 8192, 16384):
        assert tpq.payload_bits(tpq.layout_init(E, E // 64, 128)) < 4.2


@pytest.mark.parametrize("args,code", [
    ((512, 8, 128, 7), tpq.ERR_UNSUPPORTED),
    ((512, 8, 128, 1), tpq.ERR_UNSUPPORTED),
    ((512, 8, 128, 16), tpq.ERR_UNSUPPORTED),
    ((512, 8, 100, 4), tpq.ERR_UNSUPPORTED),
    ((512, 8, 16, 4), tpq.ERR_UNSUPPORTED),
    ((500, 8, 128, 4), tpq.ERR_SHAPE),
    ((0, 0, 128, 4), tpq.ERR_SHAPE),
    ((512, 513, 128, 4), tpq.ERR_SHAPE),
    ((512, -1, 128, 4), tpq.ERR_SHAPE),
    ((tpq.MAX_E + 8, 0, 128, 4), tpq.ERR_SHAPE),
])
def test_layout_init_rejects(args, code):
    with pytest.raises(tpq.TpqError) as e:
        tpq.layout_init(*args)
    assert e.value.code == code


def _fake(addr=0x10000):
    return ctypes.c_void_p(addr)


def _ptrs(n, addr=0x10000):
    arr = (ctypes.c_void_p * n)()
    for i in range(n):
        arr[i] = addr + 0x1000 * i
    return arr


def test_encode_argument_errors():
    lib = tpq._load()
    L = tpq.layout_init(512, 8, 128)
    LP = ctypes.byref(L)
    ok = dict(plan=_fake(), Y=_ptrs(2), ldY=512, n=2, T=4, c=_ptrs(2), s=_ptrs(2), z=_ptrs(2), o=_ptrs(2))

    def call(**kw):
        a = dict(ok, **kw)
        return lib.tpq_encode(a.get("L", LP), a["plan"], a["Y"], a["ldY"], a["n"], a["T"], a["c"],
                              a["s"], a["z"], a["o"], None)
    assert call(L=None) == tpq.ERR_NULL
    assert call(plan=None) == tpq.ERR_NULL
    assert call(Y=None) == tpq.ERR_NULL
    assert call(c=None) == tpq.ERR_NULL
    assert call(o=None) == tpq.ERR_NULL
    assert call(n=0) == tpq.ERR_SHAPE
    assert call(n=tpq.MAX_RANKS + 1) == tpq.ERR_SHAPE
    assert call(T=-1) == tpq.ERR_SHAPE
    assert call(ldY=504) == tpq.ERR_SHAPE
    assert call(ldY=516) == tpq.ERR_ALIGN
    assert call(plan=_fake(0x10008)) == tpq.ERR_ALIGN
    assert call(Y=_ptrs(2, 0x10002)) == tpq.ERR_ALIGN
    hole = _ptrs(2)
    hole[1] = None
    assert call(z=hole) == tpq.ERR_NULL
    assert call(T=0) == tpq.OK                      # nothing to do, nothing enqueued
    # a layout whose derived fields were tampered with is refused
    bad = tpq.layout_init(512, 8, 128)
    bad.ng = 3
    assert call(L=ctypes.byref(bad)) == tpq.ERR_SHAPE
    bad = tpq.layout_init(512, 8, 128)
    bad.pitch_codes = 250
    assert call(L=ctypes.byref(bad)) == tpq.ERR_ALIGN
    bad.pitch_codes = 240
    assert call(L=ctypes.byref(bad)) == tpq.ERR_SHAPE


def test_decode_argument_errors():
    lib = tpq._load()
    L = tpq.layout_init(512, 8, 128)
    LP = ctypes.byref(L)
    ok = dict(plan=_fake(), n=2, T=4, c=_ptrs(2), s=_ptrs(2), z=_ptrs(2), o=_ptrs(2), acc=0, od=0,
              out=_fake(0x90000), ld=512)

    def call(**kw):
        a = dict(ok, **kw)
        return lib.tpq_decode_reduce(LP, a["plan"], a["n"], a["T"], a["c"], a["s"], a["z"], a["o"],
                                     a["acc"], a["od"], a["out"], a["ld"], None)
    assert call(acc=3) == tpq.ERR_UNSUPPORTED  # 0, 1, 2 are the modes
    assert call(od=3) == tpq.ERR_UNSUPPORTED
    assert call(out=None) == tpq.ERR_NULL
    assert call(out=_fake(0x90004)) == tpq.ERR_ALIGN
    assert call(ld=500) == tpq.ERR_SHAPE
    assert call(ld=516) == tpq.ERR_ALIGN
    assert call(ld=518, od=1) == tpq.ERR_ALIGN      # fp32 rows: multiples of 4 elements
    assert call(n=65) == tpq.ERR_SHAPE
    assert call(s=None) == tpq.ERR_NULL
    assert call(T=0) == tpq.OK


@pytest.mark.parametrize("G,most", [(32, 65535 * 128), (128, 65535 * 128), (256, 65535 * 64)])
def test_linear_layer_refuses_more_rows_than_it_states(G, most):
    """With a misaligned message, so that nothing is enqueued for a row count that is taken either."""
    lib = tpq._load()
    L = tpq.layout_init(512, 8, G)
    for T, want in ((most, tpq.ERR_ALIGN), (most + 1, tpq.ERR_SHAPE), (1 << 26, tpq.ERR_SHAPE)):
        assert lib.tpq_gemm_encode(ctypes.byref(L), _fake(), T, 8, 8, _fake(), _fake(0x10008), _fake(), _fake(), _fake(),
                                   None, 0, None) == want


def test_calibrate_and_plan_argument_errors():
    lib = tpq._load()
    f = _fake
    assert tpq.calibrate_workspace_bytes(16384, 4608) > 0
    assert tpq.calibrate_workspace_bytes(16384, 4609) == 0
    ws = tpq.calibrate_workspace_bytes(64, 512)
    call = lib.tpq_calibrate
    assert call(None, 64, 512, 512, 0, 4, 0, 0.01, f(), f(), f(), ws, None) == tpq.ERR_NULL
    assert call(f(), 64, 512, 512, 4, 4, 0, 0.01, f(), f(), f(), ws, None) == tpq.ERR_SHAPE
    assert call(f(), 64, 512, 512, 0, 4, -1, 0.01, f(), f(), f(), ws, None) == tpq.ERR_SHAPE
    assert call(f(), 64, 512, 512, 0, 4, 0, 1.5, f(), f(), f(), ws, None) == tpq.ERR_SHAPE
    assert call(f(), 64, 500, 512, 0, 4, 0, 0.01, f(), f(), f(), ws, None) == tpq.ERR_SHAPE
    assert call(f(), 64, 520, 512, 0, 4, 0, 0.01, f(), f(), f(), ws - 1, None) == tpq.ERR_WORKSPACE
    assert call(f(0x10002), 64, 512, 512, 0, 4, 0, 0.01, f(), f(), f(), ws, None) == tpq.ERR_ALIGN
    assert call(f(), 0, 512, 512, 0, 4, 0, 0.01, f(), f(), f(), ws, None) == tpq.OK
    fin = lib.tpq_calibrate_finalize
    wsf = tpq.calibrate_finalize_workspace_bytes(512)
    assert fin(f(), f(), 4, 512, 513, None, f(), f(), None, f(), wsf, None) == tpq.ERR_SHAPE
    assert fin(f(), f(), 4, 512, 8, None, None, f(), None, f(), wsf, None) == tpq.ERR_NULL
    assert fin(f(), f(), 4, 512, 8, None, f(), f(), None, f(), wsf - 1, None) == tpq.ERR_WORKSPACE
    L = tpq.layout_init(512, 8, 128)
    assert lib.tpq_plan_build(ctypes.byref(L), f(), f(), tpq.plan_bytes(L) - 1, None) == tpq.ERR_WORKSPACE
    assert lib.tpq_plan_build(ctypes.byref(L), None, f(), tpq.plan_bytes(L), None) == tpq.ERR_NULL
    assert lib.tpq_plan_build(ctypes.byref(L), f(), f(0x10004), tpq.plan_bytes(L), None) == tpq.ERR_ALIGN


class _NullStream:
    cuda_stream = 0


@pytest.mark.parametrize("seq", [list, tuple])
def test_binding_checks_tensors_before_anything_is_enqueued(seq):
    """The native half of the binding: what the Python entry points assert (types, shapes, strides),
    the library's own errors as TpqError, immediate and marshalled calls alike."""
    E, T = 512, 4
    L = tpq.layout_init(E, 8, 128)
    plan = torch.zeros(tpq.plan_bytes(L), dtype=torch.uint8)
    Y = [torch.zeros((T, E), dtype=torch.bfloat16) for _ in range(3)]
    msgs = [tpq.Message(L, T, "cpu") for _ in range(3)]
    out = torch.zeros((T, E), dtype=torch.float32)
    bad = {"dtype": torch.zeros((T, E)), "shape": Y[0][:3], "columns": torch.zeros((E, T), dtype=torch.bfloat16).t(),
           "row stride": torch.zeros((T, E + 8), dtype=torch.bfloat16)[:, :E]}
    for what, y in bad.items():
        for f in (lambda: tpq.encode(L, plan, seq([Y[0], y]), seq(msgs[:2]), stream=_NullStream()),
                  lambda: tpq.encode_call(L, plan, seq([Y[0], y]), seq(msgs[:2]))):
            with pytest.raises(AssertionError):
                f()
    with pytest.raises(IndexError):
        tpq.encode(L, plan, seq(Y), seq(msgs[:2]), stream=_NullStream())
    with pytest.raises(AssertionError):
        tpq.hop_call(L, plan, seq(Y), seq(msgs[:2]), seq(msgs))
    with pytest.raises(AssertionError):
        tpq.decode_reduce(L, plan, seq(msgs), out.double(), stream=_NullStream())
    with pytest.raises(AssertionError):
        tpq.decode_reduce_fused(L, plan, seq(msgs), out, addend=out, stream=_NullStream())
    with pytest.raises(AssertionError):
        tpq.decode_reduce_static(L, plan, seq(msgs), out[:2], out, stream=_NullStream())
    with pytest.raises(AssertionError):
        tpq.gemm_encode_call(L, Y[0], torch.zeros((E, 8), dtype=torch.bfloat16), msgs[0])
    with pytest.raises(TypeError):
        tpq.encode(L, plan, seq([1.0]), seq(msgs), stream=_NullStream())
    # the library's answer: more ranks than it takes, an accumulate mode it does not know
    many = seq([msgs[0]] * (tpq.MAX_RANKS + 1))
    for f in (lambda: tpq.decode_reduce(L, plan, many, out, stream=_NullStream()),
              lambda: tpq.decode_reduce_call(L, plan, many, out)(_NullStream())):
        with pytest.raises(tpq.TpqError) as e:
            f()
        assert e.value.code == tpq.ERR_SHAPE
    with pytest.raises(tpq.TpqError) as e:
        tpq.decode_reduce_call(L, plan, seq(msgs), out, 7)(stream=_NullStream())
    assert e.value.code == tpq.ERR_UNSUPPORTED
    with pytest.raises(TypeError):
        tpq.decode_reduce_call(L, plan, seq(msgs), out)(1, 2)


def _binding_case(T=4, E=512):
    L = tpq.layout_init(E, 8, 128)
    plan = torch.zeros(tpq.plan_bytes(L), dtype=torch.uint8)
    return (L, plan, [torch.zeros((T, E), dtype=torch.bfloat16) for _ in range(2)],
            [tpq.Message(L, T, "cpu") for _ in range(2)])


def _without_address(what):
    """Each ends the process if the binding trusts the tensor (run in a process of its own)."""
    L, plan, Y, msgs = _binding_case()
    sparse = torch.zeros((4, 512), dtype=torch.bfloat16).to_sparse()
    state = torch.zeros((2, 512))
    if what == "section":
        msgs[0].codes = sparse
        tpq.encode_call(L, plan, Y, msgs)
    elif what == "plan":
        tpq.decode_reduce(L, sparse, msgs, torch.zeros((4, 512)), stream=_NullStream())
    elif what == "plan to build":
        tpq.plan_build(L, torch.zeros(8, dtype=torch.int32), sparse, stream=_NullStream())
    elif what == "no plan":
        tpq._native().plan_build(L, torch.zeros(8, dtype=torch.int32), None, _NullStream())
    elif what == "calibrate":
        tpq.calibrate(sparse, 0, 2, 0, 0.01, state, state, tpq.calibrate_workspace(4, 512, "cpu"), stream=_NullStream())
    elif what == "calibrate_fixed":
        tpq.calibrate_fixed(sparse, 0, 2, 0, 0.01, state, state, stream=_NullStream())
    elif what == "proxy":
        tpq.encode_call(L, plan, [weakref.proxy(y) for y in Y], msgs)
    elif what == "vmap":
        torch.vmap(lambda y: tpq.encode(L, plan, [y], msgs, stream=_NullStream()))(torch.stack(Y))
    elif what == "jvp":
        torch.func.jvp(lambda y: tpq.encode_call(L, plan, [y], msgs), (Y[0],), (Y[1],))


@pytest.mark.parametrize("what", ["section", "plan", "plan to build", "no plan", "calibrate", "calibrate_fixed", "proxy", "vmap",
                                  "jvp"])
def test_binding_raises_where_a_tensor_has_no_address(what):
    code = ("import sys; sys.path[:0] = %r\nimport test_api_host as t\ntry:\n    t._without_address(%r)\n"
            "except (RuntimeError, TypeError) as e:\n    print('raised', e)" % ([ROOT, os.path.join(ROOT, "tests")], what))
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("raised"), (r.returncode, r.stdout, r.stderr[-400:])


class _Made:
    """A sequence whose elements exist only while someone holds them."""

    def __init__(self, make):
        self.make = make

    def __len__(self):
        return 2

    def __getitem__(self, i):
        if i >= 2:
            raise IndexError(i)
        return self.make()


@pytest.mark.parametrize("seq", [list, tuple, collections.deque, _Made])
def test_marshalled_calls_keep_what_they_point_to(seq):
    """A call's tensors and messages live as long as it does, whatever sequence they came in."""
    L, plan, _, _ = _binding_case()
    alive = []

    def tensor():
        t = torch.zeros((4, 512), dtype=torch.bfloat16)
        alive.append(weakref.ref(t))
        return t

    def message():
        m = tpq.Message(L, 4, "cpu")
        alive.append(weakref.ref(m))
        return m
    if seq is _Made:
        Y, msgs = _Made(tensor), _Made(message)
    else:
        Y, msgs = (seq([f(), f()]) for f in (tensor, message))
    call = tpq.encode_call(L, plan, Y, msgs)
    for s in (Y, msgs):
        if hasattr(s, "clear"):
            s.clear()
    del Y, msgs, s
    assert len(alive) == 4 and all(r() is not None for r in alive)
    del call
    assert all(r() is None for r in alive)


def test_what_has_an_address_and_rows_is_taken():
    """Objects with a data_ptr() (a storage, a tensor subclass with its own) and dimensions past rows and columns."""
    class Elsewhere(torch.Tensor):
        def data_ptr(self):
            return self.address

    L, plan, Y, msgs = _binding_case()
    out = torch.zeros((4, 512, 1))
    tpq.encode_call(L, plan.untyped_storage(), [y.unsqueeze(-1) for y in Y], msgs)
    tpq.decode_reduce_call(L, plan.untyped_storage(), msgs, out)
    tpq.gemm_encode_call(L, Y[0][:, :8], torch.zeros((512, 8), dtype=torch.bfloat16), msgs[0], Y[0].unsqueeze(-1))
    with pytest.raises(AssertionError):
        tpq.encode_call(L, plan, [Y[0].unsqueeze(-1), Y[1]], msgs)
    with pytest.raises(AttributeError):
        tpq.encode_call(L, 1.0, Y, msgs)
    for address, code in ((0x10008, tpq.ERR_ALIGN), (0, tpq.ERR_NULL)):
        for m in msgs:
            m.codes = m.codes.as_subclass(Elsewhere)
            m.codes.address = address
        with pytest.raises(tpq.TpqError) as e:
            tpq.decode_reduce(L, plan, msgs, out, stream=_NullStream())
        assert e.value.code == code


def test_a_message_that_holds_its_own_call_is_collected():
    L, plan, Y, msgs = _binding_case()
    msgs[0].call = tpq.encode_call(L, plan, Y, msgs)
    held = weakref.ref(msgs[0])
    del msgs
    gc.collect()
    assert held() is None


@pytest.mark.parametrize("no_sequence", [iter, set, lambda y: (t for t in y), lambda y: dict(enumerate(y))])
def test_what_is_no_sequence_is_refused(no_sequence):
    L, plan, Y, msgs = _binding_case()
    for f in (lambda: tpq.encode_call(L, plan, no_sequence(Y), msgs),
              lambda: tpq.encode(L, plan, no_sequence(Y), msgs, stream=_NullStream())):
        with pytest.raises(TypeError):
            f()
    # a tensor is one: a row per rank
    tpq.encode_call(L, plan, torch.stack(Y), msgs)


def test_strerror_covers_every_code():
    lib = tpq._load()
    seen = set()
    for code in range(0, -8, -1):
        s = lib.tpq_strerror(code).decode()
        assert s and s != "unknown error"
        seen.add(s)
    assert len(seen) == 8
    assert lib.tpq_strerror(-99).decode() == "unknown error"


def test_bench_refuses_more_than_one_gpu():
    """bench.py measures one GPU; asking for more ends with a message, before anything runs."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    p = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert p.returncode != 0
    assert "one GPU" in (p.stdout + p.stderr)
