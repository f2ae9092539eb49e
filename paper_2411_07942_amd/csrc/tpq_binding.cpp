// Native half of the Python binding: takes the tensors apart, checks what the Python entry points
// promise to check, and issues the C ABI call on the current stream.
//
// Why it is native: a small block's kernels take 4 to 5 us, a launch costs the host 2.5 to 3.8 us,
// and marshalling the same call through ctypes cost more than both -- 13 to 16 us for tpq.encode of
// 4 to 8 ranks (40 data_ptr() calls and as many checks, current_stream() 2.6 us, argument
// conversion), so that the host was what a decode step waited for.  Here encode takes 3.6 us
// including the launch, and an already marshalled call 3.0 (7.2 before).
#include <Python.h>
#include <structmember.h>

#include <string.h>

#include <exception>
#include <new>
#include <vector>

#include <torch/csrc/autograd/python_variable.h>

#include "tpq.h"

namespace {

PyObject *g_check;         // Python: raises TpqError for a code that is not TPQ_OK
PyObject *g_get_device;    // torch._C._cuda_getDevice
PyObject *g_get_stream;    // torch._C._cuda_getCurrentRawStream
PyObject *s_codes, *s_scale, *s_zero, *s_outl, *s_cuda_stream, *s_stream, *s_data_ptr;

// ---- at the boundary to C ------------------------------------------------------------------

struct Ref {  // an owned reference
    PyObject *p;
    explicit Ref(PyObject *o = nullptr) : p(o) {}
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
    ~Ref() { Py_XDECREF(p); }
};

struct WithoutGil {
    PyThreadState *state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

// torch throws where a tensor has no address or no strides (sparse, or wrapped by a transform that is
// tracing or batching it): the exception becomes Python's here, or it would end the process
// in the interpreter's C frames.
template <typename F>
PyObject *no_throw(F &&f)
{
    try {
        return f();
    } catch (const std::bad_alloc &) {
        PyErr_NoMemory();
    } catch (const c10::Error &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception");
    }
    return nullptr;
}

// ---- pieces of an argument list ---------------------------------------------------------

bool failed_check(const char *what)
{
    PyErr_SetString(PyExc_AssertionError, what);
    return false;
}

const at::Tensor *tensor(PyObject *o)
{
    // (by its real type: isinstance() also holds for a weak reference's proxy, which has no tensor inside)
    if (!THPVariable_CheckExact(o) && !PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject *>(THPVariableClass))) {
        PyErr_SetString(PyExc_TypeError, "a torch.Tensor is expected");
        return nullptr;
    }
    return &THPVariable_Unpack(o);
}

bool pointer(PyObject *o, void *&p)  // None: null; any object with a data_ptr() (a storage, say) has an address
{
    p = nullptr;
    if (o == Py_None) return true;
    if (THPVariable_CheckExact(o)) {
        p = THPVariable_Unpack(o).data_ptr();
        return true;
    }
    const Ref a(PyObject_CallMethodNoArgs(o, s_data_ptr));
    if (!a.p) return false;
    p = PyLong_AsVoidPtr(a.p);
    return !PyErr_Occurred();
}

struct Pointers {
    void *small[TPQ_MAX_RANKS];
    std::vector<void *> large;  // (more ranks than the library takes: it refuses the call)
    void **p = nullptr;
    void resize(size_t n)
    {
        if (n <= TPQ_MAX_RANKS) {
            p = small;
        } else {
            large.resize(n);
            p = large.data();
        }
    }
};

// What a call was given, held by value: a sequence as a tuple of its elements at that time, so that neither
// a list emptied later nor elements made on the way leave pointers to freed memory behind.
struct Kept {
    PyObject *p = nullptr;
    Kept() = default;
    Kept(const Kept &) = delete;
    Kept &operator=(const Kept &) = delete;
    ~Kept() { Py_XDECREF(p); }
    void object(PyObject *o)
    {
        Py_INCREF(o);
        Py_XSETREF(p, o);
    }
    bool sequence(PyObject *o)
    {
        // (what len() and indexing take; a generator or a set is refused)
        if (PyObject_Size(o) < 0) return false;
        if (!PySequence_Check(o) && !PyMapping_Check(o)) {
            PyErr_Format(PyExc_TypeError, "a sequence is expected, not %s", Py_TYPE(o)->tp_name);
            return false;
        }
        PyObject *t = PySequence_Tuple(o);
        if (!t) return false;
        Py_XSETREF(p, t);
        return true;
    }
};

struct Sequence {  // the elements of a tuple that is kept elsewhere
    Py_ssize_t n = 0;
    PyObject **item = nullptr;
    bool take(PyObject *o, Kept &kept)
    {
        if (!kept.sequence(o)) return false;
        n = PyTuple_GET_SIZE(kept.p);
        item = PySequence_Fast_ITEMS(kept.p);
        return true;
    }
};

bool sections(const Sequence &msgs, Py_ssize_t n, PyObject *name, Pointers &dst)
{
    if (msgs.n < n) {
        PyErr_SetString(PyExc_IndexError, "fewer messages than ranks");
        return false;
    }
    dst.resize(static_cast<size_t>(n));
    for (Py_ssize_t i = 0; i < n; ++i) {
        const Ref t(PyObject_GetAttr(msgs.item[i], name));
        if (!t.p || !pointer(t.p, dst.p[i])) return false;
    }
    return true;
}

// row stride of a [T, >= E] tensor: what a single row's stride says does not matter
int64_t row_stride(const at::Tensor &t, int64_t T, int64_t E)
{
    const int64_t s = t.stride(0);
    return T > 1 ? s : (s > E ? s : E);
}

// the ranks' partial sums: bf16, one shape, unit column stride, one row stride (dimensions past the second are
// the caller's, here and for the outputs: a [T, E, 1] is rows and columns too)
bool partial_sums(const Sequence &Y, int64_t E, Pointers &dst, int64_t &T, int64_t &ld)
{
    dst.resize(static_cast<size_t>(Y.n));
    if (Y.n == 0) {
        PyErr_SetString(PyExc_IndexError, "no partial sums");
        return false;
    }
    const at::Tensor *first = nullptr;
    for (Py_ssize_t i = 0; i < Y.n; ++i) {
        const at::Tensor *y = tensor(Y.item[i]);
        if (!y) return false;
        if (i == 0) {
            if (y->dim() < 2) return failed_check("partial sums have rows and columns");
            first = y;
            T = y->size(0);
            ld = row_stride(*y, T, E);
        }
        if (y->scalar_type() != at::kBFloat16 || y->sizes() != first->sizes() || y->stride(1) != 1 || (T > 1 && y->stride(0) != ld))
            return failed_check("partial sums are bf16 tensors of one shape and row stride, unit column stride");
        if (!pointer(Y.item[i], dst.p[i])) return false;
    }
    return true;
}

bool out_tensor(PyObject *o, int64_t E, int64_t &T, int &dtype, void *&p, int64_t &ld)
{
    const at::Tensor *t = tensor(o);
    if (!t) return false;
    if ((t->scalar_type() != at::kFloat && t->scalar_type() != at::kBFloat16) || t->dim() < 2 || t->stride(1) != 1)
        return failed_check("out is a bf16 or fp32 matrix with unit column stride");
    T = t->size(0);
    dtype = t->scalar_type() == at::kFloat ? TPQ_OUT_FP32 : TPQ_OUT_BF16;
    ld = row_stride(*t, T, E);
    return pointer(o, p);
}

bool table(PyObject *o, Py_ssize_t n, const float *&p)  // step or inv: fp32, contiguous, a row per rank
{
    const at::Tensor *t = tensor(o);
    if (!t) return false;
    if (t->scalar_type() != at::kFloat || !t->is_contiguous() || t->dim() < 1 || t->size(0) < n)
        return failed_check("the step table is a contiguous fp32 tensor with a row per rank");
    void *v;
    if (!pointer(o, v)) return false;
    p = static_cast<const float *>(v);
    return true;
}

bool stream_of(PyObject *o, void *&s)
{
    PyObject *v;
    if (o == Py_None) {
        PyObject *dev = PyObject_CallNoArgs(g_get_device);
        if (!dev) return false;
        v = PyObject_CallOneArg(g_get_stream, dev);
        Py_DECREF(dev);
    } else {
        v = PyObject_GetAttr(o, s_cuda_stream);
    }
    if (!v) return false;
    s = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    return !(s == nullptr && PyErr_Occurred());
}

struct Layout {  // the ctypes structure, by reference
    Py_buffer view;
    const tpq_layout *p = nullptr;
    bool take(PyObject *o)
    {
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return false;
        p = static_cast<const tpq_layout *>(view.buf);
        if (view.len >= static_cast<Py_ssize_t>(sizeof(tpq_layout))) return true;
        PyErr_SetString(PyExc_TypeError, "a Layout is expected");
        return false;
    }
    ~Layout()
    {
        if (p) PyBuffer_Release(&view);
    }
};

bool check(int rc, const char *where)
{
    if (rc == TPQ_OK) return true;
    PyObject *r = PyObject_CallFunction(g_check, "is", rc, where);
    Py_XDECREF(r);
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, where);
    return false;
}

// ---- the calls that can be marshalled once and issued many times -------------------------

enum Kind { kEncode, kHop, kGemm, kDecode, kFused, kEncodeStatic, kDecodeStatic };

constexpr Py_ssize_t kArgs[] = {4, 6, 5, 5, 7, 5, 6}, kMaxArgs = 7;

struct Call {
    Kind kind;
    Kept arg[kMaxArgs];  // every argument, as it was taken
    Layout L;
    void *plan = nullptr, *out = nullptr, *x = nullptr, *w = nullptr, *addend = nullptr, *bias = nullptr;
    const float *tab = nullptr;
    int n = 0, accum = 0, out_dtype = 0, K = 0;
    int64_t T = 0, ld = 0, ld2 = 0;
    Pointers Y, codes, scale, zero, outl, in_codes, in_scale, in_zero, in_outl;

    bool message(const Sequence &m, Py_ssize_t count, bool meta)
    {
        if (!sections(m, count, s_codes, codes) || !sections(m, count, s_outl, outl)) return false;
        return !meta || (sections(m, count, s_scale, scale) && sections(m, count, s_zero, zero));
    }
    bool accumulate(PyObject *o)
    {
        accum = static_cast<int>(PyLong_AsLong(o));
        return !(accum == -1 && PyErr_Occurred());
    }

    // args: as the Python functions take them, without the stream
    bool take(Kind k, PyObject *const *a)
    {
        kind = k;
        for (Py_ssize_t i = 0; i < kArgs[k]; ++i) arg[i].object(a[i]);
        if (!L.take(a[0])) return false;
        const int64_t E = L.p->E;
        switch (kind) {
        case kEncode: {  // L, plan, Y, msgs
            Sequence y, m;
            if (!pointer(a[1], plan) || !y.take(a[2], arg[2]) || !m.take(a[3], arg[3])) return false;
            n = static_cast<int>(y.n);
            return partial_sums(y, E, Y, T, ld) && message(m, y.n, true);
        }
        case kHop: {  // L, plan, Y, in_msgs, out_msgs, accum
            Sequence y, i, m;
            if (!pointer(a[1], plan) || !y.take(a[2], arg[2]) || !i.take(a[3], arg[3]) || !m.take(a[4], arg[4]) ||
                !accumulate(a[5]))
                return false;
            n = static_cast<int>(y.n);
            if (!partial_sums(y, E, Y, T, ld)) return false;
            if (i.n != y.n || m.n != y.n) return failed_check("a message in and out for every partial sum");
            return sections(i, y.n, s_codes, in_codes) && sections(i, y.n, s_scale, in_scale) &&
                   sections(i, y.n, s_zero, in_zero) && sections(i, y.n, s_outl, in_outl) && message(m, y.n, true);
        }
        case kGemm: {  // L, X, Wp, msg, Y_msg
            const at::Tensor *X = tensor(a[1]), *W = X ? tensor(a[2]) : nullptr;
            if (!W) return false;
            if (X->scalar_type() != at::kBFloat16 || X->dim() != 2 || X->stride(1) != 1)
                return failed_check("X is a bf16 matrix with unit column stride");
            T = X->size(0);
            K = static_cast<int>(X->size(1));
            if (W->scalar_type() != at::kBFloat16 || !W->is_contiguous() || W->dim() != 2 || W->size(0) != E || W->size(1) != K)
                return failed_check("Wp is the contiguous bf16 [E, K] of gemm_weights");
            if (!pointer(a[1], x) || !pointer(a[2], w)) return false;
            ld = row_stride(*X, T, K);
            if (a[4] != Py_None) {
                const at::Tensor *y = tensor(a[4]);
                if (!y) return false;
                if (y->scalar_type() != at::kBFloat16 || y->dim() < 2 || y->size(0) != T || y->stride(1) != 1)
                    return failed_check("Y_msg is a bf16 matrix with a row per token and unit column stride");
                if (!pointer(a[4], out)) return false;
                ld2 = row_stride(*y, T, E);
            }
            Sequence m;
            m.n = 1;
            m.item = &arg[3].p;
            return message(m, 1, true);
        }
        case kDecode:          // L, plan, msgs, out, accum
        case kFused:           // L, plan, msgs, out, addend, bias, accum
        case kDecodeStatic: {  // L, plan, msgs, step, out, accum
            Sequence m;
            if (!pointer(a[1], plan) || !m.take(a[2], arg[2])) return false;
            n = static_cast<int>(m.n);
            if (!out_tensor(a[kind == kDecodeStatic ? 4 : 3], E, T, out_dtype, out, ld)) return false;
            if (!accumulate(a[kind == kDecode ? 4 : kind == kFused ? 6 : 5])) return false;
            if (kind == kDecodeStatic && !table(a[3], m.n, tab)) return false;
            if (kind == kFused && a[4] != Py_None) {
                const at::Tensor *t = tensor(a[4]);
                if (!t) return false;
                if (t->scalar_type() != at::kBFloat16 || t->dim() != 2 || t->size(0) != T || t->size(1) != E || t->stride(1) != 1)
                    return failed_check("addend is a bf16 [T, E] with unit column stride");
                if (!pointer(a[4], addend)) return false;
                ld2 = row_stride(*t, T, E);
            }
            if (kind == kFused && a[5] != Py_None) {
                const at::Tensor *t = tensor(a[5]);
                if (!t) return false;
                if (t->scalar_type() != at::kBFloat16 || t->dim() != 1 || t->size(0) != E || !t->is_contiguous())
                    return failed_check("bias is a contiguous bf16 [E]");
                if (!pointer(a[5], bias)) return false;
            }
            return message(m, m.n, kind != kDecodeStatic);
        }
        case kEncodeStatic: {  // L, plan, Y, inv, msgs
            Sequence y, m;
            if (!pointer(a[1], plan) || !y.take(a[2], arg[2]) || !m.take(a[4], arg[4])) return false;
            n = static_cast<int>(y.n);
            return partial_sums(y, E, Y, T, ld) && table(a[3], y.n, tab) && message(m, y.n, false);
        }
        }
        return false;
    }

    int issue(void *s) const
    {
#define U8(x) reinterpret_cast<uint8_t *const *>((x).p)
#define U16(x) reinterpret_cast<uint16_t *const *>((x).p)
#define CU8(x) reinterpret_cast<const uint8_t *const *>((x).p)
#define CU16(x) reinterpret_cast<const uint16_t *const *>((x).p)
        switch (kind) {
        case kEncode:
            return tpq_encode(L.p, plan, CU16(Y), ld, n, T, U8(codes), U16(scale), U16(zero), U16(outl), s);
        case kHop:
            return tpq_hop(L.p, plan, CU16(Y), ld, n, T, CU8(in_codes), CU16(in_scale), CU16(in_zero), CU16(in_outl), accum,
                           U8(codes), U16(scale), U16(zero), U16(outl), s);
        case kGemm:
            return tpq_gemm_encode(L.p, static_cast<const uint16_t *>(x), T, ld, K, static_cast<const uint16_t *>(w),
                                   static_cast<uint8_t *>(codes.p[0]), static_cast<uint16_t *>(scale.p[0]),
                                   static_cast<uint16_t *>(zero.p[0]), static_cast<uint16_t *>(outl.p[0]),
                                   static_cast<uint16_t *>(out), ld2, s);
        case kDecode:
            return tpq_decode_reduce(L.p, plan, n, T, CU8(codes), CU16(scale), CU16(zero), CU16(outl), accum, out_dtype, out,
                                     ld, s);
        case kFused:
            return tpq_decode_reduce_fused(L.p, plan, n, T, CU8(codes), CU16(scale), CU16(zero), CU16(outl),
                                           static_cast<const uint16_t *>(addend), ld2, static_cast<const uint16_t *>(bias),
                                           accum, out_dtype, out, ld, s);
        case kEncodeStatic:
            return tpq_encode_static(L.p, plan, CU16(Y), ld, n, T, tab, U8(codes), U16(outl), s);
        case kDecodeStatic:
            return tpq_decode_reduce_static(L.p, plan, n, T, CU8(codes), CU16(outl), tab, accum, out_dtype, out, ld, s);
        }
        return TPQ_ERR_UNSUPPORTED;
#undef U8
#undef U16
#undef CU8
#undef CU16
    }

    bool run(PyObject *stream) const
    {
        static const char *const names[] = {"tpq_encode", "tpq_hop", "tpq_gemm_encode", "tpq_decode_reduce",
                                            "tpq_decode_reduce_fused", "tpq_encode_static", "tpq_decode_reduce_static"};
        void *s;
        if (!stream_of(stream, s)) return false;
        const int rc = [&] {
            const WithoutGil free;
            return issue(s);
        }();
        return check(rc, names[kind]);
    }
};

// A marshalled call: callable as call(stream=None).  Holds references to everything it was made of
// (the messages' sections must stay in place).
struct CallObject {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    Call *call;
};

PyObject *call_object_call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames)
{
    const Py_ssize_t nargs = PyVectorcall_NARGS(nargsf), nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    PyObject *stream = nargs > 0 ? args[0] : Py_None;
    if (nargs > 1 || nkw > 1 || (nkw == 1 && (nargs == 1 || PyUnicode_Compare(PyTuple_GET_ITEM(kwnames, 0), s_stream) != 0))) {
        PyErr_SetString(PyExc_TypeError, "call(stream=None)");
        return nullptr;
    }
    if (nkw == 1) stream = args[0];
    const Call *const call = reinterpret_cast<CallObject *>(self)->call;
    if (!call) {
        PyErr_SetString(PyExc_RuntimeError, "the call has been collected");
        return nullptr;
    }
    return no_throw([&]() -> PyObject * {
        if (!call->run(stream)) return nullptr;
        Py_RETURN_NONE;
    });
}

// (a cycle through a message or a module that holds its own calls is the collector's to free)
int call_object_traverse(PyObject *self, visitproc visit, void *arg)
{
    Py_VISIT(Py_TYPE(self));
    if (const Call *c = reinterpret_cast<CallObject *>(self)->call) {
        if (c->L.p) Py_VISIT(c->L.view.obj);
        for (const Kept &k : c->arg) Py_VISIT(k.p);
    }
    return 0;
}

int call_object_clear(PyObject *self)
{
    CallObject *o = reinterpret_cast<CallObject *>(self);
    Call *c = o->call;
    o->call = nullptr;
    delete c;
    return 0;
}

void call_object_free(PyObject *self)
{
    PyObject_GC_UnTrack(self);
    call_object_clear(self);
    PyTypeObject *type = Py_TYPE(self);
    type->tp_free(self);
    Py_DECREF(type);
}

PyMemberDef call_members[] = {
    {"__vectorcalloffset__", T_PYSSIZET, offsetof(CallObject, vectorcall), READONLY, nullptr},
    {nullptr, 0, 0, 0, nullptr},
};
PyType_Slot call_slots[] = {
    {Py_tp_dealloc, reinterpret_cast<void *>(call_object_free)},
    {Py_tp_traverse, reinterpret_cast<void *>(call_object_traverse)},
    {Py_tp_clear, reinterpret_cast<void *>(call_object_clear)},
    {Py_tp_call, reinterpret_cast<void *>(PyVectorcall_Call)},
    {Py_tp_members, call_members},
    {0, nullptr},
};
PyType_Spec call_spec = {"paper_2411_07942_amd._binding.Call", sizeof(CallObject), 0,
                         Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL | Py_TPFLAGS_HAVE_GC, call_slots};
PyTypeObject *g_call_type;

bool arg_count(Py_ssize_t got, Py_ssize_t want)
{
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, got);
    return false;
}

// issue once: the arguments, then the stream
template <Kind K>
PyObject *do_now(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (!arg_count(nargs, kArgs[K] + 1)) return nullptr;
    return no_throw([&]() -> PyObject * {
        Call c;
        if (!c.take(K, args) || !c.run(args[kArgs[K]])) return nullptr;
        Py_RETURN_NONE;
    });
}

template <Kind K>
PyObject *do_make(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (!arg_count(nargs, kArgs[K])) return nullptr;
    CallObject *o = reinterpret_cast<CallObject *>(g_call_type->tp_alloc(g_call_type, 0));
    if (!o) return nullptr;
    o->vectorcall = call_object_call;
    PyObject *self = reinterpret_cast<PyObject *>(o);
    if (no_throw([&]() -> PyObject * {
            o->call = new Call;
            return o->call->take(K, args) ? self : nullptr;
        }))
        return self;
    Py_DECREF(self);
    return nullptr;
}

// ---- calibration and plan -----------------------------------------------------------------

// (Y, rank, n_ranks, seq_index, gamma, m, M, workspace, stream); tpq_calibrate_fixed without the workspace
template <bool fixed>
PyObject *calibrate(PyObject *const *a)
{
    const at::Tensor *Y = tensor(a[0]);
    if (!Y) return nullptr;
    if (Y->dim() != 2) {
        PyErr_SetString(PyExc_ValueError, "a calibration sequence is two-dimensional");
        return nullptr;
    }
    const int64_t S = Y->size(0), E = Y->size(1);
    const long rank = PyLong_AsLong(a[1]), n_ranks = PyLong_AsLong(a[2]);
    const long long seq = PyLong_AsLongLong(a[3]);
    const double gamma = PyFloat_AsDouble(a[4]);
    void *m, *M, *s;
    if (PyErr_Occurred() || !pointer(a[5], m) || !pointer(a[6], M) || !stream_of(a[fixed ? 7 : 8], s)) return nullptr;
    void *ws = nullptr;
    size_t ws_bytes = 0;
    if (!fixed) {
        const at::Tensor *t = tensor(a[7]);
        if (!t) return nullptr;
        if (!pointer(a[7], ws)) return nullptr;
        ws_bytes = static_cast<size_t>(t->numel()) * t->element_size();
    }
    void *y;
    if (!pointer(a[0], y)) return nullptr;
    const int64_t ld = row_stride(*Y, S, E);
    const int rc = [&] {
        const WithoutGil free;
        return fixed ? tpq_calibrate_fixed(static_cast<const uint16_t *>(y), S, ld, static_cast<int>(E), static_cast<int>(rank), static_cast<int>(n_ranks), seq,
                                           static_cast<float>(gamma), static_cast<float *>(m), static_cast<float *>(M), s)
                     : tpq_calibrate(static_cast<const uint16_t *>(y), S, ld, static_cast<int>(E), static_cast<int>(rank), static_cast<int>(n_ranks), seq,
                                     static_cast<float>(gamma), static_cast<float *>(m), static_cast<float *>(M), ws, ws_bytes, s);
    }();
    if (!check(rc, fixed ? "tpq_calibrate_fixed" : "tpq_calibrate")) return nullptr;
    Py_RETURN_NONE;
}

template <bool fixed>
PyObject *do_calibrate(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    if (!arg_count(nargs, fixed ? 8 : 9)) return nullptr;
    return no_throw([&] { return calibrate<fixed>(a); });
}

// (L, idx_sorted, plan, stream)
PyObject *plan_build(PyObject *const *a)
{
    Layout L;
    void *idx, *plan, *s;
    const at::Tensor *buffer = tensor(a[2]);
    if (!buffer || !L.take(a[0]) || !pointer(a[1], idx) || !pointer(a[2], plan) || !stream_of(a[3], s)) return nullptr;
    const size_t bytes = static_cast<size_t>(buffer->numel());
    const int rc = [&] {
        const WithoutGil free;
        return tpq_plan_build(L.p, static_cast<const int32_t *>(idx), plan, bytes, s);
    }();
    if (!check(rc, "tpq_plan_build")) return nullptr;
    Py_RETURN_NONE;
}

PyObject *do_plan_build(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    if (!arg_count(nargs, 4)) return nullptr;
    return no_throw([&] { return plan_build(a); });
}

// (check, get_device, get_stream): what this module calls back
PyObject *do_setup(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    if (!arg_count(nargs, 3)) return nullptr;
    PyObject **slot[3] = {&g_check, &g_get_device, &g_get_stream};
    for (int i = 0; i < 3; ++i) {
        Py_INCREF(a[i]);
        Py_XSETREF(*slot[i], a[i]);
    }
    Py_RETURN_NONE;
}

#define FAST(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(fn)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    FAST("setup", do_setup),
    FAST("encode", do_now<kEncode>), FAST("encode_call", do_make<kEncode>),
    FAST("hop", do_now<kHop>), FAST("hop_call", do_make<kHop>),
    FAST("gemm_encode", do_now<kGemm>), FAST("gemm_encode_call", do_make<kGemm>),
    FAST("decode_reduce", do_now<kDecode>), FAST("decode_reduce_call", do_make<kDecode>),
    FAST("decode_reduce_fused", do_now<kFused>), FAST("decode_reduce_fused_call", do_make<kFused>),
    FAST("encode_static", do_now<kEncodeStatic>), FAST("encode_static_call", do_make<kEncodeStatic>),
    FAST("decode_reduce_static", do_now<kDecodeStatic>), FAST("decode_reduce_static_call", do_make<kDecodeStatic>),
    FAST("calibrate", do_calibrate<false>), FAST("calibrate_fixed", do_calibrate<true>), FAST("plan_build", do_plan_build),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void)
{
    s_codes = PyUnicode_InternFromString("codes");
    s_scale = PyUnicode_InternFromString("scale");
    s_zero = PyUnicode_InternFromString("zero");
    s_outl = PyUnicode_InternFromString("outl");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    s_stream = PyUnicode_InternFromString("stream");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_call_type = reinterpret_cast<PyTypeObject *>(PyType_FromSpec(&call_spec));
    if (!g_call_type || !s_codes || !s_scale || !s_zero || !s_outl || !s_cuda_stream || !s_stream || !s_data_ptr) return nullptr;
    return PyModule_Create(&module);
}
