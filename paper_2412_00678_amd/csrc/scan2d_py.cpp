// Native side of the Python binding (paper_2412_00678_amd/scan2d.py): argument checks, output allocation and the call
// through the C ABI, for the entry points that a program calls once per layer and pass.
//
// What it is for: the short calls.  Checking and converting a dozen tensors in Python and ctypes costs 10 to 14 us per
// call, more than the kernels of a small map take (a 16x16 scan runs in 4 us); here the same checks cost under 1 us, the
// rest of a call is torch's allocator and the launch.  Every function takes its arguments positionally, in the order of
// the Python function of the same name, and raises the exceptions that function documents.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>
#include <utility>

#include "../../include/scan2d.h"

namespace {

PyObject* g_error = nullptr;             // scan2d.Scan2dError

struct Raised {};                        // a Python exception is set

[[noreturn]] void raise(PyObject* type, const std::string& text) {
    PyErr_SetString(type, text.c_str());
    throw Raised{};
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

void check_rc(int rc, const char* where) {
    if (rc == SCAN2D_OK) return;
    PyObject* e = PyObject_CallFunction(g_error, "is", rc, where);
    if (e != nullptr) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    throw Raised{};
}

// The call without the interpreter's lock: it may wait (a full queue, code objects loaded by a first call), and other
// threads run meanwhile.
template <typename R, typename... P, typename... A>
R unlocked(R (*fn)(P...), A... args) {
    PyThreadState* const state = PyEval_SaveThread();
    const R r = fn(args...);
    PyEval_RestoreThread(state);
    return r;
}

std::string describe(at::ScalarType t, at::IntArrayRef shape) {
    std::string name = c10::toString(t);
    if (t == at::kFloat) name = "float32";
    else if (t == at::kBFloat16) name = "bfloat16";
    else if (t == at::kByte) name = "uint8";
    else if (t == at::kDouble) name = "float64";
    else if (t == at::kHalf) name = "float16";
    std::string s = "torch." + name + " (";
    for (size_t i = 0; i < shape.size(); ++i) s += (i ? ", " : "") + std::to_string(shape[i]);
    return s + (shape.size() == 1 ? ",)" : ")");
}

const at::Tensor& tensor(PyObject* o, const char* name) {
    if (!THPVariable_Check(o)) raise(PyExc_TypeError, std::string(name) + " must be a torch.Tensor");
    return THPVariable_Unpack(o);
}

// The device pointer of a required tensor of this type and shape.
void* need(PyObject* o, const char* name, at::ScalarType t, at::IntArrayRef shape) {
    if (o == Py_None) raise(PyExc_ValueError, std::string(name) + " is required");
    const at::Tensor& v = tensor(o, name);
    if (!v.is_cuda() || !v.is_contiguous()) raise(PyExc_ValueError, std::string(name) + " must be a contiguous device tensor");
    if (v.scalar_type() != t || v.sizes() != shape)
        raise(PyExc_ValueError, std::string(name) + ": expected " + describe(t, shape) + ", got " + describe(v.scalar_type(), v.sizes()));
    return v.data_ptr();
}
void* maybe(PyObject* o, const char* name, at::ScalarType t, at::IntArrayRef shape) { return o == Py_None ? nullptr : need(o, name, t, shape); }
float* needf(PyObject* o, const char* name, at::IntArrayRef shape) { return static_cast<float*>(need(o, name, at::kFloat, shape)); }
float* maybef(PyObject* o, const char* name, at::IntArrayRef shape) { return static_cast<float*>(maybe(o, name, at::kFloat, shape)); }

int64_t dim(PyObject* o, const char* name, int i) {
    const at::Tensor& v = tensor(o, name);
    if (v.dim() <= i) raise(PyExc_IndexError, std::string(name) + " has too few dimensions");
    return v.size(i);
}

// The map tensor a call is described by: its shape, type and device.
struct Map {
    at::ScalarType t;
    int64_t Bt, C, H, W;
    at::Device dev = at::Device(at::kCPU);
    scan2d_desc d;
    Map(PyObject* o, const char* name, int64_t N, uint32_t flags) {
        const at::Tensor& v = tensor(o, name);
        if (v.dim() != 4) raise(PyExc_ValueError, std::string(name) + ": expected 4 dimensions, got " + std::to_string(v.dim()));
        t = v.scalar_type();
        if (t != at::kFloat && t != at::kBFloat16)
            raise(PyExc_TypeError, std::string("x must be float32 or bfloat16, got ") + describe(t, {}).substr(0, describe(t, {}).size() - 3));
        Bt = v.size(0); C = v.size(1); H = v.size(2); W = v.size(3);
        dev = v.device();
        d = scan2d_desc{(int32_t)Bt, (int32_t)C, (int32_t)H, (int32_t)W, (int32_t)N, t == at::kBFloat16 ? SCAN2D_BF16 : SCAN2D_F32, flags};
    }
    at::Tensor make(at::IntArrayRef shape, at::ScalarType type) const { return at::empty(shape, at::TensorOptions().dtype(type).device(dev)); }
    at::Tensor map() const { return make({Bt, C, H, W}, t); }
};

uint32_t flags_of(PyObject* o) {
    const unsigned long v = PyLong_AsUnsignedLongMask(o);
    if (PyErr_Occurred()) throw Raised{};
    return (uint32_t)v;
}
int64_t int_of(PyObject* o) {
    const long long v = PyLong_AsLongLong(o);
    if (PyErr_Occurred()) throw Raised{};
    return v;
}

// The caller's workspace as it is, or one of the size the library asks for.
struct Workspace {
    at::Tensor own;
    void* p = nullptr;
    size_t bytes = 0;
    Workspace(PyObject* o, const Map& m, int pass) {
        if (o != Py_None) {
            const at::Tensor& v = tensor(o, "workspace");
            p = v.data_ptr();
            bytes = (size_t)v.numel() * v.element_size();
            return;
        }
        bytes = scan2d_workspace_bytes(&m.d, pass);
        if (bytes == 0) return;
        own = m.make({(int64_t)bytes}, at::kByte);
        p = own.data_ptr();
    }
};

// The tensors a caller hands over for the outputs, held until the call has returned: an iterable may make its items as it
// goes, and then nothing else keeps them.
struct Given {
    PyObject* item[6] = {};               // owned
    Given() = default;
    Given(const Given&) = delete;
    ~Given() { for (PyObject* o : item) Py_XDECREF(o); }
    // out[0] .. out[n - 1], none of them None
    void index(PyObject* out, int n, const char* text) {
        for (int i = 0; i < n; ++i) {
            PyObject* key = PyLong_FromLong(i);
            if (key == nullptr) throw Raised{};
            item[i] = PyObject_GetItem(out, key);
            Py_DECREF(key);
            if (item[i] == nullptr) throw Raised{};
            if (item[i] == Py_None) raise(PyExc_ValueError, text);
        }
    }
    // the n items of an iterable
    void unpack(PyObject* out, int n, const char* text) {
        PyObject* t = PySequence_Tuple(out);
        if (t == nullptr) throw Raised{};
        const bool all = PyTuple_GET_SIZE(t) == n;
        for (int i = 0; all && i < n; ++i) {
            item[i] = PyTuple_GET_ITEM(t, i);
            Py_INCREF(item[i]);
        }
        Py_DECREF(t);
        if (!all) raise(PyExc_ValueError, text);
    }
    PyObject* operator[](int i) const { return item[i]; }
};

// An output: the caller's tensor, checked, or a new one.
struct Out {
    PyObject* o;                          // owned
    void* p;
    Out(PyObject* given, const char* name, const Map& m, at::ScalarType t, at::IntArrayRef shape) {
        if (given != nullptr && given != Py_None) {
            p = need(given, name, t, shape);
            o = given;
            Py_INCREF(o);
        } else {
            at::Tensor v = m.make(shape, t);
            p = v.data_ptr();
            o = THPVariable_Wrap(std::move(v));
            if (o == nullptr) throw Raised{};
        }
    }
    Out() : o(Py_None), p(nullptr) { Py_INCREF(o); }     // an output that does not exist
    Out(Out&& r) noexcept : o(r.o), p(r.p) { r.o = nullptr; }
    Out(const Out&) = delete;
    ~Out() { Py_XDECREF(o); }
    float* f() const { return static_cast<float*>(p); }
    PyObject* release() { PyObject* r = o; o = nullptr; return r; }
};

template <typename... O>
PyObject* tuple(O&... outs) {
    PyObject* t = PyTuple_New(sizeof...(outs));
    if (t == nullptr) throw Raised{};
    Py_ssize_t i = 0;
    ((PyTuple_SET_ITEM(t, i++, outs.release())), ...);
    return t;
}

// The tensors every scan call has.
struct Scan {
    Map m;
    int64_t N;
    void *x, *delta, *Bm, *Cm;
    float *A, *Dskip;
    uint8_t* mask;
    Scan(PyObject* ox, PyObject* od, const char* dname, PyObject* oA, PyObject* oB, PyObject* oC, PyObject* oD, PyObject* om, uint32_t flags)
        : m(ox, "x", dim(oA, "A", 1), flags), N(m.d.N) {
        const int64_t map[] = {m.Bt, m.C, m.H, m.W}, st[] = {m.Bt, N, m.H, m.W};
        x = need(ox, "x", m.t, map);
        delta = need(od, dname, m.t, map);
        A = needf(oA, "A", {m.C, N});
        Bm = need(oB, "Bm", m.t, st);
        Cm = need(oC, "Cm", m.t, st);
        Dskip = maybef(oD, "Dskip", {m.C});
        mask = static_cast<uint8_t*>(maybe(om, "mask", at::kByte, {m.Bt, m.H, m.W}));
    }
    void* map(PyObject* o, const char* name) const { return need(o, name, m.t, {m.Bt, m.C, m.H, m.W}); }
    Out new_map(PyObject* o = nullptr, const char* name = "") const { return Out(o, name, m, m.t, {m.Bt, m.C, m.H, m.W}); }
    Out new_A(PyObject* o = nullptr) const { return Out(o, "dA", m, at::kFloat, {m.C, N}); }
    Out new_states(PyObject* o = nullptr, const char* name = "") const { return Out(o, name, m, at::kFloat, {m.Bt, N, m.H, m.W}); }
    Out new_channels(bool exists, PyObject* o = nullptr, const char* name = "") const {
        if (!exists && (o == nullptr || o == Py_None)) return Out();
        return Out(o, name, m, at::kFloat, {m.C});
    }
};

using Args = PyObject* const*;

PyObject* scan_fwd(Args a) {              // x, delta, A, Bm, Cm, Dskip, mask, y, workspace, flags
    const Scan s(a[0], a[1], "delta", a[2], a[3], a[4], a[5], a[6], flags_of(a[9]));
    Out y = s.new_map(a[7], "y");
    const Workspace w(a[8], s.m, SCAN2D_PASS_FWD);
    check_rc(unlocked(scan2d_fwd, &s.m.d, s.x, s.delta, s.A, s.Bm, s.Cm, s.Dskip, s.mask, y.p, w.p, w.bytes, stream()), "scan2d_fwd");
    return y.release();
}

PyObject* scan_fwd_softplus(Args a) {     // x, delta_raw, delta_bias, A, Bm, Cm, Dskip, mask, y, workspace, flags
    const Scan s(a[0], a[1], "delta_raw", a[3], a[4], a[5], a[6], a[7], flags_of(a[10]));
    const float* bias = maybef(a[2], "delta_bias", {s.m.C});
    Out y = s.new_map(a[8], "y");
    const Workspace w(a[9], s.m, SCAN2D_PASS_FWD);
    check_rc(unlocked(scan2d_fwd_softplus, &s.m.d, s.x, s.delta, bias, s.A, s.Bm, s.Cm, s.Dskip, s.mask, y.p, w.p, w.bytes, stream()), "scan2d_fwd_softplus");
    return y.release();
}

PyObject* scan_fwd_gated(Args a) {        // x, delta_raw, delta_bias, A, Bm, Cm, Dskip, mask, z, want_y_scan, workspace, y, y_scan, flags
    const Scan s(a[0], a[1], "delta_raw", a[3], a[4], a[5], a[6], a[7], flags_of(a[13]));
    const float* bias = maybef(a[2], "delta_bias", {s.m.C});
    const void* z = s.map(a[8], "z");
    const int want = PyObject_IsTrue(a[9]);
    if (want < 0) throw Raised{};
    Out y = s.new_map(a[11], "y");
    Out ys = want ? s.new_map(a[12], "y_scan") : Out();
    const Workspace w(a[10], s.m, SCAN2D_PASS_FWD);
    check_rc(unlocked(scan2d_fwd_softplus_gated, &s.m.d, s.x, s.delta, bias, s.A, s.Bm, s.Cm, s.Dskip, s.mask, z, ys.p, y.p, w.p, w.bytes, stream()),
             "scan2d_fwd_softplus_gated");
    return tuple(ys, y);
}

PyObject* scan_bwd(Args a) {              // x, delta, A, Bm, Cm, Dskip, mask, dy, workspace, flags, out
    const Scan s(a[0], a[1], "delta", a[2], a[3], a[4], a[5], a[6], flags_of(a[9]));
    const void* dy = s.map(a[7], "dy");
    Given given;
    if (a[10] != Py_None) {
        given.unpack(a[10], 6, "out: expected six tensors");
        const char* const names[] = {"dx", "ddelta", "dA", "dBm", "dCm"};
        for (int i = 0; i < 5; ++i)
            if (given[i] == Py_None) raise(PyExc_ValueError, std::string(names[i]) + " is required");
    }
    const bool own = a[10] == Py_None;
    Out dx = s.new_map(given[0], "dx"), dd = s.new_map(given[1], "ddelta"), dA = s.new_A(given[2]), dB = s.new_states(given[3], "dBm"),
        dC = s.new_states(given[4], "dCm"), dD = s.new_channels(own && s.Dskip != nullptr, given[5], "dDskip");
    const Workspace w(a[8], s.m, SCAN2D_PASS_BWD);
    check_rc(unlocked(scan2d_bwd, &s.m.d, s.x, s.delta, s.A, s.Bm, s.Cm, s.Dskip, s.mask, dy, dx.p, dd.p, dA.f(), dB.f(), dC.f(), dD.f(), w.p, w.bytes, stream()),
             "scan2d_bwd");
    return tuple(dx, dd, dA, dB, dC, dD);
}

PyObject* scan_bwd_softplus(Args a) {     // x, delta_raw, delta_bias, A, Bm, Cm, Dskip, mask, dy, workspace, flags
    const Scan s(a[0], a[1], "delta_raw", a[3], a[4], a[5], a[6], a[7], flags_of(a[10]));
    const float* bias = maybef(a[2], "delta_bias", {s.m.C});
    const void* dy = s.map(a[8], "dy");
    Out dx = s.new_map(), dd = s.new_map(), db = s.new_channels(bias != nullptr), dA = s.new_A(), dB = s.new_states(), dC = s.new_states(),
        dD = s.new_channels(s.Dskip != nullptr);
    const Workspace w(a[9], s.m, SCAN2D_PASS_BWD_SOFTPLUS);
    check_rc(unlocked(scan2d_bwd_softplus, &s.m.d, s.x, s.delta, bias, s.A, s.Bm, s.Cm, s.Dskip, s.mask, dy, dx.p, dd.p, db.f(), dA.f(), dB.f(), dC.f(), dD.f(),
                                 w.p, w.bytes, stream()), "scan2d_bwd_softplus");
    return tuple(dx, dd, db, dA, dB, dC, dD);
}

PyObject* scan_bwd_gated(Args a) {        // x, delta_raw, delta_bias, A, Bm, Cm, Dskip, mask, z, y_scan, dy, workspace, flags
    const Scan s(a[0], a[1], "delta_raw", a[3], a[4], a[5], a[6], a[7], flags_of(a[12]));
    const float* bias = maybef(a[2], "delta_bias", {s.m.C});
    const void *z = s.map(a[8], "z"), *ys = s.map(a[9], "y_scan"), *dy = s.map(a[10], "dy");
    Out dx = s.new_map(), dd = s.new_map(), dz = s.new_map(), db = s.new_channels(bias != nullptr), dA = s.new_A(), dB = s.new_states(),
        dC = s.new_states(), dD = s.new_channels(s.Dskip != nullptr);
    const Workspace w(a[11], s.m, SCAN2D_PASS_BWD_GATED);
    check_rc(unlocked(scan2d_bwd_softplus_gated, &s.m.d, s.x, s.delta, bias, s.A, s.Bm, s.Cm, s.Dskip, s.mask, z, ys, dy, dx.p, dd.p, db.f(), dA.f(), dB.f(),
                                       dC.f(), dD.f(), dz.p, w.p, w.bytes, stream()), "scan2d_bwd_softplus_gated");
    return tuple(dx, dd, db, dA, dB, dC, dD, dz);
}

PyObject* block_conv_silu(Args a) {       // u, w, bias, PH, PW, x
    const Map m(a[0], "u", 1, 0);
    const int64_t KH = dim(a[1], "w", 1), KW = dim(a[1], "w", 2);
    const void* u = need(a[0], "u", m.t, {m.Bt, m.C, m.H, m.W});
    const float *w = needf(a[1], "w", {m.C, KH, KW}), *bias = maybef(a[2], "bias", {m.C});
    const scan2d_conv_shape cs{(int32_t)KH, (int32_t)KW, (int32_t)(a[3] == Py_None ? KH / 2 : int_of(a[3])),
                               (int32_t)(a[4] == Py_None ? KW / 2 : int_of(a[4]))};
    Out x(a[5], "x", m, m.t, {m.Bt, m.C, m.H, m.W});
    check_rc(unlocked(scan2d_block_conv_silu, &m.d, &cs, u, w, bias, x.p, stream()), "scan2d_block_conv_silu");
    return x.release();
}

PyObject* block_xproj(Args a) {           // x, Wx, Wdt, N, out
    const int64_t N = int_of(a[3]), R = dim(a[2], "Wdt", 1);
    const Map m(a[0], "x", N, 0);
    const void *x = need(a[0], "x", m.t, {m.Bt, m.C, m.H, m.W}), *Wx = need(a[1], "Wx", m.t, {R + 2 * N, m.C});
    const float* Wdt = needf(a[2], "Wdt", {m.C, R});
    Given given;
    if (a[4] != Py_None) given.index(a[4], 3, "out: expected three tensors");
    Out dr(given[0], "delta_raw", m, m.t, {m.Bt, m.C, m.H, m.W}), B(given[1], "Bm", m, m.t, {m.Bt, N, m.H, m.W}),
        C(given[2], "Cm", m, m.t, {m.Bt, N, m.H, m.W});
    check_rc(unlocked(scan2d_block_xproj, &m.d, (int)R, x, Wx, Wdt, dr.p, B.p, C.p, stream()), "scan2d_block_xproj");
    if (a[4] != Py_None) {
        Py_INCREF(a[4]);
        return a[4];
    }
    return tuple(dr, B, C);
}

PyObject* block_linear(Args a) {          // x, Wt, bias, residual, out
    const Map m(a[0], "x", 1, 0);
    const int64_t Cout = dim(a[1], "Wt", 0);
    const void *x = need(a[0], "x", m.t, {m.Bt, m.C, m.H, m.W}), *Wt = need(a[1], "Wt", m.t, {Cout, m.C});
    const float* bias = maybef(a[2], "bias", {Cout});
    const void* res = maybe(a[3], "residual", m.t, {m.Bt, Cout, m.H, m.W});
    Out out(a[4], "out", m, m.t, {m.Bt, Cout, m.H, m.W});
    check_rc(unlocked(scan2d_block_linear, &m.d, (int)Cout, x, Wt, bias, res, out.p, stream()), "scan2d_block_linear");
    return out.release();
}

PyObject* block_norm(Args a) {            // x, gamma, beta, eps, kind, out
    const Map m(a[0], "x", 1, 0);
    const void* x = need(a[0], "x", m.t, {m.Bt, m.C, m.H, m.W});
    const float *gamma = needf(a[1], "gamma", {m.C}), *beta = maybef(a[2], "beta", {m.C});
    const double eps = PyFloat_AsDouble(a[3]);
    if (PyErr_Occurred()) throw Raised{};
    const int64_t kind = int_of(a[4]);
    Out out(a[5], "out", m, m.t, {m.Bt, m.C, m.H, m.W});
    check_rc(unlocked(scan2d_block_norm, &m.d, (int)kind, (float)eps, x, gamma, beta, out.p, stream()), "scan2d_block_norm");
    return out.release();
}

PyObject* block_attn_pool(Args a) {       // h, V, w, mask, out
    const Map m(a[0], "h", 1, 0);
    const int64_t D = dim(a[2], "w", 0);
    const void *h = need(a[0], "h", m.t, {m.Bt, m.C, m.H, m.W}), *V = need(a[1], "V", m.t, {D, m.C});
    const float* w = needf(a[2], "w", {D});
    const uint8_t* mask = static_cast<uint8_t*>(maybe(a[3], "mask", at::kByte, {m.Bt, m.H, m.W}));
    Given given;
    if (a[4] != Py_None) given.index(a[4], 2, "out: expected two tensors");
    Out z(given[0], "z", m, at::kFloat, {m.Bt, m.C}), attn(given[1], "attn", m, at::kFloat, {m.Bt, m.H, m.W});
    check_rc(unlocked(scan2d_block_attn_pool, &m.d, (int)D, h, V, w, mask, attn.f(), z.f(), stream()), "scan2d_block_attn_pool");
    if (a[4] != Py_None) {
        Py_INCREF(a[4]);
        return a[4];
    }
    return tuple(z, attn);
}

// ---- an entry point with its arguments converted once: call(address, arguments) enqueues it again on the current
// stream, which is the last argument of every entry point.  Arguments are pointers and sizes, one 64-bit register or
// stack slot each in this platform's C calling convention.
constexpr int kMostArgs = 24;
template <size_t... I>
int invoke(void* fn, const uint64_t* v, std::index_sequence<I...>) {
    using F = int (*)(decltype((void)I, uint64_t())...);
    return reinterpret_cast<F>(fn)(v[I]...);
}
template <size_t N>
int invoke_n(void* fn, const uint64_t* v) { return invoke(fn, v, std::make_index_sequence<N>()); }
template <size_t... N>
int dispatch(size_t n, void* fn, const uint64_t* v, std::index_sequence<N...>) {
    using F = int (*)(void*, const uint64_t*);
    static constexpr F table[] = {invoke_n<N + 1>...};
    return table[n - 1](fn, v);
}

int dispatch_any(size_t n, void* fn, const uint64_t* v) { return dispatch(n, fn, v, std::make_index_sequence<kMostArgs>()); }

struct Call {
    PyObject_HEAD
    void* fn;
    size_t n;                             // arguments, the stream included
    uint64_t v[kMostArgs];
};
PyObject* call_new(PyTypeObject* type, PyObject* args, PyObject*) {
    unsigned long long fn = 0;
    PyObject* list = nullptr;
    if (!PyArg_ParseTuple(args, "KO!", &fn, &PyTuple_Type, &list)) return nullptr;
    const Py_ssize_t n = PyTuple_GET_SIZE(list);
    if (fn == 0 || n + 1 > kMostArgs) {
        PyErr_SetString(PyExc_ValueError, "Call: no function, or too many arguments");
        return nullptr;
    }
    Call* c = reinterpret_cast<Call*>(type->tp_alloc(type, 0));
    if (c == nullptr) return nullptr;
    c->fn = reinterpret_cast<void*>(fn);
    c->n = (size_t)n + 1;
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject* o = PyTuple_GET_ITEM(list, i);
        c->v[i] = o == Py_None ? 0 : PyLong_AsUnsignedLongLongMask(o);
        if (PyErr_Occurred()) {
            Py_DECREF(c);
            return nullptr;
        }
    }
    return reinterpret_cast<PyObject*>(c);
}
PyObject* call_call(PyObject* self, PyObject*, PyObject*) {
    HANDLE_TH_ERRORS
    const Call* c = reinterpret_cast<Call*>(self);
    uint64_t v[kMostArgs];
    for (size_t i = 0; i + 1 < c->n; ++i) v[i] = c->v[i];
    v[c->n - 1] = reinterpret_cast<uint64_t>(stream());
    return PyLong_FromLong(unlocked(dispatch_any, c->n, c->fn, static_cast<const uint64_t*>(v)));
    END_HANDLE_TH_ERRORS
}
PyTypeObject CallType = {PyVarObject_HEAD_INIT(nullptr, 0)};

// ---- module
template <PyObject* (*F)(Args), int N>
PyObject* entry(PyObject*, Args args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Raised&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}
PyObject* set_error(PyObject*, PyObject* cls) {
    Py_INCREF(cls);
    Py_XDECREF(g_error);
    g_error = cls;
    Py_RETURN_NONE;
}

#define SCAN2D_ENTRY(name, fn, n) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<fn, n>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    SCAN2D_ENTRY("scan2d_fwd", scan_fwd, 10),
    SCAN2D_ENTRY("scan2d_fwd_softplus", scan_fwd_softplus, 11),
    SCAN2D_ENTRY("scan2d_fwd_softplus_gated", scan_fwd_gated, 14),
    SCAN2D_ENTRY("scan2d_bwd", scan_bwd, 11),
    SCAN2D_ENTRY("scan2d_bwd_softplus", scan_bwd_softplus, 11),
    SCAN2D_ENTRY("scan2d_bwd_softplus_gated", scan_bwd_gated, 13),
    SCAN2D_ENTRY("block_conv_silu", block_conv_silu, 6),
    SCAN2D_ENTRY("block_xproj", block_xproj, 5),
    SCAN2D_ENTRY("block_linear", block_linear, 5),
    SCAN2D_ENTRY("block_norm", block_norm, 6),
    SCAN2D_ENTRY("block_attn_pool", block_attn_pool, 5),
    {"set_error", set_error, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_scan2d_py", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__scan2d_py() {
    CallType.tp_name = "_scan2d_py.Call";
    CallType.tp_basicsize = sizeof(Call);
    CallType.tp_flags = Py_TPFLAGS_DEFAULT;
    CallType.tp_new = call_new;
    CallType.tp_call = call_call;
    if (PyType_Ready(&CallType) < 0) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (m == nullptr) return nullptr;
    Py_INCREF(&CallType);
    if (PyModule_AddObject(m, "Call", reinterpret_cast<PyObject*>(&CallType)) < 0 || PyModule_AddIntConstant(m, "MOST_ARGUMENTS", kMostArgs) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
