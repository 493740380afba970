// Native half of the Python binding: checks torch tensors, allocates the outputs that were not given and calls
// the C ABI of libgfwa with raw pointers and the current HIP stream.  Small problems are bound by the host: through
// ctypes and Python-level checks a prefix + forward pair took 22 us of host time and a training step of ten tensors
// 75 us, more than its kernels; here a call costs its kernel launches plus about a microsecond.
//
// The module has no link-time dependency on libgfwa: binding.py hands over the addresses of its functions once
// (bind), so that the library named by GFWA_LIB is the one that is called.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>
#include <string>

#include "../../include/gfwa.h"

namespace {

// ---- the library's functions, by name, in the order bind() takes their addresses
struct Library {
    decltype(&gfwa_gate_prefix) gate_prefix;
    decltype(&gfwa_gate_activation_prefix) gate_activation_prefix;
    decltype(&gfwa_gate_activation_backward) gate_activation_backward;
    decltype(&gfwa_gate_scan_workspace_bytes) gate_scan_workspace_bytes;
    decltype(&gfwa_gate_prefix_stp) gate_prefix_stp;
    decltype(&gfwa_forward_gqa) forward_gqa;
    decltype(&gfwa_backward_workspace_bytes) backward_workspace_bytes;
    decltype(&gfwa_backward_gqa) backward_gqa;
    decltype(&gfwa_decode_workspace_bytes) decode_workspace_bytes;
    decltype(&gfwa_decode) decode;
    decltype(&gfwa_decode_static) decode_static;
};
constexpr Py_ssize_t kFunctions = sizeof(Library) / sizeof(void*);
Library lib;
PyObject* raise_status = nullptr;  // binding._check: turns a negative status into GfwaError

struct PyError {};  // a Python exception is set

// A scope without the interpreter lock, taken again however the scope is left (looking up the stream may throw).
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked&) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};

[[noreturn]] void fail(PyObject* type, const std::string& text) {
    PyErr_SetString(type, text.c_str());
    throw PyError{};
}

std::string shape_text(at::IntArrayRef s) {  // as Python prints a tuple
    std::string r = "(";
    for (size_t i = 0; i < s.size(); ++i) r += (i ? ", " : "") + std::to_string(s[i]);
    return r + (s.size() == 1 ? ",)" : ")");
}
std::string dtype_text(at::ScalarType t) { return std::string("torch.") + torch::getTHPDtype(t)->name; }

const at::Tensor& tensor_of(PyObject* o, const char* name) {
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, std::string(name) + " must be a tensor");
    return THPVariable_Unpack(o);
}

void need(const at::Tensor& t, at::IntArrayRef shape, at::ScalarType dtype, const char* name) {
    if (!t.is_cuda()) fail(PyExc_ValueError, std::string(name) + " must live on the GPU");
    if (t.sizes() != shape)
        fail(PyExc_ValueError, std::string(name) + " has shape " + shape_text(t.sizes()) + ", expected " + shape_text(shape));
    if (t.scalar_type() != dtype)
        fail(PyExc_TypeError, std::string(name) + " has dtype " + dtype_text(t.scalar_type()) + ", expected " + dtype_text(dtype));
    if (!t.is_contiguous()) fail(PyExc_ValueError, std::string(name) + " must be contiguous");
}

const void* input(PyObject* o, at::IntArrayRef shape, at::ScalarType dtype, const char* name) {
    const at::Tensor& t = tensor_of(o, name);
    need(t, shape, dtype, name);
    return t.const_data_ptr();
}

// without the interpreter lock, as torch.empty does it: an allocation may wait for the driver
at::Tensor fresh(at::IntArrayRef shape, at::ScalarType dtype, at::Device device) {
    Unlocked other_threads_may_run;
    return at::Tensor(at::detail::empty_cuda(shape, dtype, device, std::nullopt));
}

// An output: the caller's tensor, checked, or a fresh one.
struct Output {
    PyObject* given = nullptr;
    at::Tensor made;
    void* ptr = nullptr;
    Output(PyObject* o, at::IntArrayRef shape, at::ScalarType dtype, at::Device device, const char* name) {
        if (o == Py_None) {
            made = fresh(shape, dtype, device);
            ptr = made.data_ptr();
        } else {
            const at::Tensor& t = tensor_of(o, name);
            need(t, shape, dtype, name);
            given = o;
            ptr = t.data_ptr();
        }
    }
    PyObject* object() {
        if (given == nullptr) return THPVariable_Wrap(std::move(made));
        Py_INCREF(given);
        return given;
    }
};

// Scratch: the caller's tensor, or a fresh one of `bytes`.
struct Workspace {
    at::Tensor t;
    void* ptr;
    size_t bytes;
    Workspace(PyObject* o, size_t want, at::Device device) {
        if (o == Py_None) {
            t = fresh({(int64_t)want}, at::kByte, device);
        } else {
            t = tensor_of(o, "workspace");
            if (!t.is_cuda() || !t.is_contiguous()) fail(PyExc_ValueError, "workspace must be a contiguous GPU tensor");
        }
        ptr = t.data_ptr();
        bytes = t.nbytes();
    }
};

PyObject* tuple_of(std::initializer_list<Output*> outs) {
    PyObject* r = PyTuple_New((Py_ssize_t)outs.size());
    if (r == nullptr) throw PyError{};
    Py_ssize_t i = 0;
    for (Output* o : outs) {
        PyObject* x = o->object();
        if (x == nullptr) {
            Py_DECREF(r);
            throw PyError{};
        }
        PyTuple_SET_ITEM(r, i++, x);
    }
    return r;
}

// int(x) and float(x) of a Python number; integers are passed on modulo 2^32, as ctypes does for a C int
int as_int(PyObject* o) {
    PyObject* n = PyNumber_Long(o);
    if (n == nullptr) throw PyError{};
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    if (PyErr_Occurred()) throw PyError{};
    return (int)(unsigned)v;
}
float as_float(PyObject* o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw PyError{};
    return (float)v;
}

int storage_type(const at::Tensor& t) {
    if (t.scalar_type() == at::kBFloat16) return GFWA_BF16;
    if (t.scalar_type() == at::kFloat) return GFWA_F32;
    fail(PyExc_TypeError, "unsupported dtype " + dtype_text(t.scalar_type()) + ": bfloat16 or float32");
}

int kv_heads(int64_t H, int64_t Hkv) {
    if (Hkv <= 0 || H % Hkv != 0)
        fail(PyExc_ValueError, "the number of key/value heads (" + std::to_string(Hkv) +
                                   ") must divide the number of query heads (" + std::to_string(H) + ")");
    return (int)Hkv;
}

gfwa_stream_t stream() { return c10::hip::getCurrentHIPStream().stream(); }

// The library call itself, without the interpreter lock (other host threads may launch on other streams).
template <typename F>
void call(F&& f) {
    int status;
    {
        Unlocked other_threads_may_run;
        status = f();
    }
    if (status != 0) {
        PyObject* r = PyObject_CallFunction(raise_status, "i", status);
        Py_XDECREF(r);
        if (PyErr_Occurred()) throw PyError{};
    }
}

template <PyObject* (*F)(PyObject* const*), Py_ssize_t N>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%zd arguments expected", N);
        return nullptr;
    }
    try {
        return F(a);
    } catch (const PyError&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// [B,H,N] of a gate tensor
struct Rows {
    int B, H, N;
    Rows(const at::Tensor& t, const char* name) {
        if (t.dim() != 3) fail(PyExc_ValueError, std::string(name) + " must be [B,H,N]");
        B = (int)t.size(0);
        H = (int)t.size(1);
        N = (int)t.size(2);
    }
};

PyObject* gate_prefix(PyObject* const* a) {  // alpha, c
    const at::Tensor& alpha = tensor_of(a[0], "alpha");
    const Rows r(alpha, "alpha");
    const at::IntArrayRef shape = alpha.sizes();
    need(alpha, shape, at::kFloat, "alpha");
    Output c(a[1], shape, at::kFloat, alpha.device(), "c");
    call([&] { return lib.gate_prefix((const float*)alpha.const_data_ptr(), (float*)c.ptr, r.B, r.H, r.N, stream()); });
    return c.object();
}

PyObject* gate_activation_prefix(PyObject* const* a) {  // hpre, beta, eps, c
    const at::Tensor& hpre = tensor_of(a[0], "hpre");
    const Rows r(hpre, "hpre");
    const at::IntArrayRef shape = hpre.sizes();
    need(hpre, shape, at::kFloat, "hpre");
    const void* beta = input(a[1], shape, at::kFloat, "beta");
    const float eps = as_float(a[2]);
    Output c(a[3], shape, at::kFloat, hpre.device(), "c");
    call([&] {
        return lib.gate_activation_prefix((const float*)hpre.const_data_ptr(), (const float*)beta, eps, (float*)c.ptr, r.B, r.H,
                                          r.N, stream());
    });
    return c.object();
}

PyObject* gate_activation_backward(PyObject* const* a) {  // hpre, beta, eps, dalpha, dh, dbeta
    const at::Tensor& hpre = tensor_of(a[0], "hpre");
    const Rows r(hpre, "hpre");
    const at::IntArrayRef shape = hpre.sizes();
    need(hpre, shape, at::kFloat, "hpre");
    const void* beta = input(a[1], shape, at::kFloat, "beta");
    const float eps = as_float(a[2]);
    const void* dalpha = input(a[3], shape, at::kFloat, "dalpha");
    Output dh(a[4], shape, at::kFloat, hpre.device(), "dh");
    Output dbeta(a[5], shape, at::kFloat, hpre.device(), "dbeta");
    call([&] {
        return lib.gate_activation_backward((const float*)hpre.const_data_ptr(), (const float*)beta, eps, (const float*)dalpha,
                                            (float*)dh.ptr, (float*)dbeta.ptr, r.B, r.H, r.N, stream());
    });
    return tuple_of({&dh, &dbeta});
}

PyObject* gate_prefix_stp(PyObject* const* a) {  // x, beta, eps, c, workspace
    const at::Tensor& x = tensor_of(a[0], "x");
    const Rows r(x, "x");
    const at::IntArrayRef shape = x.sizes();
    need(x, shape, at::kFloat, "x");
    const void* beta = a[1] == Py_None ? nullptr : input(a[1], shape, at::kFloat, "beta");
    const float eps = as_float(a[2]);
    Output c(a[3], shape, at::kFloat, x.device(), "c");
    Workspace ws(a[4], a[4] == Py_None ? lib.gate_scan_workspace_bytes(r.B, r.H, r.N) : 0, x.device());
    call([&] {
        return lib.gate_prefix_stp((const float*)x.const_data_ptr(), (const float*)beta, eps, (float*)c.ptr, ws.ptr, ws.bytes,
                                   r.B, r.H, r.N, stream());
    });
    return c.object();
}

// sizes of the attention calls: Q [B,H,N,d], K [B,Hkv,N,d]; `grouped` lets Hkv differ from H
struct Sizes {
    int64_t B, H, N, d, Hkv;
    int64_t q[4], kv[4], rows[3];
    Sizes(const at::Tensor& Q, const at::Tensor& K, bool grouped) {
        if (Q.dim() != 4 || (grouped && K.dim() != 4))
            fail(PyExc_ValueError, grouped ? "Q must be [B,H,N,d] and K [B,Hkv,N,d]" : "Q must be [B,H,N,d]");
        B = Q.size(0);
        H = Q.size(1);
        N = Q.size(2);
        d = Q.size(3);
        Hkv = grouped ? kv_heads(H, K.size(1)) : H;
        q[0] = kv[0] = rows[0] = B;
        q[1] = rows[1] = H;
        kv[1] = Hkv;
        q[2] = kv[2] = rows[2] = N;
        q[3] = kv[3] = d;
    }
};

PyObject* forward(PyObject* const* a) {  // grouped, Q, K, V, c, w, scale, O, L
    const at::Tensor& Q = tensor_of(a[1], "Q");
    const at::Tensor& K = tensor_of(a[2], "K");
    const Sizes s(Q, K, a[0] == Py_True);
    const int dt = storage_type(Q);
    const at::ScalarType st = Q.scalar_type();
    need(Q, s.q, st, "Q");
    need(K, s.kv, st, "K");
    const void* V = input(a[3], s.kv, st, "V");
    const void* c = input(a[4], s.rows, at::kFloat, "c");
    const int w = as_int(a[5]);
    const float scale = as_float(a[6]);
    Output O(a[7], s.q, st, Q.device(), "O");
    Output L(a[8], s.rows, at::kFloat, Q.device(), "L");
    call([&] {
        return lib.forward_gqa(dt, Q.const_data_ptr(), K.const_data_ptr(), V, (const float*)c, O.ptr, (float*)L.ptr, (int)s.B,
                               (int)s.H, (int)s.Hkv, (int)s.N, (int)s.d, w, scale, stream());
    });
    return tuple_of({&O, &L});
}

PyObject* backward(PyObject* const* a) {  // grouped, Q, K, V, O, dO, c, L, w, scale, workspace, dQ, dK, dV, dalpha
    const at::Tensor& Q = tensor_of(a[1], "Q");
    const at::Tensor& K = tensor_of(a[2], "K");
    const Sizes s(Q, K, a[0] == Py_True);
    const int dt = storage_type(Q);
    const at::ScalarType st = Q.scalar_type();
    need(Q, s.q, st, "Q");
    need(K, s.kv, st, "K");
    const void* V = input(a[3], s.kv, st, "V");
    const void* O = input(a[4], s.q, st, "O");
    const void* dO = input(a[5], s.q, st, "dO");
    const void* c = input(a[6], s.rows, at::kFloat, "c");
    const void* L = input(a[7], s.rows, at::kFloat, "L");
    const int w = as_int(a[8]);
    const float scale = as_float(a[9]);
    Output dQ(a[11], s.q, st, Q.device(), "dQ");
    Output dK(a[12], s.kv, st, Q.device(), "dK");
    Output dV(a[13], s.kv, st, Q.device(), "dV");
    Output dalpha(a[14], s.rows, at::kFloat, Q.device(), "dalpha");
    Workspace ws(a[10], a[10] == Py_None ? lib.backward_workspace_bytes(dt, (int)s.B, (int)s.H, (int)s.N, (int)s.d, w) : 0,
                 Q.device());
    call([&] {
        return lib.backward_gqa(dt, Q.const_data_ptr(), K.const_data_ptr(), V, O, dO, (const float*)c, (const float*)L, dQ.ptr,
                                dK.ptr, dV.ptr, (float*)dalpha.ptr, ws.ptr, ws.bytes, (int)s.B, (int)s.H, (int)s.Hkv, (int)s.N,
                                (int)s.d, w, scale, stream());
    });
    return tuple_of({&dQ, &dK, &dV, &dalpha});
}

// the tensors both decoding calls take: q, Kc, Vc, c, pos, w, scale, alpha_t in a[0..7]
struct Step {
    const at::Tensor& q;
    int64_t B, H, Hkv, T, d, qs[3], heads[2];
    int dt, w;
    float scale;
    const void *Kc, *Vc, *alpha;
    float* c;
    const int* pos;
    explicit Step(PyObject* const* a) : q(tensor_of(a[0], "q")) {
        const at::Tensor& K = tensor_of(a[1], "Kc");
        if (q.dim() != 3 || K.dim() != 4) fail(PyExc_ValueError, "q must be [B,H,d] and Kc [B,Hkv,T,d]");
        B = q.size(0);
        H = q.size(1);
        d = q.size(2);
        T = K.size(2);
        Hkv = kv_heads(H, K.size(1));
        dt = storage_type(q);
        qs[0] = heads[0] = B;
        qs[1] = heads[1] = H;
        qs[2] = d;
        const int64_t cache[4] = {B, Hkv, T, d}, rows[3] = {B, H, T}, batch[1] = {B};
        need(q, qs, q.scalar_type(), "q");
        need(K, cache, q.scalar_type(), "Kc");
        Kc = K.const_data_ptr();
        Vc = input(a[2], cache, q.scalar_type(), "Vc");
        const at::Tensor& ct = tensor_of(a[3], "c");
        need(ct, rows, at::kFloat, "c");
        c = (float*)ct.data_ptr();
        pos = (const int*)input(a[4], batch, at::kInt, "pos");
        w = as_int(a[5]);
        scale = as_float(a[6]);
        alpha = a[7] == Py_None ? nullptr : input(a[7], heads, at::kFloat, "alpha_t");
    }
};

PyObject* decode(PyObject* const* a) {  // q, Kc, Vc, c, pos, w, scale, alpha_t, o, L, workspace
    const Step s(a);
    Output o(a[8], s.qs, s.q.scalar_type(), s.q.device(), "o");
    Output L(a[9], s.heads, at::kFloat, s.q.device(), "L");
    Workspace ws(a[10], a[10] == Py_None ? lib.decode_workspace_bytes((int)s.B, (int)s.H, (int)s.T, (int)s.d, s.w) : 0,
                 s.q.device());
    call([&] {
        return lib.decode(s.dt, s.q.const_data_ptr(), s.Kc, s.Vc, s.c, (const float*)s.alpha, s.pos, o.ptr, (float*)L.ptr, ws.ptr,
                          ws.bytes, (int)s.B, (int)s.H, (int)s.Hkv, (int)s.T, (int)s.d, s.w, s.scale, stream());
    });
    return tuple_of({&o, &L});
}

PyObject* decode_static(PyObject* const* a) {  // q, Kc, Vc, c, pos, w, scale, alpha_t, o, L
    const Step s(a);
    const at::Tensor& o = tensor_of(a[8], "o");
    const at::Tensor& L = tensor_of(a[9], "L");
    need(o, s.qs, s.q.scalar_type(), "o");
    need(L, s.heads, at::kFloat, "L");
    call([&] {
        return lib.decode_static(s.dt, s.q.const_data_ptr(), s.Kc, s.Vc, s.c, (const float*)s.alpha, s.pos, o.data_ptr(),
                                 (float*)L.data_ptr(), (int)s.B, (int)s.H, (int)s.Hkv, (int)s.T, (int)s.d, s.w, s.scale, stream());
    });
    return PyTuple_Pack(2, a[8], a[9]);
}

// bind(check, (address, ...)): binding._check and the functions of `Library`, in its order
PyObject* bind(PyObject* const* a) {
    if (!PyTuple_Check(a[1]) || PyTuple_GET_SIZE(a[1]) != kFunctions)
        fail(PyExc_TypeError, "a tuple of " + std::to_string(kFunctions) + " addresses expected");
    void* addr[kFunctions];
    for (Py_ssize_t i = 0; i < kFunctions; ++i) {
        addr[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(a[1], i));
        if (PyErr_Occurred()) throw PyError{};
    }
    memcpy(&lib, addr, sizeof(lib));
    Py_INCREF(a[0]);
    Py_XDECREF(raise_status);
    raise_status = a[0];
    Py_RETURN_NONE;
}

#define GFWA_ENTRY(f, n) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<f, n>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {GFWA_ENTRY(bind, 2),
                         GFWA_ENTRY(gate_prefix, 2),
                         GFWA_ENTRY(gate_activation_prefix, 4),
                         GFWA_ENTRY(gate_activation_backward, 6),
                         GFWA_ENTRY(gate_prefix_stp, 5),
                         GFWA_ENTRY(forward, 9),
                         GFWA_ENTRY(backward, 15),
                         GFWA_ENTRY(decode, 11),
                         GFWA_ENTRY(decode_static, 10),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_gfwa_call", "Checked calls of libgfwa on torch tensors.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__gfwa_call(void) { return PyModule_Create(&module); }
