// The hot entry points of binding.py with their argument marshalling in native code: check the tensors, get the outputs
// and the scratch from torch's allocator, call the C ABI on the current stream.  A call of one decode layer takes 5 us on
// the GPU; the same steps in Python and ctypes took 11 us on the host, and every small layer waited for them.  The offline calls and
// the packing of a cache too: two caches packed 19.3 us of host time in Python against 17.8 on the GPU, 9.0 here; a 11008 x 4096
// weight, whose quantisation waits for the host to read the exponent, 102 -> 96 us.
//
// Every function returns its result, or an int (a non-zero status of the C ABI), or None for anything it does not take:
// a tensor of another type, dtype, device or layout, a wrong shape, an active torch-function mode, an
// exception of any kind.  binding.py then runs its own form of the call, which decides and raises.  No state is kept but the
// addresses of the C functions, handed over once by bind().
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/fireq.h"
#include "../../include/fireq_kv4_ws.h"
#include "../../include/fireq_wquant_ws.h"

namespace {

struct Api {
    decltype(&fq_quantize_act) quantize_act;
    decltype(&fq_quantize_act_ws) quantize_act_ws;
    decltype(&fq_packed_weight_bytes) packed_weight_bytes;
    decltype(&fq_w4a8_gemm_workspace_bytes) gemm_workspace_bytes;
    decltype(&fq_w4a8_gemm_ws) gemm_ws;
    decltype(&fq_w4a8_gemm_swiglu_ws) gemm_swiglu_ws;
    decltype(&fq_w4a8_gemm_add_ws) gemm_add_ws;
    decltype(&fq_w4a8_gemm_swiglu_quant_ws) gemm_swiglu_quant_ws;
    decltype(&fq_w4a8_linear_workspace_bytes) linear_workspace_bytes;
    decltype(&fq_w4a8_linear_ws) linear_ws;
    decltype(&fq_kv4_packed_bytes) kv4_packed_bytes;
    decltype(&fq_kv4_scores) kv4_scores;
    decltype(&fq_kv4_output_workspace_bytes) kv4_output_workspace_bytes;
    decltype(&fq_kv4_output_ws) kv4_output_ws;
    decltype(&fq_kv4_pack) kv4_pack;
    decltype(&fq_pack_weights) pack_weights;
    decltype(&fq_cas_scales_workspace_bytes) cas_scales_workspace_bytes;
    decltype(&fq_cas_scales_ws) cas_scales_ws;
    decltype(&fq_pts_exponent_workspace_bytes) pts_exponent_workspace_bytes;
    decltype(&fq_pts_exponent_ws) pts_exponent_ws;
    decltype(&fq_quantize_weights) quantize_weights;
};
Api api = {};
bool bound = false;

constexpr int64_t GROUP = 128;
constexpr int64_t INT_LIMIT = 0x7FFFFFFF;

struct Decline {};                                        // "not for this path": None to the caller
void want(bool ok) { if (!ok) throw Decline(); }

const at::Tensor& tensor(PyObject* o) {
    want(THPVariable_CheckExact(o));
    return THPVariable_Unpack(o);
}

const at::Tensor& dev(PyObject* o, at::ScalarType t) {
    const at::Tensor& x = tensor(o);
    want(x.is_cuda() && x.scalar_type() == t && x.is_contiguous());
    return x;
}

int whole(PyObject* o) {
    want(PyLong_CheckExact(o));
    const long v = PyLong_AsLong(o);
    want(v >= 0 && v <= INT_LIMIT);                       // (an overflow answers -1 and leaves an exception, cleared below)
    return (int)v;
}

float number(PyObject* o) {
    if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
    return (float)whole(o);
}

bool truth(PyObject* o) {
    want(o == Py_True || o == Py_False);
    return o == Py_True;
}

// A tensor as torch.empty gives it, through the dispatcher: modes, transforms, profilers, the filling of fresh memory and kernels that a
// program has registered for it see every output (straight from the allocator 0.25 us less per tensor, and the last of these would not)
at::Tensor fresh(at::IntArrayRef size, at::ScalarType t, const at::Tensor& like) {
    return at::empty(size, at::TensorOptions().dtype(t).device(like.device()));
}

// the caller's scratch, or one of `need` bytes from the (stream-ordered) allocator, or none
struct Scratch {
    at::Tensor own;
    void* p = nullptr;
    size_t bytes = 0;
    Scratch(PyObject* o, size_t need, const at::Tensor& like) {
        if (o != Py_None) {
            const at::Tensor& t = tensor(o);
            p = t.data_ptr();
            bytes = (size_t)t.numel() * t.element_size();
        } else if (need > 0) {
            own = fresh({(int64_t)need}, at::kByte, like);
            p = own.data_ptr();
            bytes = need;
        }
    }
};

at::Tensor output(PyObject* o, at::IntArrayRef size, const at::Tensor& like) {
    if (o == Py_None) return fresh(size, at::kBFloat16, like);
    const at::Tensor& t = dev(o, at::kBFloat16);
    want(t.sizes() == size);
    return t;
}

void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

template <class F>
int call(F f) {                                           // other threads run meanwhile, as they do under ctypes
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

template <class F>
PyObject* guarded(F f) {
    try {
        want(bound && at::impl::PythonTorchFunctionTLS::stack_len() == 0);
        return f();
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

PyObject* wrap(int rc, const at::Tensor& t) { return rc ? PyLong_FromLong(rc) : THPVariable_Wrap(t); }

PyObject* wrap(int rc, std::initializer_list<at::Tensor> ts) {
    if (rc) return PyLong_FromLong(rc);
    PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
    Py_ssize_t i = 0;
    for (const at::Tensor& t : ts) PyTuple_SET_ITEM(r, i++, THPVariable_Wrap(t));
    return r;
}

struct Gemm {                                             // operands shared by the GEMM calls
    const at::Tensor &A, &a_scale, &W, &gs;
    float ts;
    int M, N, K;
    Gemm(PyObject* const* a) : A(dev(a[0], at::kByte)), a_scale(dev(a[1], at::kFloat)), W(dev(a[2], at::kByte)), gs(dev(a[3], at::kByte)),
                               ts(number(a[4])), N(whole(a[5])) {
        want(A.dim() == 2 && A.size(0) <= INT_LIMIT && A.size(1) <= INT_LIMIT);
        M = (int)A.size(0);
        K = (int)A.size(1);
        want(M > 0 && N > 0 && K > 0 && K % GROUP == 0 && a_scale.numel() == M && gs.numel() == (int64_t)N * (K / GROUP) &&
             (size_t)W.numel() >= api.packed_weight_bytes(N, K));
    }
    const uint8_t* a() const { return (const uint8_t*)A.data_ptr(); }
    const float* s() const { return (const float*)a_scale.data_ptr(); }
    const uint8_t* w() const { return (const uint8_t*)W.data_ptr(); }
    const uint8_t* g() const { return (const uint8_t*)gs.data_ptr(); }
};

// quantize_act(X, workspace)
PyObject* quantize_act(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&] {
        want(n == 2);
        const at::Tensor& X = dev(a[0], at::kBFloat16);
        want(X.dim() == 2 && X.size(0) > 0 && X.size(1) > 0 && X.size(0) <= INT_LIMIT && X.size(1) <= INT_LIMIT);
        const int M = (int)X.size(0), K = (int)X.size(1);
        at::Tensor A = fresh({M, K}, at::kByte, X), s = fresh({M}, at::kFloat, X);
        const Scratch ws(a[1], 0, X);
        const uint16_t* x = (const uint16_t*)X.data_ptr();
        uint8_t* pa = (uint8_t*)A.data_ptr();
        float* ps = (float*)s.data_ptr();
        void* st = stream();
        const bool with = a[1] != Py_None;
        const int rc = call([&] { return with ? api.quantize_act_ws(x, pa, ps, M, K, ws.p, ws.bytes, st) : api.quantize_act(x, pa, ps, M, K, st); });
        return wrap(rc, {A, s});
    });
}

// gemm(A, a_scale, W, gs, ts, N, out, workspace, prepared), swiglu(the same), add(the same with the residual at the end)
enum class Mode { Plain, Swiglu, Add };
template <Mode MODE>
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&] {
        want(n == (MODE == Mode::Add ? 10 : 9));
        const Gemm o(a);
        want(MODE != Mode::Swiglu || o.N % 2 == 0);
        const at::Tensor Y = output(a[6], {o.M, MODE == Mode::Swiglu ? o.N / 2 : o.N}, o.A);
        const uint16_t* r = nullptr;
        if (MODE == Mode::Add) {
            const at::Tensor& R = dev(a[9], at::kBFloat16);
            want(R.dim() == 2 && R.size(0) == o.M && R.size(1) == o.N);
            r = (const uint16_t*)R.data_ptr();
        }
        const Scratch ws(a[7], api.gemm_workspace_bytes(o.M, o.N, o.K), o.A);
        const int prepared = truth(a[8]) && a[7] != Py_None ? 1 : 0;
        uint16_t* y = (uint16_t*)Y.data_ptr();
        const uint8_t *pa = o.a(), *pw = o.w(), *pg = o.g();
        const float* ps = o.s();
        void* st = stream();
        const int rc = call([&] {
            return MODE == Mode::Plain ? api.gemm_ws(pa, ps, pw, pg, o.ts, y, o.M, o.N, o.K, ws.p, ws.bytes, prepared, st)
                 : MODE == Mode::Swiglu ? api.gemm_swiglu_ws(pa, ps, pw, pg, o.ts, y, o.M, o.N, o.K, ws.p, ws.bytes, prepared, st)
                                        : api.gemm_add_ws(pa, ps, pw, pg, o.ts, r, y, o.M, o.N, o.K, ws.p, ws.bytes, prepared, st);
        });
        return wrap(rc, Y);
    });
}

// swiglu_quant(A, a_scale, W, gs, ts, N, out, workspace, prepared, next_workspace)
PyObject* swiglu_quant(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&] {
        want(n == 10);
        const Gemm o(a);
        want(o.N % 2 == 0);
        const int NH = o.N / 2;
        const at::Tensor H = output(a[6], {o.M, NH}, o.A);
        at::Tensor codes = fresh({o.M, NH}, at::kByte, o.A), scales = fresh({o.M}, at::kFloat, o.A);
        const Scratch ws(a[7], api.gemm_workspace_bytes(o.M, o.N, o.K), o.A), next(a[9], 0, o.A);
        const int prepared = truth(a[8]) && a[7] != Py_None ? 1 : 0;
        uint16_t* h = (uint16_t*)H.data_ptr();
        uint8_t* pc = (uint8_t*)codes.data_ptr();
        float* psc = (float*)scales.data_ptr();
        const uint8_t *pa = o.a(), *pw = o.w(), *pg = o.g();
        const float* ps = o.s();
        void* st = stream();
        const int rc = call([&] {
            return api.gemm_swiglu_quant_ws(pa, ps, pw, pg, o.ts, h, pc, psc, o.M, o.N, o.K, ws.p, ws.bytes, prepared, next.p, next.bytes, st);
        });
        return wrap(rc, {H, codes, scales});
    });
}

// linear(X, W, gs, ts, N, out, workspace)
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&] {
        want(n == 7);
        const at::Tensor &X = dev(a[0], at::kBFloat16), &W = dev(a[1], at::kByte), &G = dev(a[2], at::kByte);
        const float ts = number(a[3]);
        const int N = whole(a[4]);
        want(X.dim() == 2 && X.size(0) <= INT_LIMIT && X.size(1) <= INT_LIMIT);
        const int M = (int)X.size(0), K = (int)X.size(1);
        want(M > 0 && N > 0 && K > 0 && K % GROUP == 0 && G.numel() == (int64_t)N * (K / GROUP) &&
             (size_t)W.numel() >= api.packed_weight_bytes(N, K));
        const at::Tensor Y = output(a[5], {M, N}, X);
        const Scratch ws(a[6], a[6] == Py_None ? api.linear_workspace_bytes(M, N, K) : 0, X);
        const uint16_t* x = (const uint16_t*)X.data_ptr();
        const uint8_t *w = (const uint8_t*)W.data_ptr(), *g = (const uint8_t*)G.data_ptr();
        uint16_t* y = (uint16_t*)Y.data_ptr();
        void* st = stream();
        const int rc = call([&] { return api.linear_ws(x, w, g, ts, y, M, N, K, ws.p, ws.bytes, st); });
        return wrap(rc, Y);
    });
}

// kv4_scores(Q, q_scale, K_packed, k_scale, out_scale)
PyObject* kv4_scores(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&] {
        want(n == 5);
        const at::Tensor &Q = dev(a[0], at::kByte), &qs = dev(a[1], at::kFloat), &kp = dev(a[2], at::kByte), &ks = dev(a[3], at::kByte);
        const float scale = number(a[4]);
        want(Q.dim() == 3 && qs.dim() == 2 && ks.dim() == 2);
        const int64_t h = Q.size(0), r = Q.size(1), t = ks.size(1);
        want(h > 0 && r > 0 && t > 0 && h <= INT_LIMIT && r <= INT_LIMIT && t <= INT_LIMIT && Q.size(2) == GROUP && qs.size(0) == h &&
             qs.size(1) == r && ks.size(0) == h);
        const int H = (int)h, R = (int)r, T = (int)t;
        want((size_t)kp.numel() >= api.kv4_packed_bytes(H, T, 0));
        at::Tensor S = fresh({h, r, t}, at::kBFloat16, Q);
        const uint8_t *q = (const uint8_t*)Q.data_ptr(), *k = (const uint8_t*)kp.data_ptr(), *s = (const uint8_t*)ks.data_ptr();
        const float* f = (const float*)qs.data_ptr();
        uint16_t* o = (uint16_t*)S.data_ptr();
        void* st = stream();
        const int rc = call([&] { return api.kv4_scores(q, f, k, s, scale, o, H, R, T, st); });
        return wrap(rc, S);
    });
}

// kv4_output(P, p_scale, V_packed, v_scale)
PyObject* kv4_output(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&] {
        want(n == 4);
        const at::Tensor &P = dev(a[0], at::kByte), &ps = dev(a[1], at::kFloat), &vp = dev(a[2], at::kByte), &vs = dev(a[3], at::kByte);
        want(P.dim() == 3 && ps.dim() == 2 && vs.dim() == 2);
        const int64_t h = P.size(0), r = P.size(1), l = P.size(2), t = vs.size(1);
        want(h > 0 && r > 0 && t > 0 && h <= INT_LIMIT && r <= INT_LIMIT && l <= INT_LIMIT && l >= t && ps.size(0) == h && ps.size(1) == r &&
             vs.size(0) == h);
        const int H = (int)h, R = (int)r, T = (int)t, ldp = (int)l;
        want((size_t)vp.numel() >= api.kv4_packed_bytes(H, T, 1));
        at::Tensor O = fresh({h, r, GROUP}, at::kBFloat16, P);
        const Scratch ws(Py_None, api.kv4_output_workspace_bytes(H, R, T), P);
        const uint8_t *p = (const uint8_t*)P.data_ptr(), *v = (const uint8_t*)vp.data_ptr(), *s = (const uint8_t*)vs.data_ptr();
        const float* f = (const float*)ps.data_ptr();
        uint16_t* o = (uint16_t*)O.data_ptr();
        void* st = stream();
        const int rc = call([&] { return api.kv4_output_ws(p, f, v, s, o, H, R, T, ldp, ws.p, ws.bytes, st); });
        return wrap(rc, O);
    });
}

// kv4_pack(codes, values)
PyObject* kv4_pack(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&] {
        want(n == 2);
        const at::Tensor& C = dev(a[0], at::kChar);
        const int values = truth(a[1]) ? 1 : 0;
        want(C.dim() == 3 && C.size(0) > 0 && C.size(1) > 0 && C.size(0) <= INT_LIMIT && C.size(1) <= INT_LIMIT && C.size(2) == GROUP);
        const int H = (int)C.size(0), T = (int)C.size(1);
        at::Tensor out = fresh({(int64_t)api.kv4_packed_bytes(H, T, values)}, at::kByte, C);
        const int8_t* c = (const int8_t*)C.data_ptr();
        uint8_t* o = (uint8_t*)out.data_ptr();
        void* st = stream();
        const int rc = call([&] { return api.kv4_pack(c, o, H, T, values, st); });
        return wrap(rc, out);
    });
}

struct Matrix {                                           // a weight matrix [N,K] of the offline calls
    const at::Tensor& W;
    int N, K;
    Matrix(PyObject* o, at::ScalarType t) : W(dev(o, t)) {
        want(W.dim() == 2 && W.size(0) > 0 && W.size(1) > 0 && W.size(0) <= INT_LIMIT && W.size(1) <= INT_LIMIT);
        N = (int)W.size(0);
        K = (int)W.size(1);
    }
    const uint16_t* w() const { return (const uint16_t*)W.data_ptr(); }
    const float* lambda(PyObject* o) const {              // the channels' scales, or none
        if (o == Py_None) return nullptr;
        const at::Tensor& l = dev(o, at::kFloat);
        want(l.numel() == K);
        return (const float*)l.data_ptr();
    }
};

// pack_weights(q)
PyObject* pack_weights(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&] {
        want(n == 1);
        const Matrix m(a[0], at::kChar);
        const size_t bytes = api.packed_weight_bytes(m.N, m.K);
        want(bytes > 0);
        at::Tensor out = fresh({(int64_t)bytes}, at::kByte, m.W);
        const int8_t* q = (const int8_t*)m.W.data_ptr();
        uint8_t* o = (uint8_t*)out.data_ptr();
        void* st = stream();
        const int rc = call([&] { return api.pack_weights(q, o, m.N, m.K, st); });
        return wrap(rc, out);
    });
}

// cas_scales(W, target)
PyObject* cas_scales(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&] {
        want(n == 2);
        const Matrix m(a[0], at::kBFloat16);
        const float target = number(a[1]);
        at::Tensor out = fresh({m.K}, at::kFloat, m.W);
        const Scratch ws(Py_None, api.cas_scales_workspace_bytes(m.N, m.K), m.W);
        const uint16_t* w = m.w();
        float* o = (float*)out.data_ptr();
        void* st = stream();
        const int rc = call([&] { return api.cas_scales_ws(w, target, o, m.N, m.K, ws.p, ws.bytes, st); });
        return wrap(rc, out);
    });
}

// pts_exponent(W, lam)
PyObject* pts_exponent(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&] {
        want(n == 2);
        const Matrix m(a[0], at::kBFloat16);
        const float* lam = m.lambda(a[1]);
        at::Tensor out = fresh({16}, at::kInt, m.W);
        const Scratch ws(Py_None, api.pts_exponent_workspace_bytes(m.N, m.K), m.W);
        const uint16_t* w = m.w();
        int* o = (int*)out.data_ptr();
        void* st = stream();
        const int rc = call([&] { return api.pts_exponent_ws(w, lam, o, m.N, m.K, ws.p, ws.bytes, st); });
        return wrap(rc, out);
    });
}

// quantize_weights(W, lam, n_pts, sigma_nearest)
PyObject* quantize_weights(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&] {
        want(n == 4);
        const Matrix m(a[0], at::kBFloat16);
        const float* lam = m.lambda(a[1]);
        const int n_pts = whole(a[2]), nearest = truth(a[3]) ? 1 : 0;
        want(m.K % GROUP == 0);
        at::Tensor q = fresh({m.N, m.K}, at::kChar, m.W), gs = fresh({m.N, m.K / GROUP}, at::kByte, m.W);
        const uint16_t* w = m.w();
        int8_t* pq = (int8_t*)q.data_ptr();
        uint8_t* pg = (uint8_t*)gs.data_ptr();
        void* st = stream();
        const int rc = call([&] { return api.quantize_weights(w, lam, n_pts, nearest, pq, pg, m.N, m.K, st); });
        return wrap(rc, {q, gs});
    });
}

// gemm_workspace_bytes(M, N, K)
PyObject* gemm_workspace_bytes(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&] {
        want(n == 3);
        return PyLong_FromSize_t(api.gemm_workspace_bytes(whole(a[0]), whole(a[1]), whole(a[2])));
    });
}

// bind(addresses of the C functions, in the order of Api)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    constexpr Py_ssize_t COUNT = sizeof(Api) / sizeof(void*);
    if (n != COUNT) {
        PyErr_SetString(PyExc_TypeError, "bind() takes the address of every C function");
        return nullptr;
    }
    void* p[COUNT];
    for (Py_ssize_t i = 0; i < COUNT; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind(): a NULL address");
            return nullptr;
        }
    }
    __builtin_memcpy(&api, p, sizeof(api));
    bound = true;
    Py_RETURN_NONE;
}

#define FQ_METHOD(name, fn) {name, (PyCFunction)(void (*)(void))(fn), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    FQ_METHOD("bind", bind),
    FQ_METHOD("quantize_act", quantize_act),
    FQ_METHOD("gemm", gemm<Mode::Plain>),
    FQ_METHOD("gemm_swiglu", gemm<Mode::Swiglu>),
    FQ_METHOD("gemm_add", gemm<Mode::Add>),
    FQ_METHOD("gemm_swiglu_quant", swiglu_quant),
    FQ_METHOD("linear", linear),
    FQ_METHOD("kv4_scores", kv4_scores),
    FQ_METHOD("kv4_output", kv4_output),
    FQ_METHOD("kv4_pack", kv4_pack),
    FQ_METHOD("pack_weights", pack_weights),
    FQ_METHOD("cas_scales", cas_scales),
    FQ_METHOD("pts_exponent", pts_exponent),
    FQ_METHOD("quantize_weights", quantize_weights),
    FQ_METHOD("gemm_workspace_bytes", gemm_workspace_bytes),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fq_marshal", "argument marshalling of the fireq binding", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fq_marshal(void) { return PyModule_Create(&module); }
