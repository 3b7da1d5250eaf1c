// Native call path of the Python binding: one call checks every tensor,
// allocates the outputs that were not given, takes the current stream and
// calls the C ABI.  The same work in Python (six attribute reads and
// comparisons per tensor, a 20-argument ctypes call) took 16 to 19 us a
// call, two to three times what the kernels of a small draft take.
//
// Each function returns the call's result tuple or tensor when everything is
// as the library wants it, the status (an int) when the library refused the
// call, and None when any argument is not plainly acceptable.  For None the
// caller repeats the call through Python, whose checks say what is wrong.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <ATen/TensorSubclassLikeUtils.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>

#include "treewy.h"

namespace {

using at::Tensor;

struct Refused {};                                       // -> None

// A plain dense GPU tensor on the current device, and nothing that wraps one
// (a subclass, a tensor under vmap or another transform).
const Tensor &tensor(PyObject *x, int device) {
    if (!THPVariable_CheckExact(x)) throw Refused{};
    const Tensor &t = THPVariable_Unpack(x);
    if (!t.defined() || t.layout() != at::kStrided || !t.device().is_cuda() || t.device().index() != device ||
        !t.has_storage() || at::isTensorSubclassLike(t))
        throw Refused{};
    return t;
}

const Tensor &need(PyObject *x, int device, at::ScalarType dtype, at::IntArrayRef shape) {
    const Tensor &t = tensor(x, device);
    if (t.scalar_type() != dtype || t.sizes() != shape || !t.is_contiguous()) throw Refused{};
    return t;
}

void *ptr(const Tensor &t) { return t.data_ptr(); }

// A tensor of the wanted shape, or null for None.
void *need_or_null(PyObject *x, int device, at::ScalarType dtype, at::IntArrayRef shape) {
    return x == Py_None ? nullptr : ptr(need(x, device, dtype, shape));
}

// The given output, or a new one.
Tensor output(PyObject *x, int device, at::ScalarType dtype, at::IntArrayRef shape) {
    if (x != Py_None) return need(x, device, dtype, shape);
    return at::empty(shape, at::TensorOptions().dtype(dtype).device(at::kCUDA, device));
}

treewy_dtype token_type(const Tensor &t) {
    if (t.scalar_type() == at::kBFloat16) return TREEWY_BF16;
    if (t.scalar_type() == at::kFloat) return TREEWY_F32;
    throw Refused{};
}

int64_t dim(const Tensor &t, int nd, int i) {
    if (t.dim() != nd || t.size(i) > INT32_MAX) throw Refused{};
    return t.size(i);
}

void *stream_of(PyObject *s, int device) {
    if (s == Py_None) return c10::hip::getCurrentHIPStream((c10::DeviceIndex)device).stream();
    PyObject *h = PyObject_GetAttrString(s, "cuda_stream");
    if (!h) {
        PyErr_Clear();
        throw Refused{};
    }
    void *p = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        throw Refused{};
    }
    return p;
}

// What the call returns, wrapped before the launch: a failure up to there
// leaves the call to Python with nothing done, and past it nothing can fail
// (repeated through Python, a commit in place would be applied twice).
struct Result {
    PyObject *r = nullptr;
    explicit Result(std::initializer_list<Tensor> out) {
        r = out.size() == 1 ? THPVariable_Wrap(*out.begin()) : PyTuple_New((Py_ssize_t)out.size());
        if (!r) throw Refused{};
        if (out.size() == 1) return;
        Py_ssize_t i = 0;
        for (const Tensor &t : out) {
            PyObject *x = THPVariable_Wrap(t);
            if (!x) {
                Py_CLEAR(r);
                throw Refused{};
            }
            PyTuple_SET_ITEM(r, i++, x);
        }
    }
    Result(const Result &) = delete;
    ~Result() { Py_XDECREF(r); }
    // The result, or the status of a refused call (a small int: always there).
    PyObject *after(treewy_status st) {
        if (st != TREEWY_OK) return PyLong_FromLong(st);
        PyObject *x = r;
        r = nullptr;
        return x;
    }
};

// Runs f(args, current device); None where it threw.
template <typename F>
PyObject *guarded(PyObject *const *, Py_ssize_t n, Py_ssize_t want, F &&f) {
    if (n != want) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    try {
        return f((int)c10::hip::current_device());
    } catch (...) {                                      // (nothing is launched yet; an allocation that failed: Python says so)
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// The C call itself, without the interpreter lock.  Its arguments are values
// taken before the lock is let go: taking a tensor's pointer can throw (one
// whose storage gives none out, or a lazy copy that is made there).
template <typename T> struct Same { using type = T; };
template <typename... A> treewy_status unlocked(treewy_status (*f)(A...), typename Same<A>::type... a) {
    struct Unlocked {
        PyThreadState *state = PyEval_SaveThread();
        ~Unlocked() { PyEval_RestoreThread(state); }
    } lock;
    return f(a...);
}

constexpr at::ScalarType F32 = at::kFloat, I32 = at::kInt;

// S0, q, k, v, alpha, beta, parent, o, U, err, stream -> (o, U)
PyObject *verify(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(a, n, 11, [&](int d) {
        const Tensor &S0 = tensor(a[0], d), &q = tensor(a[1], d), &v = tensor(a[3], d);
        const int64_t B = dim(q, 4, 0), H = dim(q, 4, 1), N = dim(q, 4, 2), dk = dim(q, 4, 3), dv = dim(v, 4, 3);
        const auto dt = q.scalar_type(), sdt = S0.scalar_type();
        const treewy_dtype in = token_type(q), state = token_type(S0);
        need(a[0], d, sdt, {B, H, dv, dk});
        need(a[1], d, dt, {B, H, N, dk});
        const Tensor &k = need(a[2], d, dt, {B, H, N, dk});
        need(a[3], d, dt, {B, H, N, dv});
        const Tensor &al = need(a[4], d, F32, {B, H, N}), &be = need(a[5], d, F32, {B, H, N});
        const Tensor &par = need(a[6], d, I32, {B, N});
        void *err = need_or_null(a[9], d, I32, {B}), *s = stream_of(a[10], d);
        const Tensor o = output(a[7], d, dt, {B, H, N, dv}), U = output(a[8], d, F32, {B, H, N, dv});
        Result result({o, U});
        return result.after(unlocked(treewy_verify, ptr(S0), ptr(q), ptr(k), ptr(v), (float *)ptr(al),
                                     (float *)ptr(be), (int32_t *)ptr(par), (int)N, (int)B, (int)H, (int)dk,
                                     (int)dv, in, state, ptr(o), (float *)ptr(U), (int32_t *)err, s));
    });
}

// S0, U, k, alpha, path, path_len, parent, S_new, err, stream -> S_new
PyObject *commit(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(a, n, 10, [&](int d) {
        const Tensor &S0 = tensor(a[0], d), &U = tensor(a[1], d), &k = tensor(a[2], d), &path = tensor(a[4], d);
        const int64_t B = dim(k, 4, 0), H = dim(k, 4, 1), N = dim(k, 4, 2), dk = dim(k, 4, 3), dv = dim(U, 4, 3);
        const int64_t L = dim(path, 2, 1);
        const auto sdt = S0.scalar_type();
        const treewy_dtype in = token_type(k), state = token_type(S0);
        need(a[0], d, sdt, {B, H, dv, dk});
        need(a[1], d, F32, {B, H, N, dv});
        need(a[2], d, k.scalar_type(), {B, H, N, dk});
        const Tensor &al = need(a[3], d, F32, {B, H, N});
        need(a[4], d, I32, {B, L});
        const Tensor &len = need(a[5], d, I32, {B});
        void *par = need_or_null(a[6], d, I32, {B, N}), *err = need_or_null(a[8], d, I32, {B}), *s = stream_of(a[9], d);
        const Tensor S_new = output(a[7], d, sdt, {B, H, dv, dk});
        Result result({S_new});
        return result.after(unlocked(treewy_commit, ptr(S0), (float *)ptr(U), ptr(k), (float *)ptr(al),
                                     (int32_t *)ptr(path), (int32_t *)ptr(len), (int)L, (int32_t *)par, (int)N,
                                     (int)B, (int)H, (int)dk, (int)dv, in, state, ptr(S_new), (int32_t *)err, s));
    });
}

// S_old, U_prev, k_prev, alpha_prev, path, path_len, q, k, v, alpha, beta, parent, parent_prev, S_new, o, U, err,
// stream -> (S_new, o, U)
PyObject *commit_verify(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(a, n, 18, [&](int d) {
        const Tensor &S = tensor(a[0], d), &kp = tensor(a[2], d), &path = tensor(a[4], d), &q = tensor(a[6], d),
                     &v = tensor(a[8], d);
        const int64_t B = dim(q, 4, 0), H = dim(q, 4, 1), N = dim(q, 4, 2), dk = dim(q, 4, 3), dv = dim(v, 4, 3);
        const int64_t Np = dim(kp, 4, 2), L = dim(path, 2, 1);
        const auto dt = q.scalar_type(), sdt = S.scalar_type();
        const treewy_dtype in = token_type(q), state = token_type(S);
        need(a[0], d, sdt, {B, H, dv, dk});
        const Tensor &Up = need(a[1], d, F32, {B, H, Np, dv});
        need(a[2], d, dt, {B, H, Np, dk});
        const Tensor &alp = need(a[3], d, F32, {B, H, Np});
        need(a[4], d, I32, {B, L});
        const Tensor &len = need(a[5], d, I32, {B});
        need(a[6], d, dt, {B, H, N, dk});
        const Tensor &k = need(a[7], d, dt, {B, H, N, dk});
        need(a[8], d, dt, {B, H, N, dv});
        const Tensor &al = need(a[9], d, F32, {B, H, N}), &be = need(a[10], d, F32, {B, H, N});
        const Tensor &par = need(a[11], d, I32, {B, N});
        void *parp = need_or_null(a[12], d, I32, {B, Np}), *err = need_or_null(a[16], d, I32, {B}),
             *s = stream_of(a[17], d);
        const Tensor S_new = output(a[13], d, sdt, {B, H, dv, dk}), o = output(a[14], d, dt, {B, H, N, dv}),
                     U = output(a[15], d, F32, {B, H, N, dv});
        Result result({S_new, o, U});
        return result.after(unlocked(treewy_commit_verify, ptr(S), (float *)ptr(Up), ptr(kp), (float *)ptr(alp),
                                     (int32_t *)ptr(path), (int32_t *)ptr(len), (int)L, (int32_t *)parp, (int)Np,
                                     ptr(q), ptr(k), ptr(v), (float *)ptr(al), (float *)ptr(be),
                                     (int32_t *)ptr(par), (int)N, (int)B, (int)H, (int)dk, (int)dv, in, state,
                                     ptr(S_new), ptr(o), (float *)ptr(U), (int32_t *)err, s));
    });
}

// S0, q, k, v, alpha, beta, S_T, o, err, stream -> (S_T, o)
PyObject *chain_prefill(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(a, n, 10, [&](int d) {
        const Tensor &S0 = tensor(a[0], d), &q = tensor(a[1], d), &v = tensor(a[3], d);
        const int64_t B = dim(q, 4, 0), H = dim(q, 4, 1), T = dim(q, 4, 2), dk = dim(q, 4, 3), dv = dim(v, 4, 3);
        const auto dt = q.scalar_type(), sdt = S0.scalar_type();
        const treewy_dtype in = token_type(q), state = token_type(S0);
        need(a[0], d, sdt, {B, H, dv, dk});
        need(a[1], d, dt, {B, H, T, dk});
        const Tensor &k = need(a[2], d, dt, {B, H, T, dk});
        need(a[3], d, dt, {B, H, T, dv});
        const Tensor &al = need(a[4], d, F32, {B, H, T}), &be = need(a[5], d, F32, {B, H, T});
        void *err = need_or_null(a[8], d, I32, {B}), *s = stream_of(a[9], d);
        const Tensor S_T = output(a[6], d, sdt, {B, H, dv, dk}), o = output(a[7], d, dt, {B, H, T, dv});
        Result result({S_T, o});
        return result.after(unlocked(treewy_chain_prefill, ptr(S0), ptr(q), ptr(k), ptr(v), (float *)ptr(al),
                                     (float *)ptr(be), (int)T, (int)B, (int)H, (int)dk, (int)dv, in, state,
                                     ptr(S_T), ptr(o), (int32_t *)err, s));
    });
}

// parent, draft_token, target_token, root_token, L_max, path, path_len, bonus, err, stream -> (path, path_len, bonus)
PyObject *accept_greedy(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(a, n, 10, [&](int d) {
        const Tensor &par = tensor(a[0], d);
        const int64_t B = dim(par, 2, 0), N = dim(par, 2, 1);
        if (!PyLong_CheckExact(a[4])) throw Refused{};
        int overflow = 0;
        const long L = PyLong_AsLongAndOverflow(a[4], &overflow);
        if (overflow || L < 0 || L > INT32_MAX) throw Refused{};
        need(a[0], d, I32, {B, N});
        const Tensor &dr = need(a[1], d, I32, {B, N}), &tg = need(a[2], d, I32, {B, N}), &rt = need(a[3], d, I32, {B});
        void *err = need_or_null(a[8], d, I32, {B}), *s = stream_of(a[9], d);
        const Tensor path = output(a[5], d, I32, {B, L}), len = output(a[6], d, I32, {B}), bonus = output(a[7], d, I32, {B});
        Result result({path, len, bonus});
        return result.after(unlocked(treewy_accept_greedy, (int32_t *)ptr(par), (int32_t *)ptr(dr),
                                     (int32_t *)ptr(tg), (int32_t *)ptr(rt), (int)N, (int)B, (int)L,
                                     (int32_t *)ptr(path), (int32_t *)ptr(len), (int32_t *)ptr(bonus),
                                     (int32_t *)err, s));
    });
}

#define TREEWY_METHOD(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {TREEWY_METHOD(verify),        TREEWY_METHOD(commit),        TREEWY_METHOD(commit_verify),
                         TREEWY_METHOD(chain_prefill), TREEWY_METHOD(accept_greedy), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
