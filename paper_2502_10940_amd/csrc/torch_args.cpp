// torch_args.cpp -- the layer and group calls of cola.py with their checks in
// native code (CPython extension _torch_args).
//
// cola.py checks every tensor against the descriptor before a call (dtype,
// shape, strides, storage, device).  In Python that and the argument conversion
// cost 10 us of a forward call and 17 us of a backward call, as much as the
// kernels of a small layer take; here about 1 us.  Each function takes the
// arguments of the cola.py function of the same name (with the stream as an
// integer) and returns the library's status, or None when any argument is not
// the plain case (a tensor of the expected kind, or None where that is allowed):
// cola.py then runs its own checks, which raise the error or take the call.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/cola.h"

namespace {

// dims a tensor must cover, in elements
struct Need {
    int64_t rows, width, ld;
    at::ScalarType dtype;
};

// Device pointer of a plain tensor on a GPU that holds `need`; false if it is
// anything else.
bool take(PyObject* o, const Need& need, void** out) {
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.has_storage() || !t.is_cuda() || t.scalar_type() != need.dtype || t.dim() != 2) return false;
    if (t.size(0) < need.rows || t.size(1) < need.width) return false;
    if (t.stride(1) != 1 || (need.rows > 1 && t.stride(0) != need.ld)) return false;
    const int64_t es = (int64_t)t.element_size();
    if ((int64_t)t.storage().nbytes() - t.storage_offset() * es < need.rows * need.ld * es) return false;
    *out = t.data_ptr();
    return true;
}

bool take_or_none(PyObject* o, const Need& need, void** out) {
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    return take(o, need, out);
}

bool take_list(PyObject* o, const Need* need, int n, void** out) {
    if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return false;
    if (PySequence_Fast_GET_SIZE(o) != n) return false;
    for (int i = 0; i < n; ++i)
        if (!take(PySequence_Fast_GET_ITEM(o, i), need[i], &out[i])) return false;
    return true;
}

// The workspace and its size (None: the whole tensor).
bool take_ws(PyObject* ws, PyObject* bytes, void** out, size_t* n) {
    *out = nullptr;
    *n = 0;
    if (ws == Py_None) return bytes == Py_None;
    if (!THPVariable_CheckExact(ws)) return false;
    const at::Tensor& t = THPVariable_Unpack(ws);
    if (!t.has_storage() || !t.is_cuda() || !t.is_contiguous()) return false;
    const int64_t have = (int64_t)t.numel() * (int64_t)t.element_size();
    int64_t want = have;
    if (bytes != Py_None) {
        if (!PyLong_CheckExact(bytes)) return false;
        want = PyLong_AsLongLong(bytes);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            return false;
        }
    }
    if (want < 0 || want > have) return false;
    *out = t.data_ptr();
    *n = (size_t)want;
    return true;
}

bool take_int(PyObject* o, int64_t* out) {
    if (!PyLong_CheckExact(o)) return false;
    *out = PyLong_AsLongLong(o);
    if (!PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}

// A ctypes descriptor's bytes.
template <class Desc>
bool take_desc(PyObject* o, Desc* out) {
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return false;
    }
    const bool ok = b.len == (Py_ssize_t)sizeof(Desc);
    if (ok) memcpy(out, b.buf, sizeof(Desc));
    PyBuffer_Release(&b);
    return ok;
}

constexpr int64_t kMaxDim = int64_t(1) << 31;          // products of two dimensions stay below 2^63
bool dim_ok(int64_t v) { return v >= 1 && v <= kMaxDim; }

struct Layer {
    cola_desc d;
    Need x, y, z, a, b, da, db;

    bool init(PyObject* o) {
        if (!take_desc(o, &d) || (d.dtype != COLA_F32 && d.dtype != COLA_BF16)) return false;
        if (d.ldx < 0 || d.ldy < 0 || d.ldz < 0) return false;
        const int64_t ldx = d.ldx ? d.ldx : d.d_in, ldy = d.ldy ? d.ldy : d.d_out, ldz = d.ldz ? d.ldz : d.r;
        for (int64_t v : {d.T, d.d_in, d.d_out, d.r, ldx, ldy, ldz})
            if (!dim_ok(v)) return false;
        const at::ScalarType t = d.dtype == COLA_BF16 ? at::kBFloat16 : at::kFloat;
        x = Need{d.T, d.d_in, ldx, t};
        y = Need{d.T, d.d_out, ldy, t};
        z = Need{d.T, d.r, ldz, t};
        a = Need{d.r, d.d_in, d.d_in, t};
        b = Need{d.d_out, d.r, d.r, t};
        da = Need{d.r, d.d_in, d.d_in, at::kFloat};
        db = Need{d.d_out, d.r, d.r, at::kFloat};
        return true;
    }
};

struct Group {
    cola_group_desc d;
    Need x, z, a, da, y[COLA_GROUP_MAX], b[COLA_GROUP_MAX], db[COLA_GROUP_MAX];

    bool init(PyObject* o) {
        if (!take_desc(o, &d) || (d.dtype != COLA_F32 && d.dtype != COLA_BF16)) return false;
        if (d.n < 1 || d.n > COLA_GROUP_MAX || d.ldx < 0 || d.ldz < 0) return false;
        const at::ScalarType t = d.dtype == COLA_BF16 ? at::kBFloat16 : at::kFloat;
        int64_t R = 0;
        for (int p = 0; p < d.n; ++p) {
            if (d.ldy[p] < 0 || !dim_ok(d.r[p]) || !dim_ok(d.d_out[p])) return false;
            const int64_t ldy = d.ldy[p] ? d.ldy[p] : d.d_out[p];
            if (!dim_ok(ldy)) return false;
            R += d.r[p];
            y[p] = Need{d.T, d.d_out[p], ldy, t};
            b[p] = Need{d.d_out[p], d.r[p], d.r[p], t};
            db[p] = Need{d.d_out[p], d.r[p], d.r[p], at::kFloat};
        }
        const int64_t ldx = d.ldx ? d.ldx : d.d_in, ldz = d.ldz ? d.ldz : R;
        for (int64_t v : {d.T, d.d_in, R, ldx, ldz})
            if (!dim_ok(v)) return false;
        x = Need{d.T, d.d_in, ldx, t};
        z = Need{d.T, R, ldz, t};
        a = Need{R, d.d_in, d.d_in, t};
        da = Need{R, d.d_in, d.d_in, at::kFloat};
        return true;
    }
};

using Args = PyObject* const*;

// Runs f (false: not the plain case; else *st holds the status).  No C++
// exception leaves.
template <class F>
PyObject* call(F&& f) {
    int st = 0;
    bool plain = false;
    try {
        plain = f(&st);
    } catch (...) {
        plain = false;
    }
    if (!plain) Py_RETURN_NONE;
    return PyLong_FromLong(st);
}

struct Tail {                                            // ws, ws_bytes, stream
    void* ws;
    size_t n;
    int64_t stream;
    bool init(Args v) { return take_ws(v[0], v[1], &ws, &n) && take_int(v[2], &stream); }
    cola_stream_t s() const { return reinterpret_cast<cola_stream_t>(stream); }
};

// The library call itself, without the interpreter lock.
#define COLA_CALL(expr)        \
    Py_BEGIN_ALLOW_THREADS     \
    *st = (expr);              \
    Py_END_ALLOW_THREADS       \
    return true

PyObject* fwd(PyObject*, Args v, Py_ssize_t n) {         // d, X, A, B, Y, Z, H, ws, ws_bytes, stream
    return call([&](int* st) {
        Layer l;
        Tail t;
        void *X, *A, *B, *Y, *Z, *H;
        if (n != 10 || !l.init(v[0]) || !take(v[1], l.x, &X) || !take(v[2], l.a, &A) || !take(v[3], l.b, &B) ||
            !take(v[4], l.y, &Y) || !take(v[5], l.z, &Z) || !take_or_none(v[6], l.z, &H) || !t.init(v + 7))
            return false;
        COLA_CALL(cola_fwd(&l.d, X, A, B, Y, Z, H, t.ws, t.n, t.s()));
    });
}

PyObject* fwd_outer(PyObject*, Args v, Py_ssize_t n) {   // d, outer, X, A, B, Y, P, Z, H, ws, ws_bytes, stream
    return call([&](int* st) {
        Layer l;
        Tail t;
        int64_t outer;
        void *X, *A, *B, *Y, *P, *Z, *H;
        if (n != 12 || !l.init(v[0]) || !take_int(v[1], &outer) || outer < 0 || outer > 1000 || !take(v[2], l.x, &X) ||
            !take(v[3], l.a, &A) || !take(v[4], l.b, &B) || !take(v[5], l.y, &Y) || !take(v[6], l.y, &P) ||
            !take(v[7], l.z, &Z) || !take_or_none(v[8], l.z, &H) || !t.init(v + 9))
            return false;
        COLA_CALL(cola_fwd_outer(&l.d, (int)outer, X, A, B, Y, P, Z, H, t.ws, t.n, t.s()));
    });
}

PyObject* infer(PyObject*, Args v, Py_ssize_t n) {       // d, X, A, B, Y, ws, ws_bytes, stream
    return call([&](int* st) {
        Layer l;
        Tail t;
        void *X, *A, *B, *Y;
        if (n != 8 || !l.init(v[0]) || !take(v[1], l.x, &X) || !take(v[2], l.a, &A) || !take(v[3], l.b, &B) ||
            !take(v[4], l.y, &Y) || !t.init(v + 5))
            return false;
        COLA_CALL(cola_infer(&l.d, X, A, B, Y, t.ws, t.n, t.s()));
    });
}

PyObject* bwd(PyObject*, Args v, Py_ssize_t n) {         // d, dY, X, Z, H, A, B, dX, dA, dB, ws, ws_bytes, stream
    return call([&](int* st) {
        Layer l;
        Tail t;
        void *dY, *X, *Z, *H, *A, *B, *dX, *dA, *dB;
        if (n != 13 || !l.init(v[0]) || !take(v[1], l.y, &dY) || !take(v[2], l.x, &X) || !take(v[3], l.z, &Z) ||
            !take_or_none(v[4], l.z, &H) || !take(v[5], l.a, &A) || !take(v[6], l.b, &B) || !take(v[7], l.x, &dX) ||
            !take(v[8], l.da, &dA) || !take(v[9], l.db, &dB) || !t.init(v + 10))
            return false;
        COLA_CALL(cola_bwd(&l.d, dY, X, Z, H, A, B, dX, static_cast<float*>(dA), static_cast<float*>(dB), t.ws, t.n,
                           t.s()));
    });
}

PyObject* bwd_outer(PyObject*, Args v, Py_ssize_t n) {   // d, outer, dY, P, X, Z, H, A, B, dX, dA, dB, ws, ws_bytes, stream
    return call([&](int* st) {
        Layer l;
        Tail t;
        int64_t outer;
        void *dY, *P, *X, *Z, *H, *A, *B, *dX, *dA, *dB;
        if (n != 15 || !l.init(v[0]) || !take_int(v[1], &outer) || outer < 0 || outer > 1000 || !take(v[2], l.y, &dY) ||
            !take(v[3], l.y, &P) || !take(v[4], l.x, &X) || !take(v[5], l.z, &Z) || !take_or_none(v[6], l.z, &H) ||
            !take(v[7], l.a, &A) || !take(v[8], l.b, &B) || !take(v[9], l.x, &dX) || !take(v[10], l.da, &dA) ||
            !take(v[11], l.db, &dB) || !t.init(v + 12))
            return false;
        COLA_CALL(cola_bwd_outer(&l.d, (int)outer, dY, P, X, Z, H, A, B, dX, static_cast<float*>(dA),
                                 static_cast<float*>(dB), t.ws, t.n, t.s()));
    });
}

PyObject* group_fwd(PyObject*, Args v, Py_ssize_t n) {   // d, X, A_all, B, Y, Z_all, H_all, ws, ws_bytes, stream
    return call([&](int* st) {
        Group g;
        Tail t;
        void *X, *A, *Z, *H, *B[COLA_GROUP_MAX], *Y[COLA_GROUP_MAX];
        if (n != 10 || !g.init(v[0]) || !take(v[1], g.x, &X) || !take(v[2], g.a, &A) || !take_list(v[3], g.b, g.d.n, B) ||
            !take_list(v[4], g.y, g.d.n, Y) || !take(v[5], g.z, &Z) || !take_or_none(v[6], g.z, &H) || !t.init(v + 7))
            return false;
        COLA_CALL(cola_group_fwd(&g.d, X, A, B, Y, Z, H, t.ws, t.n, t.s()));
    });
}

PyObject* group_infer(PyObject*, Args v, Py_ssize_t n) { // d, X, A_all, B, Y, ws, ws_bytes, stream
    return call([&](int* st) {
        Group g;
        Tail t;
        void *X, *A, *B[COLA_GROUP_MAX], *Y[COLA_GROUP_MAX];
        if (n != 8 || !g.init(v[0]) || !take(v[1], g.x, &X) || !take(v[2], g.a, &A) || !take_list(v[3], g.b, g.d.n, B) ||
            !take_list(v[4], g.y, g.d.n, Y) || !t.init(v + 5))
            return false;
        COLA_CALL(cola_group_infer(&g.d, X, A, B, Y, t.ws, t.n, t.s()));
    });
}

PyObject* group_bwd(PyObject*, Args v, Py_ssize_t n) {   // d, dY, X, Z_all, H_all, A_all, B, dX, dA_all, dB, ws, ws_bytes, stream
    return call([&](int* st) {
        Group g;
        Tail t;
        void *X, *Z, *H, *A, *dX, *dA, *dY[COLA_GROUP_MAX], *B[COLA_GROUP_MAX], *dB[COLA_GROUP_MAX];
        if (n != 13 || !g.init(v[0]) || !take_list(v[1], g.y, g.d.n, dY) || !take(v[2], g.x, &X) || !take(v[3], g.z, &Z) ||
            !take_or_none(v[4], g.z, &H) || !take(v[5], g.a, &A) || !take_list(v[6], g.b, g.d.n, B) ||
            !take(v[7], g.x, &dX) || !take(v[8], g.da, &dA) || !take_list(v[9], g.db, g.d.n, dB) || !t.init(v + 10))
            return false;
        float* dBf[COLA_GROUP_MAX];
        for (int p = 0; p < g.d.n; ++p) dBf[p] = static_cast<float*>(dB[p]);
        COLA_CALL(cola_group_bwd(&g.d, dY, X, Z, H, A, B, dX, static_cast<float*>(dA), dBf, t.ws, t.n, t.s()));
    });
}

#define COLA_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {COLA_METHOD(fwd),       COLA_METHOD(fwd_outer), COLA_METHOD(infer),       COLA_METHOD(bwd),
                         COLA_METHOD(bwd_outer), COLA_METHOD(group_fwd), COLA_METHOD(group_infer), COLA_METHOD(group_bwd),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_args", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_args() { return PyModule_Create(&module); }
