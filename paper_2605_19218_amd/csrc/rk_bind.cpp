// CPython side of the calls that a program makes once per generated token and layer: the arguments of rk_decode_attn,
// rk_append_decode_attn, rk_decode_attn_dual and rk_append_text_decode_attn_dual, marshalled in C.  The same through ctypes costs some 5 us a
// call (structures built field by field, a converter per argument), which is as long as a short decode runs on the device: 8 KV heads x
// 1024 tokens were called every 8.7 us, of which the device needed 5.8.
//
// Only plain arguments are taken here (the binding's own Layout and Text, integers, objects with data_ptr()); whatever else a caller
// passes is answered with None before anything has been called, and the ctypes path, which says what it accepts and what it
// raises, takes the call.  The entry points come as addresses from the loaded librotatek.so, so both paths enter the same library.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "rotatek.h"

namespace {

typedef rk_status (*decode_fn)(rk_ctx*, const rk_layout*, const void*, const void*, const void*, const float*, const float*, float,
                               void*, void*, size_t, void*);
typedef rk_status (*append_decode_fn)(rk_ctx*, const rk_layout*, const void*, const void*, const void*, const float*, const float*,
                                      void*, void*, int32_t*, float, void*, void*, size_t, void*);
typedef rk_status (*dual_fn)(rk_ctx*, const rk_layout*, const void*, const void*, const void*, const float*, const float*,
                             const rk_text*, float, void*, void*, size_t, void*);
typedef rk_status (*append_dual_fn)(rk_ctx*, const rk_layout*, const void*, const void*, const void*, const void*, const void*,
                                    const float*, const float*, const rk_text*, float, void*, void*, size_t, void*);

decode_fn fn_decode;
append_decode_fn fn_append_decode;
dual_fn fn_dual;
append_dual_fn fn_append_dual;
PyTypeObject *layout_type, *text_type;      // the binding's classes (kept alive)

PyObject *s_batch, *s_nq, *s_nkv, *s_hd, *s_keep, *s_dtype, *s_cap, *s_max_seq, *s_seq, *s_data_ptr, *s_numel, *s_esize, *s_cuda_stream,
    *s_k, *s_v, *s_max_len, *s_len, *s_strides, *s_stride, *s_shape;

// All of these return false where the argument is not of the plain kind; an exception may then be set, and the caller clears it.
bool integer(PyObject* o, long long* out)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    *out = PyLong_AsLongLongAndOverflow(o, &over);
    return over == 0 && !(*out == -1 && PyErr_Occurred());
}
bool address(PyObject* o, void** out)
{
    *out = nullptr;
    if (o == Py_None) return true;
    PyObject* p = nullptr;
    if (!PyLong_CheckExact(o)) {
        if (PyLong_Check(o)) return false;
        o = p = PyObject_CallMethodNoArgs(o, s_data_ptr);
        if (!p || !PyLong_CheckExact(p)) { Py_XDECREF(p); return false; }
    }
    const unsigned long long a = PyLong_AsUnsignedLongLong(o);
    Py_XDECREF(p);
    if (a == (unsigned long long)-1 && PyErr_Occurred()) return false;
    *out = (void*)(uintptr_t)a;
    return true;
}
bool int32_of(PyObject* o, PyObject* name, int32_t* out)
{
    PyObject* v = PyObject_GetAttr(o, name);
    long long x = 0;
    const bool ok = v && integer(v, &x) && x >= INT32_MIN && x <= INT32_MAX;
    Py_XDECREF(v);
    *out = (int32_t)x;
    return ok;
}
bool address_of(PyObject* o, PyObject* name, void** out)
{
    PyObject* v = PyObject_GetAttr(o, name);
    const bool ok = v && address(v, out);
    Py_XDECREF(v);
    return ok;
}
bool call_int(PyObject* o, PyObject* name, long long* out)
{
    PyObject* v = PyObject_CallMethodNoArgs(o, name);
    const bool ok = v && integer(v, out);
    Py_XDECREF(v);
    return ok;
}
bool layout(PyObject* o, rk_layout* L)
{
    void* seq = nullptr;
    if (Py_TYPE(o) != layout_type || !int32_of(o, s_batch, &L->batch) || !int32_of(o, s_nq, &L->n_q_heads) ||
        !int32_of(o, s_nkv, &L->n_kv_heads) || !int32_of(o, s_hd, &L->head_dim) || !int32_of(o, s_keep, &L->keep) ||
        !int32_of(o, s_dtype, &L->dtype) || !int32_of(o, s_cap, &L->capacity) || !int32_of(o, s_max_seq, &L->max_seq_len) ||
        !address_of(o, s_seq, &seq))
        return false;
    L->seq_len = (decltype(L->seq_len))seq;
    return true;
}
bool three(PyObject* t, int64_t* out)       // the first three of a tuple
{
    if (!PyTuple_Check(t) || PyTuple_GET_SIZE(t) < 3) return false;
    for (int i = 0; i < 3; ++i) {
        long long x;
        if (!integer(PyTuple_GET_ITEM(t, i), &x)) return false;
        out[i] = x;
    }
    return true;
}
bool text(PyObject* o, rk_text* T)
{
    if (Py_TYPE(o) != text_type) return false;
    void *k = nullptr, *v = nullptr, *len = nullptr;
    int64_t st[3];
    if (!address_of(o, s_k, &k) || !address_of(o, s_v, &v) || !address_of(o, s_len, &len) || !int32_of(o, s_max_len, &T->max_len)) return false;
    PyObject* key = PyObject_GetAttr(o, s_k);
    PyObject* given = key ? PyObject_GetAttr(o, s_strides) : nullptr;
    PyObject* cap = given ? PyObject_GetAttr(o, s_cap) : nullptr;
    bool ok = cap != nullptr;
    if (ok && given == Py_None) {
        PyObject* s = PyObject_CallMethodNoArgs(key, s_stride);
        ok = s && three(s, st);
        Py_XDECREF(s);
    } else if (ok) {
        ok = PyTuple_Check(given) && PyTuple_GET_SIZE(given) == 3 && three(given, st);
    }
    long long rows = 0;
    if (ok && cap == Py_None) {
        PyObject* shape = PyObject_GetAttr(key, s_shape);
        ok = shape && PyTuple_Check(shape) && PyTuple_GET_SIZE(shape) > 2 && integer(PyTuple_GET_ITEM(shape, 2), &rows);
        Py_XDECREF(shape);
    } else if (ok) {
        ok = integer(cap, &rows);
    }
    Py_XDECREF(cap);
    Py_XDECREF(given);
    Py_XDECREF(key);
    if (!ok || rows < INT32_MIN || rows > INT32_MAX) return false;
    T->k = (decltype(T->k))k;
    T->v = (decltype(T->v))v;
    T->len = (decltype(T->len))len;
    T->stride_b = st[0];
    T->stride_h = st[1];
    T->stride_t = st[2];
    T->capacity = (int32_t)rows;
    return true;
}
// scale, out, workspace, stream, workspace_bytes: how every call ends
struct Tail { float scale; void *out, *ws, *stream; size_t bytes; };
bool tail(PyObject* const* a, Tail* t)
{
    if (!PyFloat_CheckExact(a[0]) && !PyLong_CheckExact(a[0])) return false;
    const double s = PyFloat_AsDouble(a[0]);
    if (s == -1.0 && PyErr_Occurred()) return false;
    t->scale = (float)s;
    if (!address(a[1], &t->out) || !address(a[2], &t->ws)) return false;
    if (a[3] == Py_None || PyLong_CheckExact(a[3])) {
        if (!address(a[3], &t->stream)) return false;
    } else if (!address_of(a[3], s_cuda_stream, &t->stream)) {
        return false;
    }
    long long n = 0, e = 1;
    if (a[4] != Py_None) {
        if (!integer(a[4], &n)) return false;
    } else if (a[2] != Py_None) {
        if (PyLong_Check(a[2]) || !call_int(a[2], s_numel, &n) || !call_int(a[2], s_esize, &e)) return false;
    }
    t->bytes = (size_t)(n * e);
    return n >= 0 && e >= 0;
}
// To ctypes, which meets what an argument raised here again, and says it.  An interrupt or an exit comes once: it goes on.
PyObject* other_path()
{
    if (PyErr_Occurred() && !PyErr_ExceptionMatches(PyExc_Exception)) return nullptr;
    PyErr_Clear();
    Py_RETURN_NONE;
}
PyObject* answer(rk_status s) { return PyLong_FromLong((long)s); }

bool addresses(PyObject* const* a, int n, void** out)
{
    for (int i = 0; i < n; ++i)
        if (!address(a[i], out + i)) return false;
    return true;
}

// (ctx, layout, q, k_packed, v_cache, R_r, delta_mu, scale, out, workspace, stream, workspace_bytes)
PyObject* py_decode(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    void *ctx, *p[5];
    rk_layout L;
    Tail t;
    if (n != 12 || !fn_decode || !address(a[0], &ctx) || !layout(a[1], &L) || !addresses(a + 2, 5, p) || !tail(a + 7, &t)) return other_path();
    rk_status s;
    Py_BEGIN_ALLOW_THREADS
    s = fn_decode((rk_ctx*)ctx, &L, p[0], p[1], p[2], (const float*)p[3], (const float*)p[4], t.scale, t.out, t.ws, t.bytes, t.stream);
    Py_END_ALLOW_THREADS
    return answer(s);
}
// (ctx, layout, k_new, v_new, q, R_r, delta_mu, k_packed, v_cache, seq_len, scale, out, workspace, stream, workspace_bytes)
PyObject* py_append_decode(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    void *ctx, *p[8];
    rk_layout L;
    Tail t;
    if (n != 15 || !fn_append_decode || !address(a[0], &ctx) || !layout(a[1], &L) || !addresses(a + 2, 8, p) || !tail(a + 10, &t))
        return other_path();
    rk_status s;
    Py_BEGIN_ALLOW_THREADS
    s = fn_append_decode((rk_ctx*)ctx, &L, p[0], p[1], p[2], (const float*)p[3], (const float*)p[4], p[5], p[6], (int32_t*)p[7], t.scale,
                         t.out, t.ws, t.bytes, t.stream);
    Py_END_ALLOW_THREADS
    return answer(s);
}
// (ctx, layout, q, k_packed, v_cache, R_r, delta_mu, text, scale, out, workspace, stream, workspace_bytes)
PyObject* py_dual(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    void *ctx, *p[5];
    rk_layout L;
    rk_text T;
    Tail t;
    if (n != 13 || !fn_dual || !address(a[0], &ctx) || !layout(a[1], &L) || !addresses(a + 2, 5, p) || !text(a[7], &T) || !tail(a + 8, &t))
        return other_path();
    rk_status s;
    Py_BEGIN_ALLOW_THREADS
    s = fn_dual((rk_ctx*)ctx, &L, p[0], p[1], p[2], (const float*)p[3], (const float*)p[4], &T, t.scale, t.out, t.ws, t.bytes, t.stream);
    Py_END_ALLOW_THREADS
    return answer(s);
}
// (ctx, layout, k_new, v_new, q, k_packed, v_cache, R_r, delta_mu, text, scale, out, workspace, stream, workspace_bytes)
PyObject* py_append_dual(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    void *ctx, *p[7];
    rk_layout L;
    rk_text T;
    Tail t;
    if (n != 15 || !fn_append_dual || !address(a[0], &ctx) || !layout(a[1], &L) || !addresses(a + 2, 7, p) || !text(a[9], &T) ||
        !tail(a + 10, &t))
        return other_path();
    rk_status s;
    Py_BEGIN_ALLOW_THREADS
    s = fn_append_dual((rk_ctx*)ctx, &L, p[0], p[1], p[2], p[3], p[4], (const float*)p[5], (const float*)p[6], &T, t.scale, t.out, t.ws,
                       t.bytes, t.stream);
    Py_END_ALLOW_THREADS
    return answer(s);
}

// bind(Layout, Text, addresses of the four entry points)
PyObject* py_bind(PyObject*, PyObject* args)
{
    PyObject *lt, *tt;
    unsigned long long f[4];
    if (!PyArg_ParseTuple(args, "O!O!KKKK", &PyType_Type, &lt, &PyType_Type, &tt, f, f + 1, f + 2, f + 3)) return nullptr;
    Py_INCREF(lt);
    Py_INCREF(tt);
    Py_XDECREF((PyObject*)layout_type);
    Py_XDECREF((PyObject*)text_type);
    layout_type = (PyTypeObject*)lt;
    text_type = (PyTypeObject*)tt;
    fn_decode = (decode_fn)(uintptr_t)f[0];
    fn_append_decode = (append_decode_fn)(uintptr_t)f[1];
    fn_dual = (dual_fn)(uintptr_t)f[2];
    fn_append_dual = (append_dual_fn)(uintptr_t)f[3];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", py_bind, METH_VARARGS, "bind(Layout, Text, four entry point addresses)"},
    {"decode", (PyCFunction)(void (*)(void))py_decode, METH_FASTCALL, "rk_decode_attn; its status, or None for arguments not taken here"},
    {"append_decode", (PyCFunction)(void (*)(void))py_append_decode, METH_FASTCALL, "rk_append_decode_attn, likewise"},
    {"dual", (PyCFunction)(void (*)(void))py_dual, METH_FASTCALL, "rk_decode_attn_dual, likewise"},
    {"append_dual", (PyCFunction)(void (*)(void))py_append_dual, METH_FASTCALL, "rk_append_text_decode_attn_dual, likewise"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_rkbind", "Argument marshalling of the per-token calls", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__rkbind(void)
{
    struct { PyObject** at; const char* text; } names[] = {
        {&s_batch, "batch"}, {&s_nq, "n_q_heads"}, {&s_nkv, "n_kv_heads"}, {&s_hd, "head_dim"}, {&s_keep, "keep"}, {&s_dtype, "dtype"},
        {&s_cap, "capacity"}, {&s_max_seq, "max_seq_len"}, {&s_seq, "seq_len"}, {&s_data_ptr, "data_ptr"}, {&s_numel, "numel"},
        {&s_esize, "element_size"}, {&s_cuda_stream, "cuda_stream"}, {&s_k, "k"}, {&s_v, "v"}, {&s_max_len, "max_len"}, {&s_len, "len"},
        {&s_strides, "strides"}, {&s_stride, "stride"}, {&s_shape, "shape"}};
    for (auto& x : names)
        if (!(*x.at = PyUnicode_InternFromString(x.text))) return nullptr;
    return PyModule_Create(&module);
}
