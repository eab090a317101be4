// Argument marshalling of paper_2011_10170_amd/binding.py for the entry points that a training or serving loop calls: what ctypes and Python code
// took 2 us for per call (4 us per ten tensors of a list) takes 0.3 here. The functions return the call's status; the binding raises on
// failure. They hold no state but the entry points' addresses, which the binding takes from the library that it loads.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <string.h>

#include <new>
#include <tuple>
#include <utility>
#include <vector>

#include "pc.h"

namespace {

PyObject *g_data_ptr;      // the interned name of the method that tensors have
PyObject *g_desc, *g_address;      // from the binding: the descriptor's type, and what makes an address of a handle that is no integer

// A Python integer, or what int() makes of the object; *ok turns false with an exception set.
long long as_int(PyObject *o, bool *ok)
{
    PyObject *n = PyLong_CheckExact(o) ? o : PyNumber_Long(o);
    if (!n) { *ok = false; return 0; }
    int over = 0;
    const long long v = PyLong_AsLongLongAndOverflow(n, &over);
    if (over > 0) {          // addresses use all 64 bits
        const unsigned long long u = PyLong_AsUnsignedLongLong(n);
        if (PyErr_Occurred()) *ok = false;
        if (n != o) Py_DECREF(n);
        return (long long)u;
    }
    if (over < 0) PyErr_SetString(PyExc_OverflowError, "integer out of range");
    if (over < 0 || (v == -1 && PyErr_Occurred())) *ok = false;
    if (n != o) Py_DECREF(n);
    return v;
}

// None, a tensor (anything with data_ptr()) or an address
void *as_ptr(PyObject *o, bool *ok)
{
    if (o == Py_None) return nullptr;
    if (PyLong_CheckExact(o)) return (void *)as_int(o, ok);
    PyObject *m = PyObject_CallMethodNoArgs(o, g_data_ptr);
    if (!m) {
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) { *ok = false; return nullptr; }
        PyErr_Clear();
        return (void *)as_int(o, ok);
    }
    void *p = (void *)as_int(m, ok);
    Py_DECREF(m);
    return p;
}

// A context or a pack: None, an integer or what ctypes takes for a void pointer. Not a tensor: the library reads a handle on the host.
void *as_handle(PyObject *o, bool *ok)
{
    if (o == Py_None) return nullptr;
    if (PyLong_Check(o)) return (void *)as_int(o, ok);
    PyObject *m = PyObject_CallOneArg(g_address, o);
    if (!m) { *ok = false; return nullptr; }
    void *p = m == Py_None ? nullptr : (void *)as_int(m, ok);
    Py_DECREF(m);
    return p;
}

// A pack of a list: what int() takes
void *as_listed_handle(PyObject *o, bool *ok)
{
    if (!PyLong_Check(o) && PyObject_HasAttr(o, g_data_ptr)) {
        PyErr_SetString(PyExc_TypeError, "a tensor is no pack");
        *ok = false;
        return nullptr;
    }
    return (void *)as_int(o, ok);
}

// The kinds of arguments. Each is made from the caller's object; count() is the length of a list that has one entry per layer, EXACT whether
// it may be no longer than the call's number of layers (none may be shorter).
struct Scalar {
    enum { EXACT = 0 };
    Py_ssize_t count() const { return -1; }
};
struct Ptr : Scalar {
    void *v;
    bool set(PyObject *const *a) { bool ok = true; v = as_ptr(a[0], &ok); return ok; }
    template <class T> T *get() const { return (T *)v; }
};
struct Handle : Scalar {
    void *v;
    bool set(PyObject *const *a) { bool ok = true; v = as_handle(a[0], &ok); return ok; }
    template <class T> T *get() const { return (T *)v; }
};
struct Int : Scalar {
    long long v;
    bool set(PyObject *const *a) { bool ok = true; v = as_int(a[0], &ok); return ok; }
};
struct Real : Scalar {
    double v;
    bool set(PyObject *const *a)
    {
        PyObject *f = PyNumber_Float(a[0]);
        if (!f) return false;
        v = PyFloat_AS_DOUBLE(f);
        Py_DECREF(f);
        return true;
    }
};
struct Desc : Scalar {       // a ctypes structure
    pc_conv_desc v;
    bool set(PyObject *const *a)
    {
        Py_buffer b;
        if (!PyObject_TypeCheck(a[0], (PyTypeObject *)g_desc)) {
            PyErr_Format(PyExc_TypeError, "a pc_conv_desc is wanted, not %.100s", Py_TYPE(a[0])->tp_name);
            return false;
        }
        if (PyObject_GetBuffer(a[0], &b, PyBUF_SIMPLE) != 0) return false;
        const bool ok = b.len >= (Py_ssize_t)sizeof(v);
        if (ok) memcpy(&v, b.buf, sizeof(v));
        else PyErr_SetString(PyExc_TypeError, "not a pc_conv_desc");
        PyBuffer_Release(&b);
        return ok;
    }
};
template <class E, class F> bool fill(PyObject *o, std::vector<E> &v, F one)
{
    PyObject *s = PySequence_Fast(o, "a list is wanted");
    if (!s) return false;
    v.reserve((size_t)PySequence_Fast_GET_SIZE(s));
    bool ok = true;
    for (Py_ssize_t i = 0; i < PySequence_Fast_GET_SIZE(s) && ok; ++i) {      // (an entry's code may change the caller's list)
        PyObject *o = PySequence_Fast_GET_ITEM(s, i);
        Py_INCREF(o);
        v.push_back(one(o, &ok));
        Py_DECREF(o);
    }
    Py_DECREF(s);
    return ok;
}
struct Ptrs {                // a list of tensors or of handles; None stands for no list
    enum { EXACT = 0 };
    Py_ssize_t count() const { return none ? -1 : (Py_ssize_t)v.size(); }
    std::vector<void *> v;
    bool none = false;
    bool set(PyObject *const *a)
    {
        none = a[0] == Py_None;
        return none || fill(a[0], v, as_ptr);
    }
    template <class T> T *get() { return none ? nullptr : (T *)v.data(); }
};
struct Handles : Ptrs {
    enum { EXACT = 1 };
    bool set(PyObject *const *a) { return fill(a[0], v, as_listed_handle); }
};
template <class T, int E = 0> struct Ints {
    enum { EXACT = E };
    Py_ssize_t count() const { return (Py_ssize_t)v.size(); }
    std::vector<T> v;
    bool set(PyObject *const *a) { return fill(a[0], v, [](PyObject *o, bool *ok) { return (T)as_int(o, ok); }); }
};
struct Pool : Ints<uint16_t> {      // the pattern pool: of no layer; its length follows from the list
    enum { EXACT = 0 };
    Py_ssize_t count() const { return -1; }
    int32_t size() const { return (int32_t)v.size(); }
};
struct Descs {
    enum { EXACT = 0 };
    Py_ssize_t count() const { return (Py_ssize_t)v.size(); }
    std::vector<pc_conv_desc> v;
    bool set(PyObject *const *a)
    {
        return fill(a[0], v, [](PyObject *o, bool *ok) {
            Desc d = {};
            PyObject *made = PyTuple_Check(o) ? PyObject_CallObject(g_desc, o) : nullptr;      // (as in an array of ctypes)
            if (PyTuple_Check(o) && !made) *ok = false;
            else *ok = d.set(made ? &made : &o);
            Py_XDECREF(made);
            return d.v;
        });
    }
};

// The entry points by the place of their address.
enum Entry {
    E_fwd, E_fwd_relu, E_bwd_data, E_bwd_data_relu, E_bwd_weight, E_bwd_weight_batch, E_scatter_dense, E_unpack_dense, E_act_pool_fwd, E_act_pool_bwd,
    E_pattern_select, E_pattern_select_batch, E_pack, E_pack_batch, E_update_values, E_update_values_batch, E_finalize_count, E_finalize_pick,
    E_finalize_count_batch, E_finalize_pick_batch, E_dppg_accumulate_batch, E_group_lasso_grad_batch, E_COUNT
};
const char *const kNames[E_COUNT] = {
    "pc_conv_fwd", "pc_conv_fwd_relu", "pc_conv_bwd_data", "pc_conv_bwd_data_relu", "pc_conv_bwd_weight", "pc_conv_bwd_weight_batch", "pc_scatter_dense",
    "pc_unpack_dense", "pc_act_pool_fwd", "pc_act_pool_bwd", "pc_pattern_select", "pc_pattern_select_batch", "pc_pack", "pc_pack_batch", "pc_update_values",
    "pc_update_values_batch", "pc_finalize_count", "pc_finalize_pick", "pc_finalize_count_batch", "pc_finalize_pick_batch", "pc_dppg_accumulate_batch",
    "pc_group_lasso_grad_batch"};
void *g_entry[E_COUNT];

template <class Tuple, size_t... I> bool set_all(Tuple &t, PyObject *const *a, std::index_sequence<I...>) { return (std::get<I>(t).set(a + I) && ...); }

// Every list has an entry for each of the layers, of which argument MAIN tells the number.
template <int MAIN, class... K> bool lengths(const std::tuple<K...> &t)
{
    if constexpr (MAIN >= 0) {
        const Py_ssize_t n = std::get<MAIN>(t).count();
        const bool ok = n >= 0 && std::apply([n](const K &...k) { return ((k.count() < 0 || k.count() == n || (k.count() > n && !K::EXACT)) && ...); }, t);
        if (!ok) PyErr_SetString(PyExc_ValueError, "lists of different lengths");
        return ok;
    }
    return true;
}

// Converts the arguments and calls `go` with them, without the interpreter's lock.
template <int MAIN, class... K, class Go> PyObject *call(int entry, PyObject *const *a, Py_ssize_t n, Go go)
{
    if (n != (Py_ssize_t)sizeof...(K)) {
        PyErr_Format(PyExc_TypeError, "%s: %zd arguments, %zd are wanted", kNames[entry], n, (Py_ssize_t)sizeof...(K));
        return nullptr;
    }
    if (!g_entry[entry]) {
        PyErr_Format(PyExc_RuntimeError, "%s: the library is not loaded", kNames[entry]);
        return nullptr;
    }
    try {
        std::tuple<K...> t;
        if (!set_all(t, a, std::index_sequence_for<K...>()) || !lengths<MAIN>(t)) return nullptr;
        int status;
        Py_BEGIN_ALLOW_THREADS              // (nothing is thrown from here: the lists are made, the library's entry points return errors)
        status = std::apply(go, t);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(status);
    } catch (const std::bad_alloc &) {      // (of the lists above)
        return PyErr_NoMemory();
    }
}

#define ENTRY(name) PyObject *name(PyObject *, PyObject *const *a, Py_ssize_t n)
#define FN(name) ((decltype(&pc_##name))g_entry[E_at])
#define P(x, T) (x).get<T>()

ENTRY(conv_fwd) { constexpr int E_at = E_fwd; return call<-1, Handle, Desc, Handle, Ptr, Ptr>(E_at, a, n, [](Handle &c, Desc &d, Handle &k, Ptr &x, Ptr &y) {
    return (int)FN(conv_fwd)(P(c, pc_ctx), &d.v, P(k, const pc_packed), P(x, const void), P(y, void)); }); }
ENTRY(conv_fwd_relu) { constexpr int E_at = E_fwd_relu; return call<-1, Handle, Desc, Handle, Ptr, Ptr>(E_at, a, n, [](Handle &c, Desc &d, Handle &k, Ptr &x, Ptr &y) {
    return (int)FN(conv_fwd_relu)(P(c, pc_ctx), &d.v, P(k, const pc_packed), P(x, const void), P(y, void)); }); }
ENTRY(conv_bwd_data) { constexpr int E_at = E_bwd_data; return call<-1, Handle, Desc, Handle, Ptr, Ptr>(E_at, a, n, [](Handle &c, Desc &d, Handle &k, Ptr &x, Ptr &y) {
    return (int)FN(conv_bwd_data)(P(c, pc_ctx), &d.v, P(k, const pc_packed), P(x, const void), P(y, void)); }); }
ENTRY(conv_bwd_data_relu) { constexpr int E_at = E_bwd_data_relu; return call<-1, Handle, Desc, Handle, Ptr, Ptr, Ptr>(E_at, a, n, [](Handle &c, Desc &d, Handle &k, Ptr &x, Ptr &m, Ptr &y) {
    return (int)FN(conv_bwd_data_relu)(P(c, pc_ctx), &d.v, P(k, const pc_packed), P(x, const void), P(m, const void), P(y, void)); }); }
ENTRY(conv_bwd_weight) { constexpr int E_at = E_bwd_weight; return call<-1, Handle, Desc, Handle, Ptr, Ptr, Ptr>(E_at, a, n, [](Handle &c, Desc &d, Handle &k, Ptr &x, Ptr &g, Ptr &w) {
    return (int)FN(conv_bwd_weight)(P(c, pc_ctx), &d.v, P(k, const pc_packed), P(x, const void), P(g, const void), P(w, float)); }); }
ENTRY(conv_bwd_weight_batch) { constexpr int E_at = E_bwd_weight_batch; return call<1, Handle, Descs, Handles, Ptrs, Ptrs, Ptrs>(E_at, a, n,
    [](Handle &c, Descs &d, Handles &k, Ptrs &x, Ptrs &g, Ptrs &w) {
    return (int)FN(conv_bwd_weight_batch)(P(c, pc_ctx), (int32_t)d.v.size(), d.v.data(), P(k, const pc_packed *), P(x, const void *), P(g, const void *), P(w, float *)); }); }
ENTRY(scatter_dense) { constexpr int E_at = E_scatter_dense; return call<-1, Handle, Handle, Ptr, Ptr>(E_at, a, n, [](Handle &c, Handle &k, Ptr &w, Ptr &d) {
    return (int)FN(scatter_dense)(P(c, pc_ctx), P(k, const pc_packed), P(w, const float), P(d, float)); }); }
ENTRY(unpack_dense) { constexpr int E_at = E_unpack_dense; return call<-1, Handle, Handle, Ptr>(E_at, a, n, [](Handle &c, Handle &k, Ptr &d) {
    return (int)FN(unpack_dense)(P(c, pc_ctx), P(k, const pc_packed), P(d, float)); }); }
ENTRY(act_pool_fwd) { constexpr int E_at = E_act_pool_fwd; return call<-1, Handle, Ptr, Int, Int, Int, Int, Int, Int, Ptr, Ptr>(E_at, a, n,
    [](Handle &c, Ptr &z, Int &N, Int &H, Int &W, Int &C, Int &t, Int &q, Ptr &o, Ptr &s) {
    return (int)FN(act_pool_fwd)(P(c, pc_ctx), P(z, const void), (int32_t)N.v, (int32_t)H.v, (int32_t)W.v, (int32_t)C.v, (pc_dtype)t.v, (int32_t)q.v, P(o, void), P(s, uint8_t)); }); }
ENTRY(act_pool_bwd) { constexpr int E_at = E_act_pool_bwd; return call<-1, Handle, Ptr, Ptr, Int, Int, Int, Int, Int, Int, Ptr>(E_at, a, n,
    [](Handle &c, Ptr &g, Ptr &s, Int &N, Int &H, Int &W, Int &C, Int &t, Int &q, Ptr &z) {
    return (int)FN(act_pool_bwd)(P(c, pc_ctx), P(g, const void), P(s, const uint8_t), (int32_t)N.v, (int32_t)H.v, (int32_t)W.v, (int32_t)C.v, (pc_dtype)t.v, (int32_t)q.v, P(z, void)); }); }
ENTRY(pattern_select) { constexpr int E_at = E_pattern_select; return call<-1, Handle, Ptr, Ptr, Int, Int, Pool, Int, Int, Int, Ptr, Ptr>(E_at, a, n,
    [](Handle &c, Ptr &w, Ptr &g, Int &F, Int &C, Pool &m, Int &km, Int &k, Int &sm, Ptr &p, Ptr &q) {
    return (int)FN(pattern_select)(P(c, pc_ctx), P(w, const float), P(g, const float), (int32_t)F.v, (int32_t)C.v, m.v.data(), m.size(), (pc_keep_mode)km.v, k.v,
                                   (pc_score_mode)sm.v, P(p, uint8_t), P(q, uint8_t)); }); }
ENTRY(pattern_select_batch) { constexpr int E_at = E_pattern_select_batch;
    return call<1, Handle, Ptrs, Ptrs, Ints<int32_t, 1>, Ints<int32_t, 1>, Pool, Int, Ints<int64_t, 1>, Int, Ptrs, Ptrs>(E_at, a, n,
    [](Handle &c, Ptrs &w, Ptrs &g, Ints<int32_t, 1> &F, Ints<int32_t, 1> &C, Pool &m, Int &km, Ints<int64_t, 1> &k, Int &sm, Ptrs &p, Ptrs &q) {
    return (int)FN(pattern_select_batch)(P(c, pc_ctx), (int32_t)w.v.size(), P(w, const float *), P(g, const float *), F.v.data(), C.v.data(), m.v.data(), m.size(),
                                         (pc_keep_mode)km.v, k.v.data(), (pc_score_mode)sm.v, P(p, uint8_t *), P(q, uint8_t *)); }); }
// (the handle to be re-packed)
ENTRY(pack) { constexpr int E_at = E_pack; return call<-1, Handle, Ptr, Ptr, Ptr, Int, Int, Pool, Int, Handle>(E_at, a, n,
    [](Handle &c, Ptr &w, Ptr &p, Ptr &q, Int &F, Int &C, Pool &m, Int &t, Handle &k) {
    pc_packed *handle = P(k, pc_packed);
    return (int)FN(pack)(P(c, pc_ctx), P(w, const float), P(p, const uint8_t), P(q, const uint8_t), (int32_t)F.v, (int32_t)C.v, m.v.data(), m.size(), (pc_dtype)t.v, &handle); }); }
ENTRY(pack_batch) { constexpr int E_at = E_pack_batch; return call<1, Handle, Ptrs, Ptrs, Ptrs, Pool, Handles>(E_at, a, n,
    [](Handle &c, Ptrs &w, Ptrs &p, Ptrs &q, Pool &m, Handles &k) {
    return (int)FN(pack_batch)(P(c, pc_ctx), (int32_t)w.v.size(), P(w, const float *), P(p, const uint8_t *), P(q, const uint8_t *), m.v.data(), m.size(), P(k, pc_packed *)); }); }
ENTRY(update_values) { constexpr int E_at = E_update_values; return call<-1, Handle, Handle, Ptr>(E_at, a, n, [](Handle &c, Handle &k, Ptr &w) {
    return (int)FN(update_values)(P(c, pc_ctx), P(k, pc_packed), P(w, const float)); }); }
ENTRY(update_values_batch) { constexpr int E_at = E_update_values_batch; return call<1, Handle, Handles, Ptrs>(E_at, a, n, [](Handle &c, Handles &k, Ptrs &w) {
    return (int)FN(update_values_batch)(P(c, pc_ctx), (int32_t)k.v.size(), P(k, pc_packed *), P(w, const float *)); }); }
ENTRY(finalize_count) { constexpr int E_at = E_finalize_count; return call<-1, Handle, Ptr, Int, Int, Int, Ptr>(E_at, a, n, [](Handle &c, Ptr &p, Int &F, Int &C, Int &q, Ptr &o) {
    return (int)FN(finalize_count)(P(c, pc_ctx), P(p, const uint8_t), (int32_t)F.v, (int32_t)C.v, (int32_t)q.v, P(o, uint32_t)); }); }
ENTRY(finalize_pick) { constexpr int E_at = E_finalize_pick; return call<-1, Handle, Ptr, Int, Int, Int, Ptr>(E_at, a, n, [](Handle &c, Ptr &o, Int &F, Int &C, Int &q, Ptr &p) {
    return (int)FN(finalize_pick)(P(c, pc_ctx), P(o, const uint32_t), (int32_t)F.v, (int32_t)C.v, (int32_t)q.v, P(p, uint8_t)); }); }
ENTRY(finalize_count_batch) { constexpr int E_at = E_finalize_count_batch; return call<1, Handle, Ptrs, Ints<int32_t>, Ints<int32_t>, Int, Ptrs>(E_at, a, n,
    [](Handle &c, Ptrs &p, Ints<int32_t> &F, Ints<int32_t> &C, Int &q, Ptrs &o) {
    return (int)FN(finalize_count_batch)(P(c, pc_ctx), (int32_t)p.v.size(), P(p, const uint8_t *), F.v.data(), C.v.data(), (int32_t)q.v, P(o, uint32_t *)); }); }
ENTRY(finalize_pick_batch) { constexpr int E_at = E_finalize_pick_batch; return call<5, Handle, Ptrs, Ints<int32_t>, Ints<int32_t>, Int, Ptrs>(E_at, a, n,
    [](Handle &c, Ptrs &o, Ints<int32_t> &F, Ints<int32_t> &C, Int &q, Ptrs &p) {
    return (int)FN(finalize_pick_batch)(P(c, pc_ctx), (int32_t)p.v.size(), P(o, const uint32_t *), F.v.data(), C.v.data(), (int32_t)q.v, P(p, uint8_t *)); }); }
ENTRY(dppg_accumulate_batch) { constexpr int E_at = E_dppg_accumulate_batch; return call<1, Handle, Ptrs, Ptrs, Ints<int32_t>, Ints<int32_t>, Ptr, Ptrs>(E_at, a, n,
    [](Handle &c, Ptrs &w, Ptrs &g, Ints<int32_t> &F, Ints<int32_t> &C, Ptr &h, Ptrs &m) {
    return (int)FN(dppg_accumulate_batch)(P(c, pc_ctx), (int32_t)w.v.size(), P(w, const float *), P(g, const float *), F.v.data(), C.v.data(), P(h, uint32_t), P(m, uint16_t *)); }); }
ENTRY(group_lasso_grad_batch) { constexpr int E_at = E_group_lasso_grad_batch;
    return call<1, Handle, Ptrs, Ptrs, Ptrs, Ints<int32_t>, Ints<int32_t>, Pool, Real, Real, Ptrs, Ptr>(E_at, a, n,
    [](Handle &c, Ptrs &w, Ptrs &p, Ptrs &q, Ints<int32_t> &F, Ints<int32_t> &C, Pool &m, Real &lp, Real &li, Ptrs &d, Ptr &o) {
    return (int)FN(group_lasso_grad_batch)(P(c, pc_ctx), (int32_t)w.v.size(), P(w, const float *), P(p, const uint8_t *), P(q, const uint8_t *), F.v.data(), C.v.data(), m.v.data(),
                                           m.size(), (float)lp.v, (float)li.v, P(d, float *), P(o, double)); }); }

// bind({name: address}, descriptor type, address of a handle): the entry points to be called from here on
PyObject *bind(PyObject *, PyObject *args)
{
    PyObject *d, *desc, *address;
    if (!PyArg_ParseTuple(args, "O!O!O", &PyDict_Type, &d, &PyType_Type, &desc, &address)) return nullptr;
    Py_INCREF(desc);
    Py_XSETREF(g_desc, desc);
    Py_INCREF(address);
    Py_XSETREF(g_address, address);
    for (int i = 0; i < E_COUNT; ++i) {
        PyObject *o = PyDict_GetItemString(d, kNames[i]);
        if (!o) return PyErr_Format(PyExc_KeyError, "%s", kNames[i]);
        bool ok = true;
        void *p = (void *)as_int(o, &ok);
        if (!ok) return nullptr;
        g_entry[i] = p;
    }
    Py_RETURN_NONE;
}

#define M(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {M(conv_fwd), M(conv_fwd_relu), M(conv_bwd_data), M(conv_bwd_data_relu), M(conv_bwd_weight), M(conv_bwd_weight_batch), M(scatter_dense),
                          M(unpack_dense), M(act_pool_fwd), M(act_pool_bwd), M(pattern_select), M(pattern_select_batch), M(pack), M(pack_batch), M(update_values),
                          M(update_values_batch), M(finalize_count), M(finalize_pick), M(finalize_count_batch), M(finalize_pick_batch), M(dppg_accumulate_batch),
                          M(group_lasso_grad_batch), {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    return g_data_ptr ? PyModule_Create(&kModule) : nullptr;
}
