// The binding's calls with every argument of its usual kind (torch tensors, int32 numpy arrays, a KVCache of plain numbers): the
// ampd_kv_cache and ampd_batch structures are filled and the entry point is called without an interpreted step per field.  call()
// returns the status, or None, before anything is called, when an argument is of another kind: the binding then takes its general path.
// A C++ exception out of an entry point (host memory gone in the planner, say) becomes a Python one, with the interpreter's lock held
// again: work may be enqueued by then, so the call is never made a second time.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cfloat>
#include <climits>
#include <cmath>
#include <cstdlib>
#include <exception>
#include <new>

#include <torch/csrc/autograd/python_variable.h>

#include "ampd.h"

namespace {

PyObject *s_num_q_heads, *s_num_kv_heads, *s_head_dim, *s_page_size, *s_kv_dtype, *s_k_pool, *s_v_pool, *s_k_scale, *s_v_scale, *s_softmax_scale;
// torch's functions: current device; raw stream of a device; whether this process was forked from one that used the GPU (or null)
PyObject *g_device = nullptr, *g_raw_stream = nullptr, *g_bad_fork = nullptr;

struct Ref {                                             // an owned reference
    PyObject* o;
    explicit Ref(PyObject* p) : o(p) {}
    ~Ref() { Py_XDECREF(o); }
    Ref(const Ref&) = delete;
    Ref& operator=(const Ref&) = delete;
};

struct Lengths {                                         // a one-dimensional contiguous int32 array
    Py_buffer b;
    bool held = false;
    bool take(PyObject* o) {
        if (PyObject_GetBuffer(o, &b, PyBUF_ND | PyBUF_FORMAT) != 0) {
            PyErr_Clear();
            return false;
        }
        held = true;
        return b.ndim == 1 && b.itemsize == 4 && b.format && b.format[0] == 'i' && b.format[1] == 0 && b.shape[0] <= INT_MAX;
    }
    ~Lengths() {
        if (held) PyBuffer_Release(&b);
    }
};

bool int_attr(PyObject* o, PyObject* name, int32_t* out) {
    Ref v(PyObject_GetAttr(o, name));
    if (!v.o || !PyLong_CheckExact(v.o)) return false;
    int over = 0;
    const long x = PyLong_AsLongAndOverflow(v.o, &over);
    if (over || x < INT_MIN || x > INT_MAX) return false;
    *out = (int32_t)x;
    return true;
}

bool tensor(PyObject* o, const at::Tensor** t) {
    if (!THPVariable_CheckExact(o)) return false;
    *t = &THPVariable_Unpack(o);
    return (*t)->defined();
}
bool address(PyObject* o, void** p) {
    const at::Tensor* t;
    if (!tensor(o, &t)) return false;
    *p = t->data_ptr();
    return true;
}
bool address_attr(PyObject* o, PyObject* name, void** p, bool may_be_none, int64_t* first_dim = nullptr) {
    Ref v(PyObject_GetAttr(o, name));
    if (!v.o) return false;
    if (may_be_none && v.o == Py_None) {
        *p = nullptr;
        return true;
    }
    if (!address(v.o, p)) return false;
    if (first_dim) {
        const at::Tensor& t = THPVariable_Unpack(v.o);
        if (t.dim() < 1) return false;
        *first_dim = t.size(0);
    }
    return true;
}

bool current_stream(void** stream) {
    if (g_bad_fork) {                                    // torch refuses to look for the stream there: so does the general path
        Ref bad(PyObject_CallNoArgs(g_bad_fork));
        if (!bad.o || bad.o != Py_False) return false;
    }
    Ref dev(PyObject_CallNoArgs(g_device));
    if (!dev.o) return false;
    Ref raw(PyObject_CallOneArg(g_raw_stream, dev.o));
    if (!raw.o) return false;
    *stream = PyLong_AsVoidPtr(raw.o);
    return !PyErr_Occurred();
}

typedef ampd_status (*AttnFn)(const ampd_kv_cache*, const ampd_batch*, const void*, const void*, const void*, void*, void*, size_t, void*,
                              const ampd_plan_options*);
typedef ampd_status (*AppendFn)(const ampd_kv_cache*, const ampd_batch*, const void*, const void*, void*);
typedef ampd_status (*MoveFn)(const ampd_kv_cache*, const ampd_batch*, int32_t, int32_t, const void*, const void*, void*);

struct Unlocked {                                        // the interpreter's lock is given up while this lives
    PyThreadState* state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

struct Call {                                            // the arguments of an entry point
    void* fn;
    Py_ssize_t n;
    ampd_kv_cache c = {};
    ampd_batch b = {};
    Lengths ctx, incr;                                   // (b points into them)
    int32_t heads[2] = {0, 0};
    void* p[5];
    size_t ws_bytes = 0;
    void* stream;
};

// args: the entry point's address, cache, ctx_len, incr_len, block_table, rest...; rest: q, k_new, v_new, out, workspace (attention);
// k, v (append); head_begin, head_count, k, v (pack, unpack).  Runs on torch's current stream.  False: not of the usual kind.
bool marshal(PyObject* const* a, Py_ssize_t n, Call& x) {
    if (n != 7 && n != 9 && n != 10) return false;
    if (!g_device || !PyLong_CheckExact(a[0])) return false;
    x.n = n;
    x.fn = PyLong_AsVoidPtr(a[0]);
    if (!x.fn) return false;
    ampd_kv_cache& c = x.c;
    PyObject* cache = a[1];
    if (!int_attr(cache, s_num_q_heads, &c.num_q_heads) || !int_attr(cache, s_num_kv_heads, &c.num_kv_heads) ||
        !int_attr(cache, s_head_dim, &c.head_dim) || !int_attr(cache, s_page_size, &c.page_size) || !int_attr(cache, s_kv_dtype, &c.kv_dtype))
        return false;
    void *k, *v, *ks, *vs;
    if (!address_attr(cache, s_k_pool, &k, false, &c.num_pages) || !address_attr(cache, s_v_pool, &v, false) ||
        !address_attr(cache, s_k_scale, &ks, true) || !address_attr(cache, s_v_scale, &vs, true))
        return false;
    c.k_pool = k;
    c.v_pool = v;
    c.k_scale = static_cast<float*>(ks);
    c.v_scale = static_cast<float*>(vs);
    {
        Ref f(PyObject_GetAttr(cache, s_softmax_scale));
        if (!f.o || !PyFloat_CheckExact(f.o)) return false;
        const double scale = PyFloat_AS_DOUBLE(f.o);
        if (!(std::fabs(scale) <= FLT_MAX)) return false;
        c.softmax_scale = (float)scale;
    }
    if (!x.ctx.take(a[2]) || !x.incr.take(a[3]) || x.ctx.b.shape[0] != x.incr.b.shape[0]) return false;
    const at::Tensor* bt;
    if (!tensor(a[4], &bt) || bt->dim() != 2 || !bt->is_cuda() || bt->size(1) > INT_MAX) return false;
    x.b.num_reqs = (int32_t)x.ctx.b.shape[0];
    x.b.max_pages_per_req = (int32_t)bt->size(1);
    x.b.h_ctx_len = static_cast<const int32_t*>(x.ctx.b.buf);
    x.b.h_incr_len = static_cast<const int32_t*>(x.incr.b.buf);
    x.b.d_block_table = static_cast<const int32_t*>(bt->data_ptr());
    for (int i = 0; n == 9 && i < 2; ++i) {
        if (!PyLong_CheckExact(a[5 + i])) return false;
        int over = 0;
        const long h = PyLong_AsLongAndOverflow(a[5 + i], &over);
        if (over || h < INT_MIN || h > INT_MAX) return false;
        x.heads[i] = (int32_t)h;
    }
    const int first = n == 9 ? 7 : 5;
    for (int i = first; i < n; ++i)
        if (!address(a[i], &x.p[i - first])) return false;
    if (n == 10) x.ws_bytes = THPVariable_Unpack(a[9]).nbytes();
    return current_stream(&x.stream);
}

ampd_status enter(const Call& x) {
    Unlocked u;
    if (x.n == 10)
        return reinterpret_cast<AttnFn>(x.fn)(&x.c, &x.b, x.p[0], x.p[1], x.p[2], x.p[3], x.p[4], x.ws_bytes, x.stream, nullptr);
    if (x.n == 9) return reinterpret_cast<MoveFn>(x.fn)(&x.c, &x.b, x.heads[0], x.heads[1], x.p[0], x.p[1], x.stream);
    return reinterpret_cast<AppendFn>(x.fn)(&x.c, &x.b, x.p[0], x.p[1], x.stream);
}

PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Call x;
    bool usual = false;
    try {
        usual = marshal(args, n, x);
    } catch (...) {                                      // a tensor without storage, say: the general path reports it
    }
    if (!usual) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    try {
        return PyLong_FromLong(enter(x));
    } catch (const std::bad_alloc&) {
        return PyErr_NoMemory();
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// streams(current device, raw stream of a device[, forked from a process that used the GPU]): torch's functions
PyObject* streams(PyObject*, PyObject* const* args, Py_ssize_t n) {
    bool ok = n == 2 || n == 3;
    for (Py_ssize_t i = 0; ok && i < n; ++i) ok = PyCallable_Check(args[i]);
    if (!ok) {
        PyErr_SetString(PyExc_TypeError, "two or three functions");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < n; ++i) Py_INCREF(args[i]);
    g_device = args[0];
    g_raw_stream = args[1];
    g_bad_fork = n == 3 ? args[2] : nullptr;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(call)), METH_FASTCALL, nullptr},
                         {"streams", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(streams)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// The module is built for one Python and one torch: a file left over from before either changed is no module (its name carries no
// version), instead of one that reads objects of another layout.  The binding compares torch_version.
PyMODINIT_FUNC PyInit__fastcall() {
    const char* v = Py_GetVersion();
    char* end = nullptr;
    const long major = std::strtol(v, &end, 10), minor = *end == '.' ? std::strtol(end + 1, nullptr, 10) : -1;
    if (major != PY_MAJOR_VERSION || minor != PY_MINOR_VERSION) {
        PyErr_Format(PyExc_ImportError, "built for Python %d.%d", PY_MAJOR_VERSION, PY_MINOR_VERSION);
        return nullptr;
    }
    struct { PyObject** at; const char* name; } names[] = {
        {&s_num_q_heads, "num_q_heads"}, {&s_num_kv_heads, "num_kv_heads"}, {&s_head_dim, "head_dim"}, {&s_page_size, "page_size"},
        {&s_kv_dtype, "kv_dtype"}, {&s_k_pool, "k_pool"}, {&s_v_pool, "v_pool"}, {&s_k_scale, "k_scale"}, {&s_v_scale, "v_scale"},
        {&s_softmax_scale, "softmax_scale"}};
    for (auto& n : names)
        if (!(*n.at = PyUnicode_InternFromString(n.name))) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", AMPD_TORCH_VERSION) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
