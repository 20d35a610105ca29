// The marshalling of the calls a serving loop makes, as a CPython module: arguments as the functions of binding.py take
// them, read from the tensors without going through Python attributes, into the C entry points of libagattn.so (whose addresses
// binding.py hands over; nothing is linked).  A call of 9 tensors took 6.3 us of host time through ctypes, of which the launch
// itself is 3.0; this way 3.4 (an append; 36 calls of a small fp32 session 220 -> 181 us).
//
// Only plain arguments are taken here: exact tensor, KVCache, int and float types, tensors on the GPU, contiguous, of the
// right dtype, numbers in range.  For anything else - a missing or strided tensor, a subclass, a foreign int type - the function
// returns None and binding.py takes its ctypes path, which accepts or refuses it.  Nothing is kept from one call for the next.
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "ag.h"

namespace {

struct Entries {
    decltype(&ag_kv_append) kv_append;
    decltype(&ag_attn_prefill) attn_prefill;
    decltype(&ag_attn_resume) attn_resume;
    decltype(&ag_attn_decode) attn_decode;
    decltype(&ag_attn_decode_static) attn_decode_static;
    decltype(&ag_decode_step) decode_step;
    decltype(&ag_attn_merged) attn_merged;
};
Entries entries;
PyObject* cache_type;           // binding.KVCache
PyObject* get_device;           // torch._C._cuda_getDevice
PyObject* get_raw_stream;       // torch._C._cuda_getCurrentRawStream
PyObject *n_k_pool, *n_v_pool, *n_num_pages, *n_page_size, *n_num_kv_heads, *n_head_dim, *n_dtype, *n_cuda_stream;

// Reads arguments; `plain` becomes false at the first that is not for this path, and the rest is not looked at.
struct Reader {
    bool plain = true;

    const at::Tensor* tensor(PyObject* o)
    {
        if (plain && THPVariable_CheckExact(o)) {
            const at::Tensor& t = THPVariable_Unpack(o);
            if (t.defined()) return &t;
        }
        plain = false;
        return nullptr;
    }
    void* device(PyObject* o, const at::Tensor** out = nullptr)
    {
        const at::Tensor* t = tensor(o);
        if (!t) return nullptr;
        if (!t->is_cuda() || !t->is_contiguous()) { plain = false; return nullptr; }
        if (out) *out = t;
        return t->data_ptr();
    }
    const int32_t* ints(PyObject* o, const at::Tensor** out = nullptr)
    {
        const at::Tensor* t = nullptr;
        void* p = device(o, &t);
        if (t && t->scalar_type() != at::kInt) plain = false;
        if (out) *out = t;
        return (const int32_t*)p;
    }
    int32_t size(const at::Tensor* t, int dim)
    {
        if (!plain || t->dim() <= dim || t->size(dim) > INT32_MAX) { plain = false; return 0; }
        return (int32_t)t->size(dim);
    }
    int32_t number(PyObject* o)
    {
        if (!plain || !PyLong_CheckExact(o)) { plain = false; return 0; }
        int over = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &over);
        if (over || v < INT32_MIN || v > INT32_MAX) { plain = false; return 0; }
        return (int32_t)v;
    }
    float real(PyObject* o)
    {
        if (!plain || !PyFloat_CheckExact(o)) { plain = false; return 0.f; }
        return (float)PyFloat_AS_DOUBLE(o);
    }
    void cache(PyObject* o, ag_kv_cache& c)
    {
        if (!plain || (PyObject*)Py_TYPE(o) != cache_type) { plain = false; return; }
        auto get = [&](PyObject* name, auto use) {
            PyObject* v = plain ? PyObject_GetAttr(o, name) : nullptr;
            if (!v) { PyErr_Clear(); plain = false; return; }
            use(v);
            Py_DECREF(v);
        };
        get(n_k_pool, [&](PyObject* v) { if (const at::Tensor* t = tensor(v)) c.k_pool = t->data_ptr(); });
        get(n_v_pool, [&](PyObject* v) { if (const at::Tensor* t = tensor(v)) c.v_pool = t->data_ptr(); });
        get(n_num_pages, [&](PyObject* v) { c.num_pages = number(v); });
        get(n_page_size, [&](PyObject* v) { c.page_size = number(v); });
        get(n_num_kv_heads, [&](PyObject* v) { c.num_kv_heads = number(v); });
        get(n_head_dim, [&](PyObject* v) { c.head_dim = number(v); });
        get(n_dtype, [&](PyObject* v) { c.dtype = number(v); });
    }
    // None: torch's current stream; an int: a raw handle; a torch stream: its handle (a call 6.0 -> 3.1 us)
    void* stream(PyObject* o)
    {
        if (!plain) return nullptr;
        void* s = nullptr;
        if (o != Py_None) {
            PyObject* handle = PyLong_CheckExact(o) ? Py_NewRef(o) : PyObject_GetAttr(o, n_cuda_stream);
            if (handle && PyLong_CheckExact(handle)) s = PyLong_AsVoidPtr(handle);
            else plain = false;
            Py_XDECREF(handle);
            if (PyErr_Occurred()) { PyErr_Clear(); plain = false; }
            return s;
        }
        PyObject* dev = PyObject_CallNoArgs(get_device);
        PyObject* raw = dev ? PyObject_CallOneArg(get_raw_stream, dev) : nullptr;
        if (raw) s = PyLong_AsVoidPtr(raw);
        Py_XDECREF(dev);
        Py_XDECREF(raw);
        if (PyErr_Occurred()) { PyErr_Clear(); plain = false; }
        return s;
    }
};

// The call itself without the interpreter's lock, as ctypes makes it; None if the arguments are not plain.
template <class Read>
PyObject* guarded(Py_ssize_t have, Py_ssize_t want, Read read)
{
    if (have != want) Py_RETURN_NONE;
    try {
        return read();
    } catch (...) {             // a tensor without storage or the like: the other path says what is wrong
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}
template <class Call>
PyObject* finish(const Reader& r, Call call)
{
    if (!r.plain) Py_RETURN_NONE;
    ag_status st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

PyObject* kv_append(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded(n, 9, [&] {
        Reader r;
        ag_kv_cache c;
        const at::Tensor *bt, *lens;
        r.cache(a[0], c);
        const void *k = r.device(a[1]), *v = r.device(a[2]);
        const int32_t *b = r.ints(a[3], &bt), *prefix = r.ints(a[4]), *len = r.ints(a[5], &lens), *cu = r.ints(a[6]);
        const int32_t pages = r.size(bt, 1), batch = r.size(lens, 0), total = r.number(a[7]);
        void* s = r.stream(a[8]);
        return finish(r, [&] { return entries.kv_append(&c, k, v, b, pages, prefix, len, cu, batch, total, s); });
    });
}

PyObject* attn_prefill(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded(n, 11, [&] {
        Reader r;
        ag_kv_cache c;
        const at::Tensor *bt, *lens;
        r.cache(a[0], c);
        void *q = r.device(a[1]), *out = r.device(a[2]);
        const int32_t *b = r.ints(a[3], &bt), *len = r.ints(a[4], &lens), *cu = r.ints(a[5]);
        const int32_t pages = r.size(bt, 1), batch = r.size(lens, 0), total = r.number(a[6]), max_new = r.number(a[7]), hq = r.number(a[8]);
        const float scale = r.real(a[9]);
        void* s = r.stream(a[10]);
        return finish(r, [&] { return entries.attn_prefill(&c, q, out, b, pages, len, cu, batch, total, max_new, hq, scale, s); });
    });
}

// resume prefill, and the merged batch, which takes a workspace as well
template <bool kMerged>
PyObject* attn_resume(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded(n, kMerged ? 14 : 13, [&] {
        Reader r;
        ag_kv_cache c;
        const at::Tensor *bt, *lens, *ws = nullptr;
        r.cache(a[0], c);
        void *q = r.device(a[1]), *out = r.device(a[2]);
        const int32_t *b = r.ints(a[3], &bt), *prefix = r.ints(a[4]), *len = r.ints(a[5], &lens), *cu = r.ints(a[6]);
        const int32_t pages = r.size(bt, 1), batch = r.size(lens, 0), total = r.number(a[7]), max_new = r.number(a[8]),
                      max_ctx = r.number(a[9]), hq = r.number(a[10]);
        const float scale = r.real(a[11]);
        void* w = kMerged ? r.device(a[12], &ws) : nullptr;
        const size_t bytes = ws && r.plain ? (size_t)ws->numel() * ws->element_size() : 0;
        void* s = r.stream(a[n - 1]);
        return finish(r, [&] {
            return kMerged ? entries.attn_merged(&c, q, out, b, pages, prefix, len, cu, batch, total, max_new, max_ctx, hq, scale, w, bytes, s)
                           : entries.attn_resume(&c, q, out, b, pages, prefix, len, cu, batch, total, max_new, max_ctx, hq, scale, s);
        });
    });
}

// decode with the caller's workspace or the library's own
template <bool kStatic>
PyObject* attn_decode(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded(n, kStatic ? 9 : 10, [&] {
        Reader r;
        ag_kv_cache c;
        const at::Tensor *bt, *lens, *ws = nullptr;
        r.cache(a[0], c);
        void *q = r.device(a[1]), *out = r.device(a[2]);
        const int32_t *b = r.ints(a[3], &bt), *ctx = r.ints(a[4], &lens);
        const int32_t pages = r.size(bt, 1), batch = r.size(lens, 0), max_ctx = r.number(a[5]), hq = r.number(a[6]);
        const float scale = r.real(a[7]);
        void* w = kStatic ? nullptr : r.device(a[8], &ws);
        const size_t bytes = ws && r.plain ? (size_t)ws->numel() * ws->element_size() : 0;
        void* s = r.stream(a[n - 1]);
        return finish(r, [&] {
            return kStatic ? entries.attn_decode_static(&c, q, out, b, pages, ctx, batch, max_ctx, hq, scale, s)
                           : entries.attn_decode(&c, q, out, b, pages, ctx, batch, max_ctx, hq, scale, w, bytes, s);
        });
    });
}

PyObject* decode_step(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded(n, 12, [&] {
        Reader r;
        ag_kv_cache c;
        const at::Tensor *bt, *lens, *ws = nullptr;
        r.cache(a[0], c);
        void *k = r.device(a[1]), *v = r.device(a[2]), *q = r.device(a[3]), *out = r.device(a[4]);
        const int32_t *b = r.ints(a[5], &bt), *ctx = r.ints(a[6], &lens);
        const int32_t pages = r.size(bt, 1), batch = r.size(lens, 0), max_ctx = r.number(a[7]), hq = r.number(a[8]);
        const float scale = r.real(a[9]);
        void* w = r.device(a[10], &ws);
        const size_t bytes = ws && r.plain ? (size_t)ws->numel() * ws->element_size() : 0;
        void* s = r.stream(a[11]);
        return finish(r, [&] { return entries.decode_step(&c, k, v, q, out, b, pages, ctx, batch, max_ctx, hq, scale, w, bytes, s); });
    });
}

// setup(KVCache, _cuda_getDevice, _cuda_getCurrentRawStream, addresses of the entry points in the order of Entries)
PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    void** at = reinterpret_cast<void**>(&entries);
    constexpr Py_ssize_t kEntries = sizeof(Entries) / sizeof(void*);
    if (n != 3 + kEntries) { PyErr_SetString(PyExc_TypeError, "setup: wrong number of arguments"); return nullptr; }
    for (Py_ssize_t i = 0; i < kEntries; ++i) {
        at[i] = PyLong_AsVoidPtr(a[3 + i]);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_INCREF(a[0]);
    Py_INCREF(a[1]);
    Py_INCREF(a[2]);
    cache_type = a[0];
    get_device = a[1];
    get_raw_stream = a[2];
    Py_RETURN_NONE;
}

#define AG_METHOD(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(+fn)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    AG_METHOD("setup", setup), AG_METHOD("kv_append", kv_append), AG_METHOD("attn_prefill", attn_prefill),
    AG_METHOD("attn_resume", attn_resume<false>), AG_METHOD("attn_merged", attn_resume<true>),
    AG_METHOD("attn_decode", attn_decode<false>), AG_METHOD("attn_decode_static", attn_decode<true>),
    AG_METHOD("decode_step", decode_step), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "agcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_agcall()
{
    struct { PyObject** at; const char* name; } names[] = {
        {&n_k_pool, "k_pool"}, {&n_v_pool, "v_pool"}, {&n_num_pages, "num_pages"}, {&n_page_size, "page_size"},
        {&n_num_kv_heads, "num_kv_heads"}, {&n_head_dim, "head_dim"}, {&n_dtype, "dtype"}, {&n_cuda_stream, "cuda_stream"}};
    for (auto& x : names)
        if (!(*x.at = PyUnicode_InternFromString(x.name))) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", AG_BUILT_FOR) < 0) { Py_DECREF(m); return nullptr; }       // binding.py looks at it first
    return m;
}
