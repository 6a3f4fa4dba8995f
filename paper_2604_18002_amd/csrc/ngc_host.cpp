// CPython front of the C ABI: turns tensors into the plain pointers and structs of ngc.h and calls the entry point.
//
// The Python binding used ctypes for this: building an ngc_cache out of a dozen attribute reads and converting a dozen
// arguments took ~6 us of the 8.5 us a decode step cost on the host, more than the kernel runs for a small cache.  Here it took
// 1.1 us through the tensors' methods, and takes 0.3 us with plain tensors read directly (ngc_torch.cpp).  Marshalling only: no
// state is kept between calls, nothing is remembered about a tensor, and every check is the C ABI's own (plus the contiguity the binding always asked for).  What it takes is what ctypes took: a cache
// with a view() of its own is asked for it, a structure must be of its type, a number may be a ctypes one.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <dlfcn.h>
#include <stdint.h>
#include <string.h>

#include "../../include/ngc.h"
#include "ngc_torch.h"

namespace {

#define NGC_HOST_ENTRIES(X) \
    X(perturbed_keys) X(keep_counts) X(evict) X(subset_logprob) X(subset_logprob_backward) X(lmem) X(cache_append) \
    X(decode_attn) X(decode_step) X(decode_attn_static) X(score_keys) X(replay_attn) X(paged_evict) X(paged_append) \
    X(paged_decode_attn) X(paged_score_keys)

// the library's entry points, looked up once by open()
struct Entries {
#define X(name) decltype(&::ngc_##name) name = nullptr;
    NGC_HOST_ENTRIES(X)
#undef X
} lib;

// attribute and method names, interned once
struct Names {
    PyObject *k, *v, *len, *pos, *Hq, *k_pool, *v_pool, *pos_pool, *table, *free_stack, *free_count, *shape, *data_ptr,
        *numel, *is_contiguous, *view, *value;
} names;

// reads plain tensors directly; null until torch_reader() (torch may be imported later, or never) and without a reader that fits
ngc_read_tensor_fn read_tensor = nullptr;
// what stream_readers() was given: the current device, and the raw stream of a device
PyObject *device_of = nullptr, *stream_of = nullptr;

// what types() was given: the binding's own classes and functions
struct Types {
    PyObject *argument_error;               // raised for an argument of the wrong type
    PyObject *cache_class, *paged_class;    // Cache and PagedCache, and their view(): what the front reads in its place
    PyObject *cache, *paged, *params;       // the ctypes structures
    PyObject *simple;                       // base of ctypes' numbers
    PyObject *cache_view, *paged_view;
} types;

struct Ref {   // a new reference, released at the end of the scope
    PyObject *o;
    explicit Ref(PyObject *p) : o(p) {}
    ~Ref() { Py_XDECREF(o); }
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
};

// Readers of one argument.  On failure a Python error is set and the value is 0; once one is set the others read
// nothing (Python code must not run then), and call() does not call.
void *ptr(PyObject *t)
{
    if (t == Py_None || PyErr_Occurred()) return nullptr;
    ngc_tensor x;
    if (read_tensor && read_tensor(t, &x)) return x.data;
    const Ref r(PyObject_CallMethodNoArgs(t, names.data_ptr));
    return r.o ? PyLong_AsVoidPtr(r.o) : nullptr;
}
void wrong_type(PyObject *o, const char *wanted)
{
    PyErr_Clear();
    PyErr_Format(types.argument_error ? types.argument_error : PyExc_TypeError, "%s expected instead of %s instance", wanted,
                 Py_TYPE(o)->tp_name);
}
// Numbers as ctypes takes them: anything with __index__ (__float__), or a ctypes number.
template <class T, class Read>
T number(PyObject *o, const char *wanted, Read read)
{
    if (PyErr_Occurred()) return 0;
    T x = (T)read(o);
    if (x != (T)-1 || !PyErr_Occurred()) return x;
    PyErr_Clear();
    if (types.simple && PyObject_IsInstance(o, types.simple) == 1) {
        const Ref v(PyObject_GetAttr(o, names.value));
        if (v.o) {
            x = (T)read(v.o);
            if (x != (T)-1 || !PyErr_Occurred()) return x;
        }
    }
    wrong_type(o, wanted);
    return 0;
}
int64_t i64(PyObject *o) { return number<int64_t>(o, "int", PyLong_AsUnsignedLongLongMask); }
int32_t i32(PyObject *o) { return (int32_t)i64(o); }
float f32(PyObject *o) { return number<float>(o, "float", PyFloat_AsDouble); }
size_t bytes(PyObject *t)   // elements of a uint8 workspace tensor
{
    if (PyErr_Occurred()) return 0;
    ngc_tensor x;
    if (read_tensor && read_tensor(t, &x)) return (size_t)x.numel;
    const Ref r(PyObject_CallMethodNoArgs(t, names.numel));
    return r.o ? PyLong_AsSize_t(r.o) : 0;
}
void *stream(PyObject *o) { return o == Py_None || PyErr_Occurred() ? nullptr : PyLong_AsVoidPtr(o); }

// The attributes of a cache.  `dict`: where they are if the object is of the binding's own class, else null.
struct Object {
    PyObject *o, *dict = nullptr;
    ~Object() { Py_XDECREF(dict); }
    PyObject *get(PyObject *name) const      // a new reference
    {
        PyObject *v = dict ? PyDict_GetItemWithError(dict, name) : nullptr;
        Py_XINCREF(v);
        return v || PyErr_Occurred() ? v : PyObject_GetAttr(o, name);
    }
};

void *attr_ptr(const Object &o, PyObject *name, bool contiguous)
{
    if (PyErr_Occurred()) return nullptr;
    const Ref t(o.get(name));
    if (!t.o) return nullptr;
    ngc_tensor x;
    if (read_tensor && read_tensor(t.o, &x) && (x.contiguous || !contiguous)) return x.data;
    if (contiguous) {
        const Ref c(PyObject_CallMethodNoArgs(t.o, names.is_contiguous));
        if (!c.o) return nullptr;
        if (!PyObject_IsTrue(c.o)) {
            PyErr_Format(PyExc_AssertionError, "%U must be contiguous", name);
            return nullptr;
        }
    }
    return ptr(t.o);
}

// The first `count` sizes of o.name into d; the tensor must have exactly that many dimensions.
void sizes(const Object &o, PyObject *name, int32_t *d, Py_ssize_t count)
{
    if (PyErr_Occurred()) return;
    const Ref t(o.get(name));
    if (!t.o) return;
    ngc_tensor x;
    if (read_tensor && read_tensor(t.o, &x) && x.dims == count) {
        for (Py_ssize_t i = 0; i < count; ++i) d[i] = (int32_t)x.sizes[i];
        return;
    }
    const Ref s(PyObject_GetAttr(t.o, names.shape));
    if (!s.o) return;
    if (!PyTuple_Check(s.o) || PyTuple_GET_SIZE(s.o) != count) {
        PyErr_Format(PyExc_ValueError, "%U must have %zd dimensions", name, count);
        return;
    }
    for (Py_ssize_t i = 0; i < count; ++i) d[i] = i32(PyTuple_GET_ITEM(s.o, i));
}

int32_t attr_i32(const Object &o, PyObject *name)
{
    if (PyErr_Occurred()) return 0;
    const Ref v(o.get(name));
    return v.o ? i32(v.o) : 0;
}

// Copies a ctypes structure; an object of another type raises.
template <class T>
void copy_struct(PyObject *o, PyObject *type, const char *wanted, T *to)
{
    const int is = type ? PyObject_IsInstance(o, type) : 1;
    if (is < 0) return;
    Py_buffer b;
    if (!is || PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return wrong_type(o, wanted);
    if (b.len == (Py_ssize_t)sizeof(T)) __builtin_memcpy(to, b.buf, sizeof(T));
    else wrong_type(o, wanted);
    PyBuffer_Release(&b);
}

// Whether c.o.view() is the binding's own method, whose reading of the tensors is done here.  Anything else is called and
// its structure copied.
template <class T>
bool own_view(Object &c, PyObject *own_class, PyObject *own, PyObject *type, const char *wanted, T *v)
{
    if (PyErr_Occurred()) return false;
    PyTypeObject *const t = Py_TYPE(c.o);
    if (reinterpret_cast<PyObject *>(t) == own_class && PyDict_GetItemWithError(t->tp_dict, names.view) == own) {
        c.dict = PyObject_GenericGetDict(c.o, nullptr);
        if (!c.dict) return false;
        if (!PyDict_GetItemWithError(c.dict, names.view)) return !PyErr_Occurred();
        Py_CLEAR(c.dict);
    }
    const Ref m(PyObject_GetAttr(c.o, names.view));
    if (!m.o) return false;
    if (PyMethod_Check(m.o) && PyMethod_GET_SELF(m.o) == c.o && PyMethod_GET_FUNCTION(m.o) == own) return true;
    const Ref r(PyObject_CallNoArgs(m.o));
    if (r.o) copy_struct(r.o, type, wanted, v);
    return false;
}

ngc_cache cache_of(PyObject *o)
{
    ngc_cache v{};
    Object c{o};
    if (!own_view(c, types.cache_class, types.cache_view, types.cache, "ngc_cache", &v)) return v;
    int32_t d[5] = {};
    sizes(c, names.k, d, 5);
    v.L = d[0]; v.B = d[1]; v.Hkv = d[2]; v.cap = d[3]; v.D = d[4];
    v.Hq = attr_i32(c, names.Hq);
    v.k = attr_ptr(c, names.k, true);
    v.v = attr_ptr(c, names.v, true);
    v.len = (int32_t *)attr_ptr(c, names.len, true);
    v.pos = (int32_t *)attr_ptr(c, names.pos, false);
    return v;
}

ngc_paged_cache paged_of(PyObject *o)
{
    ngc_paged_cache v{};
    Object c{o};
    if (!own_view(c, types.paged_class, types.paged_view, types.paged, "ngc_paged_cache", &v)) return v;
    int32_t d[3] = {}, t[4] = {};
    sizes(c, names.k_pool, d, 3);
    sizes(c, names.table, t, 4);
    v.num_pages = d[0]; v.page_rows = d[1]; v.D = d[2];
    v.L = t[0]; v.B = t[1]; v.Hkv = t[2]; v.max_pages = t[3];
    v.Hq = attr_i32(c, names.Hq);
    v.k_pool = attr_ptr(c, names.k_pool, true);
    v.v_pool = attr_ptr(c, names.v_pool, true);
    v.pos_pool = (int32_t *)attr_ptr(c, names.pos_pool, false);
    v.table = (int32_t *)attr_ptr(c, names.table, true);
    v.len = (int32_t *)attr_ptr(c, names.len, true);
    v.free_stack = (int32_t *)attr_ptr(c, names.free_stack, true);
    v.free_count = (int32_t *)attr_ptr(c, names.free_count, true);
    return v;
}

// A copy of the ngc_evict_params inside a ctypes structure.
ngc_evict_params params_of(PyObject *p)
{
    ngc_evict_params v{};
    if (!PyErr_Occurred()) copy_struct(p, types.params, "ngc_evict_params", &v);
    return v;
}

// Calls the entry point unless reading the arguments failed; its return code comes back as an int.
template <class... P, class... A>
PyObject *call(int (*fn)(P...), A... args)
{
    if (PyErr_Occurred()) return nullptr;
    if (!fn) {
        PyErr_SetString(PyExc_RuntimeError, "the library has not been opened");
        return nullptr;
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(static_cast<P>(args)...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

bool want(Py_ssize_t got, Py_ssize_t count)
{
    if (got == count) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", count, got);
    return false;
}

#define ENTRY(name, count) \
    PyObject *name##_(PyObject *, PyObject *const *a, Py_ssize_t n) { if (!want(n, count)) return nullptr;
#define END }
template <class T> T *as(PyObject *o) { return reinterpret_cast<T *>(ptr(o)); }

ENTRY(perturbed_keys, 7)
    const ngc_cache c = cache_of(a[0]);
    const ngc_evict_params p = params_of(a[3]);
    return call(lib.perturbed_keys, &c, i32(a[1]), as<float>(a[2]), &p, as<float>(a[4]), ptr(a[5]), bytes(a[5]),
                stream(a[6]));
END
ENTRY(keep_counts, 10)
    return call(lib.keep_counts, as<int32_t>(a[0]), i32(a[1]), i32(a[2]), i32(a[3]), i32(a[4]), i32(a[5]), i32(a[6]),
                i32(a[7]), as<int32_t>(a[8]), stream(a[9]));
END
ENTRY(evict, 11)
    const ngc_cache c = cache_of(a[0]);
    const ngc_evict_params p = params_of(a[4]);
    return call(lib.evict, &c, i32(a[1]), as<float>(a[2]), as<int32_t>(a[3]), &p, i32(a[5]), as<int32_t>(a[6]),
                as<int32_t>(a[7]), as<float>(a[8]), ptr(a[9]), bytes(a[9]), stream(a[10]));
END
ENTRY(subset_logprob, 10)
    return call(lib.subset_logprob, as<float>(a[0]), as<int32_t>(a[1]), as<int32_t>(a[2]), as<int32_t>(a[3]), i32(a[4]),
                i64(a[5]), i32(a[6]), as<float>(a[7]), ptr(a[8]), bytes(a[8]), stream(a[9]));
END
ENTRY(subset_logprob_backward, 12)
    return call(lib.subset_logprob_backward, as<float>(a[0]), as<int32_t>(a[1]), as<int32_t>(a[2]), as<int32_t>(a[3]),
                i32(a[4]), i64(a[5]), i32(a[6]), i32(a[7]), as<float>(a[8]), as<float>(a[9]), ptr(a[10]), bytes(a[10]),
                stream(a[11]));
END
ENTRY(lmem, 13)
    return call(lib.lmem, as<float>(a[0]), as<int32_t>(a[1]), as<float>(a[2]), i32(a[3]), i32(a[4]), i32(a[5]),
                i32(a[6]), i32(a[7]), as<float>(a[8]), as<float>(a[9]), as<float>(a[10]), as<float>(a[11]), stream(a[12]));
END
ENTRY(cache_append, 7)
    const ngc_cache c = cache_of(a[0]);
    return call(lib.cache_append, &c, i32(a[1]), ptr(a[2]), ptr(a[3]), as<int32_t>(a[4]), ptr(a[5]), bytes(a[5]),
                stream(a[6]));
END
ENTRY(decode_attn, 9)
    const ngc_cache c = cache_of(a[0]);
    return call(lib.decode_attn, &c, i32(a[1]), ptr(a[2]), f32(a[3]), i32(a[4]), as<float>(a[5]), as<float>(a[6]),
                ptr(a[7]), bytes(a[7]), stream(a[8]));
END
ENTRY(decode_step, 12)
    const ngc_cache c = cache_of(a[0]);
    return call(lib.decode_step, &c, i32(a[1]), ptr(a[2]), ptr(a[3]), as<int32_t>(a[4]), ptr(a[5]), f32(a[6]),
                i32(a[7]), as<float>(a[8]), as<float>(a[9]), ptr(a[10]), bytes(a[10]), stream(a[11]));
END
ENTRY(decode_attn_static, 9)
    const ngc_cache c = cache_of(a[0]);
    return call(lib.decode_attn_static, &c, i32(a[1]), ptr(a[2]), f32(a[3]), i32(a[4]), as<float>(a[5]),
                as<float>(a[6]), as<int32_t>(a[7]), stream(a[8]));
END
ENTRY(score_keys, 11)
    const ngc_cache c = cache_of(a[0]);
    return call(lib.score_keys, &c, i32(a[1]), ptr(a[2]), as<float>(a[3]), i32(a[4]), f32(a[5]), i32(a[6]), i32(a[7]),
                as<float>(a[8]), ptr(a[9]), bytes(a[9]), stream(a[10]));
END
ENTRY(replay_attn, 14)
    return call(lib.replay_attn, ptr(a[0]), ptr(a[1]), ptr(a[2]), as<int32_t>(a[3]), i32(a[4]), i32(a[5]), i32(a[6]),
                i32(a[7]), i32(a[8]), i32(a[9]), f32(a[10]), as<float>(a[11]), ptr(a[12]), bytes(a[12]), stream(a[13]));
END
ENTRY(paged_evict, 12)
    const ngc_paged_cache c = paged_of(a[0]);
    const ngc_evict_params p = params_of(a[5]);
    return call(lib.paged_evict, &c, i32(a[1]), as<float>(a[2]), i64(a[3]), as<int32_t>(a[4]), &p, i32(a[6]),
                as<int32_t>(a[7]), as<int32_t>(a[8]), as<float>(a[9]), ptr(a[10]), bytes(a[10]), stream(a[11]));
END
ENTRY(paged_append, 7)
    const ngc_paged_cache c = paged_of(a[0]);
    return call(lib.paged_append, &c, i32(a[1]), ptr(a[2]), ptr(a[3]), as<int32_t>(a[4]), ptr(a[5]), bytes(a[5]),
                stream(a[6]));
END
ENTRY(paged_decode_attn, 9)
    const ngc_paged_cache c = paged_of(a[0]);
    return call(lib.paged_decode_attn, &c, i32(a[1]), ptr(a[2]), f32(a[3]), i32(a[4]), as<float>(a[5]),
                as<float>(a[6]), ptr(a[7]), bytes(a[7]), stream(a[8]));
END
ENTRY(paged_score_keys, 11)
    const ngc_paged_cache c = paged_of(a[0]);
    return call(lib.paged_score_keys, &c, i32(a[1]), ptr(a[2]), as<float>(a[3]), i32(a[4]), f32(a[5]), i32(a[6]),
                i32(a[7]), as<float>(a[8]), ptr(a[9]), bytes(a[9]), stream(a[10]));
END

// open(path): the library the calls go to (already loaded by the binding, so this only finds its entry points)
PyObject *open_(PyObject *, PyObject *path)
{
    const char *p = PyUnicode_AsUTF8(path);
    if (!p) return nullptr;
    void *h = dlopen(p, RTLD_NOW | RTLD_LOCAL);
    if (!h) return PyErr_Format(PyExc_RuntimeError, "%s", dlerror());
    Entries e;
#define X(name) \
    e.name = reinterpret_cast<decltype(e.name)>(dlsym(h, "ngc_" #name)); \
    if (!e.name) return PyErr_Format(PyExc_RuntimeError, "%s: no entry point ngc_" #name, p);
    NGC_HOST_ENTRIES(X)
#undef X
    lib = e;
    Py_RETURN_NONE;
}

// torch_reader(path, identity) -> whether plain tensors are read by this library from now on.  Not if it cannot be loaded or
// was compiled against another torch than the one that has been imported, `identity`: then all tensors go by their methods.
ENTRY(torch_reader, 2)
    const char *path = PyUnicode_AsUTF8(a[0]);
    const char *identity = path ? PyUnicode_AsUTF8(a[1]) : nullptr;
    if (!identity) return nullptr;
    read_tensor = nullptr;
    void *h = dlopen(path, RTLD_NOW | RTLD_LOCAL);
    if (!h) Py_RETURN_FALSE;
    const auto built_for = reinterpret_cast<ngc_torch_identity_fn>(dlsym(h, "ngc_torch_identity"));
    const auto fn = reinterpret_cast<ngc_read_tensor_fn>(dlsym(h, "ngc_read_tensor"));
    if (!built_for || !fn || strcmp(built_for(), identity) != 0) {
        dlclose(h);
        Py_RETURN_FALSE;
    }
    read_tensor = fn;
    Py_RETURN_TRUE;
END

// stream_readers(device, stream): torch's own functions for the current device and a device's current raw stream.
ENTRY(stream_readers, 2)
    Py_INCREF(a[0]);
    Py_XSETREF(device_of, a[0]);
    Py_INCREF(a[1]);
    Py_XSETREF(stream_of, a[1]);
    Py_RETURN_NONE;
END

// current_stream() -> the raw stream as an int
PyObject *current_stream(PyObject *, PyObject *)
{
    if (!device_of || !stream_of) {
        PyErr_SetString(PyExc_RuntimeError, "stream_readers() has not been called");
        return nullptr;
    }
    const Ref device(PyObject_CallNoArgs(device_of));
    return device.o ? PyObject_CallOneArg(stream_of, device.o) : nullptr;
}

// types(ArgumentError, Cache, PagedCache, ngc_cache, ngc_paged_cache, ngc_evict_params, _SimpleCData)
ENTRY(types, 7)
    PyObject **const to[] = {&types.argument_error, &types.cache_class, &types.paged_class, &types.cache, &types.paged,
                             &types.params, &types.simple};
    for (int i = 0; i < 7; ++i) {
        Py_INCREF(a[i]);
        Py_XSETREF(*to[i], a[i]);
    }
    Py_XSETREF(types.cache_view, PyObject_GetAttr(a[1], names.view));
    Py_XSETREF(types.paged_view, PyObject_GetAttr(a[2], names.view));
    if (!types.cache_view || !types.paged_view) return nullptr;
    Py_RETURN_NONE;
END

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(&name##_)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"open", open_, METH_O, nullptr}, FAST(torch_reader),
    {"current_stream", current_stream, METH_NOARGS, nullptr}, FAST(stream_readers), FAST(types),
    FAST(perturbed_keys), FAST(keep_counts), FAST(evict), FAST(subset_logprob), FAST(subset_logprob_backward), FAST(lmem),
    FAST(cache_append), FAST(decode_attn), FAST(decode_step), FAST(decode_attn_static), FAST(score_keys),
    FAST(replay_attn), FAST(paged_evict), FAST(paged_append), FAST(paged_decode_attn), FAST(paged_score_keys),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ngc_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ngc_host(void)
{
    struct { PyObject **at; const char *name; } const all[] = {
        {&names.k, "k"}, {&names.v, "v"}, {&names.len, "len"}, {&names.pos, "pos"}, {&names.Hq, "Hq"},
        {&names.k_pool, "k_pool"}, {&names.v_pool, "v_pool"}, {&names.pos_pool, "pos_pool"}, {&names.table, "table"},
        {&names.free_stack, "free_stack"}, {&names.free_count, "free_count"}, {&names.shape, "shape"},
        {&names.data_ptr, "data_ptr"}, {&names.numel, "numel"}, {&names.is_contiguous, "is_contiguous"},
        {&names.view, "view"}, {&names.value, "value"}};
    for (const auto &x : all)
        if (!(*x.at = PyUnicode_InternFromString(x.name))) return nullptr;
    return PyModule_Create(&module);
}
