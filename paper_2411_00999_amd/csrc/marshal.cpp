// Python's side of the C ABI: a CPython extension that takes tensors, numbers and None and calls the library's entry points
// with their addresses.  Argument marshalling only, as binding.py, which keeps the checks, defaults and errors of the public
// functions.  The calls of one small layer are bound by the host: through ctypes, with the addresses taken in Python, those of
// B=4 T=128 D=256 fp32 took 5.8 (forward), 11.7 (backward, two launches) and 5.5 us (estimate) of host time where a launch
// takes 2.4 to 3.6; so 4.0, 9.4 and 4.2, and the three in a row 22.5 -> 16.6 us.
//
// The entry points are looked up in the library that the process has loaded already (bind), so nothing is linked against
// it.  Like ctypes, a call releases the interpreter's lock while it runs.
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/core/Tensor.h>
#include <dlfcn.h>

#include <exception>
#include <tuple>
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/lnpegn.h"

namespace {

struct Raised {};                    // a Python error has been set

PyObject *g_get_device, *g_get_raw_stream;                   // torch._C's
PyObject *s_data_ptr, *s_cuda_stream, *s_dtype;              // interned names

struct Owned {                       // a reference to be given back
    PyObject *o;
    explicit Owned(PyObject *p) : o(p)
    {
        if (!o) throw Raised{};
    }
    ~Owned() { Py_XDECREF(o); }
    Owned(const Owned &) = delete;
    Owned &operator=(const Owned &) = delete;
};

// Integers are taken modulo their width, as ctypes takes them.
unsigned long long integer(PyObject *o)
{
    if (PyLong_CheckExact(o)) {
        const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
        if (v == (unsigned long long)-1 && PyErr_Occurred()) throw Raised{};
        return v;
    }
    const Owned index(PyNumber_Index(o));
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(index.o);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) throw Raised{};
    return v;
}

// None or a tensor (subclasses and other objects by their own data_ptr method; a number is no address).
void *address(PyObject *o)
{
    if (o == Py_None) return nullptr;
    if (THPVariable_CheckExact(o)) return THPVariable_Unpack(o).data_ptr();
    const Owned at(PyObject_CallMethodNoArgs(o, s_data_ptr));
    return reinterpret_cast<void *>((uintptr_t)integer(at.o));
}

// A tensor of a type that the library has, or the type's number.
lnpegn_dtype element_type(PyObject *o)
{
    if (THPVariable_Check(o)) {
        const at::ScalarType t = THPVariable_Unpack(o).scalar_type();
        if (t == at::kFloat) return LNPEGN_F32;
        if (t == at::kBFloat16) return LNPEGN_BF16;
        const Owned dtype(PyObject_GetAttr(o, s_dtype));
        PyErr_Format(PyExc_TypeError, "unsupported dtype %S", dtype.o);
        throw Raised{};
    }
    return (lnpegn_dtype)(int)integer(o);
}

// A stream object, or None for the current device's current one.
void *stream_handle(PyObject *o)
{
    if (o == Py_None) {
        const Owned device(PyObject_CallNoArgs(g_get_device));
        const Owned raw(PyObject_CallOneArg(g_get_raw_stream, device.o));
        return reinterpret_cast<void *>((uintptr_t)integer(raw.o));
    }
    const Owned raw(PyObject_GetAttr(o, s_cuda_stream));
    return raw.o == Py_None ? nullptr : reinterpret_cast<void *>((uintptr_t)integer(raw.o));
}

template <typename A>
A argument(PyObject *o)
{
    if constexpr (std::is_pointer_v<A>) {
        return static_cast<A>(address(o));
    } else if constexpr (std::is_same_v<A, lnpegn_dtype>) {
        return element_type(o);
    } else if constexpr (std::is_floating_point_v<A>) {
        const double v = PyFloat_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) throw Raised{};
        return (A)v;
    } else {
        return (A)integer(o);
    }
}

template <typename F>
PyObject *guarded(F body)            // C++ exceptions (a tensor without storage) become Python's
{
    try {
        return body();
    } catch (const Raised &) {
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

bool expect(const char *name, Py_ssize_t n, Py_ssize_t want)
{
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, not %zd", name, want, n);
    return false;
}

// The last argument of every entry point is the stream.
template <typename... A, size_t... I>
PyObject *invoke(int (*fn)(A...), const char *name, PyObject *const *args, Py_ssize_t n, std::index_sequence<I...>)
{
    constexpr size_t kArgs = sizeof...(A);
    if (!expect(name, n, (Py_ssize_t)kArgs)) return nullptr;
    if (!fn) return PyErr_Format(PyExc_RuntimeError, "%s: no library bound", name);
    return guarded([&]() -> PyObject * {
        std::tuple<A...> values{[&]() -> A {
            if constexpr (I == kArgs - 1) return stream_handle(args[I]);
            else return argument<A>(args[I]);
        }()...};
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = fn(std::get<I>(values)...);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    });
}
template <typename... A>
PyObject *invoke(int (*fn)(A...), const char *name, PyObject *const *args, Py_ssize_t n)
{
    return invoke(fn, name, args, n, std::index_sequence_for<A...>{});
}

#define ENTRY_POINTS(X)                                                                                              \
    X(ln_fwd_stats) X(ln_fwd) X(ln_bwd) X(ln_bwd_pegn) X(ln_bwd_pegn_static) X(ln_bwd_deferred) X(ln_bwd_pegn_deferred) \
    X(ln_bwd_ex) X(rms_fwd) X(rms_bwd_ex) X(gns_estimate) X(gns_ema_update) X(gns_offline) X(linear_pegn)              \
    X(embedding_pegn) X(embedding_sort_ids) X(embedding_pegn_presorted) X(lnpegn_stream_probe)

#define DEFINE(name)                                                                                   \
    decltype(&::name) p_##name;                                                                        \
    PyObject *py_##name(PyObject *, PyObject *const *args, Py_ssize_t n) { return invoke(p_##name, #name, args, n); }
ENTRY_POINTS(DEFINE)
#undef DEFINE

decltype(&::lnpegn_reduce_deferred) p_lnpegn_reduce_deferred;
// (workspaces: a collection of tensors, whose number it can tell, B, T, D, the type's number, stream)
PyObject *py_reduce_deferred(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (!expect("reduce_deferred", n, 6)) return nullptr;
    if (!p_lnpegn_reduce_deferred) return PyErr_Format(PyExc_RuntimeError, "reduce_deferred: no library bound");
    return guarded([&]() -> PyObject * {
        if (PyObject_Size(args[0]) < 0) throw Raised{};
        const Owned list(PySequence_Tuple(args[0]));               // (a tuple: no other thread changes its length)
        std::vector<void *> at((size_t)PyTuple_GET_SIZE(list.o));
        for (size_t i = 0; i < at.size(); ++i) at[i] = address(PyTuple_GET_ITEM(list.o, (Py_ssize_t)i));
        const int B = argument<int>(args[1]), T = argument<int>(args[2]), D = argument<int>(args[3]);
        const lnpegn_dtype dt = (lnpegn_dtype)argument<int>(args[4]);
        void *stream = stream_handle(args[5]);
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = p_lnpegn_reduce_deferred(at.data(), (int)at.size(), B, T, D, dt, stream);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    });
}

// The shape of a contiguous tensor [B,T,D] on the GPU.
PyObject *py_check3(PyObject *, PyObject *o)
{
    return guarded([&]() -> PyObject * {
        if (!THPVariable_Check(o)) {
            PyErr_SetString(PyExc_TypeError, "expected a tensor");
            return nullptr;
        }
        const at::Tensor &t = THPVariable_Unpack(o);
        if (t.dim() != 3 || !t.is_contiguous() || !t.is_cuda()) {
            PyErr_SetString(PyExc_ValueError, "expected a contiguous CUDA tensor [B,T,D]");
            return nullptr;
        }
        return Py_BuildValue("LLL", (long long)t.size(0), (long long)t.size(1), (long long)t.size(2));
    });
}

// (n_groups, B) of the norms that gns_estimate takes.
PyObject *py_check_norms(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (!expect("check_norms", n, 2)) return nullptr;
    return guarded([&]() -> PyObject * {
        if (!THPVariable_Check(args[0]) || !THPVariable_Check(args[1])) {
            PyErr_SetString(PyExc_TypeError, "expected tensors");
            return nullptr;
        }
        const at::Tensor &pe = THPVariable_Unpack(args[0]), &big = THPVariable_Unpack(args[1]);
        if (pe.scalar_type() != at::kFloat || big.scalar_type() != at::kFloat) {
            PyErr_SetString(PyExc_TypeError, "gns_estimate takes fp32 norms");
            return nullptr;
        }
        if (!pe.is_contiguous() || !big.is_contiguous()) {
            PyErr_SetString(PyExc_ValueError, "gns_estimate takes contiguous tensors");
            return nullptr;
        }
        if (pe.dim() != 2) {
            PyErr_SetString(PyExc_ValueError, "pe_sq must be [n_groups,B]");
            return nullptr;
        }
        if (big.numel() != pe.size(0)) {
            PyErr_SetString(PyExc_ValueError, "big_sq must hold one value per group");
            return nullptr;
        }
        return Py_BuildValue("LL", (long long)pe.size(0), (long long)pe.size(1));
    });
}

// bind(path of the library): looks the entry points up in the library loaded from there.
PyObject *py_bind(PyObject *, PyObject *path)
{
    return guarded([&]() -> PyObject * {
        const char *name = PyUnicode_AsUTF8(path);
        if (!name) return nullptr;
        void *lib = dlopen(name, RTLD_NOW | RTLD_NOLOAD);
        if (!lib) {
            PyErr_Format(PyExc_RuntimeError, "%s is not loaded", name);
            return nullptr;
        }
        auto find = [&](auto &fn, const char *symbol) {
            fn = reinterpret_cast<std::remove_reference_t<decltype(fn)>>(dlsym(lib, symbol));
            if (fn) return;
            PyErr_Format(PyExc_RuntimeError, "%s has no %s", name, symbol);
            throw Raised{};
        };
#define FIND(name) find(p_##name, #name);
        ENTRY_POINTS(FIND)
#undef FIND
        find(p_lnpegn_reduce_deferred, "lnpegn_reduce_deferred");
        const Owned torch_c(PyImport_ImportModule("torch._C"));
        Py_XSETREF(g_get_device, PyObject_GetAttrString(torch_c.o, "_cuda_getDevice"));
        Py_XSETREF(g_get_raw_stream, PyObject_GetAttrString(torch_c.o, "_cuda_getCurrentRawStream"));
        if (!g_get_device || !g_get_raw_stream) return nullptr;
        Py_RETURN_NONE;
    });
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr},
PyMethodDef g_methods[] = {ENTRY_POINTS(METHOD) METHOD(reduce_deferred) METHOD(check_norms)
                           {"check3", py_check3, METH_O, nullptr},
                           {"bind", py_bind, METH_O, nullptr},
                           {nullptr, nullptr, 0, nullptr}};
#undef METHOD

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal()
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    s_dtype = PyUnicode_InternFromString("dtype");
    if (!s_data_ptr || !s_cuda_stream || !s_dtype) return nullptr;
    return PyModule_Create(&g_module);
}
