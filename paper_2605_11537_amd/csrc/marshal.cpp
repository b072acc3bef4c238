// Python extension that marshals the arguments of the library's calls: tensors to device pointers, ints, a stream handle.  Host code only.
//
// What a small call costs a Python program is its marshalling: through ctypes a tensor takes about 0.5 us (three attribute look-ups in Python and
// a conversion) and an int 0.1 us, a dozen of them per call.  Here a tensor's pointer is read from the tensor itself.  The calls keep
// their argument order and return their error code.  A tensor has to be on the device and contiguous (ValueError else).  An int may be any whole
// number, numpy's too (TypeError else).  The fields of a layer have to fit the struct's (OverflowError else); arguments of the other calls are
// reduced to their parameter's width, as ctypes does.
// Functions are typed by the C header and bound to the addresses of the library that binding.lib() has loaded and checked.
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cstring>
#include <exception>
#include <tuple>
#include <utility>

#include "../../include/moe_mpmc.h"

namespace {

struct Failed {};                       // a Python exception is set

// None is a null pointer
void *pointer_of(PyObject *o)
{
    if (o == Py_None) return nullptr;
    if (THPVariable_CheckExact(o)) {
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.is_contiguous()) {
            PyErr_SetString(PyExc_ValueError, "device-resident contiguous tensors only");
            throw Failed();
        }
        return t.data_ptr();
    }
    // a subclass, or anything else that answers as a tensor does
    auto truth = [](PyObject *v) {
        const int r = v ? PyObject_IsTrue(v) : -1;
        Py_XDECREF(v);
        if (r < 0) throw Failed();
        return r == 1;
    };
    if (!truth(PyObject_GetAttrString(o, "is_cuda")) || !truth(PyObject_CallMethod(o, "is_contiguous", nullptr))) {
        PyErr_SetString(PyExc_ValueError, "device-resident contiguous tensors only");
        throw Failed();
    }
    PyObject *p = PyObject_CallMethod(o, "data_ptr", nullptr);
    if (!p) throw Failed();
    const unsigned long long a = PyLong_AsUnsignedLongLongMask(p);
    Py_DECREF(p);
    if (a == (unsigned long long)-1 && PyErr_Occurred()) throw Failed();
    return reinterpret_cast<void *>(a);
}

unsigned long long integer_of(PyObject *o)
{
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);      // takes what has __index__
    if (v == (unsigned long long)-1 && PyErr_Occurred()) throw Failed();
    return v;
}

// a whole number that the field holds
void fit(PyObject *o, size_t &field)
{
    PyObject *whole = PyNumber_Index(o);
    if (!whole) throw Failed();
    field = PyLong_AsSize_t(whole);
    Py_DECREF(whole);
    if (field == (size_t)-1 && PyErr_Occurred()) throw Failed();
}
void fit(PyObject *o, int &field)
{
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);                  // takes what has __index__
    if (v == -1 && PyErr_Occurred()) throw Failed();
    if (over || v < INT_MIN || v > INT_MAX) {
        PyErr_Format(PyExc_OverflowError, "%R does not fit an int", o);
        throw Failed();
    }
    field = (int)v;
}

// what is no tensor comes as an address, an int itself: a stream, a struct in host memory
void *address_of(PyObject *o)
{
    if (o == Py_None) return nullptr;
    if (!PyLong_Check(o)) {
        PyErr_Format(PyExc_TypeError, "an address expected instead of %s instance", Py_TYPE(o)->tp_name);
        throw Failed();
    }
    return reinterpret_cast<void *>(integer_of(o));
}

template <class T, bool STREAM>
struct Arg {
    static T from(PyObject *o) { return static_cast<T>(integer_of(o)); }
};
template <class T, bool STREAM>
struct Arg<T *, STREAM> {
    static T *from(PyObject *o) { return static_cast<T *>(STREAM ? address_of(o) : pointer_of(o)); }
};
template <>
struct Arg<const sru_weights *, false> {
    static const sru_weights *from(PyObject *o) { return static_cast<const sru_weights *>(address_of(o)); }
};

// any C++ exception (torch throws where a tensor has no storage) becomes a Python one
template <class F>
PyObject *guarded(F &&f)
{
    try {
        return PyLong_FromLong(f());
    } catch (const Failed &) {
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception");
        return nullptr;
    }
}

bool counted(const char *name, Py_ssize_t n, size_t want)
{
    if ((size_t)n == want) return true;
    PyErr_Format(PyExc_TypeError, "%s takes %zu arguments (%zd given)", name, want, n);
    return false;
}

// the interpreter's lock is given back for the call itself: a launch may wait for room in the queue
template <class F>
int unlocked(F &&f)
{
    PyThreadState *state = PyEval_SaveThread();
    const int rc = f();                 // C functions: nothing is thrown
    PyEval_RestoreThread(state);
    return rc;
}

template <class... A, size_t... I>
PyObject *invoke(int (*f)(A...), PyObject *const *args, std::index_sequence<I...>)
{
    return guarded([&] {
        const std::tuple<A...> a{Arg<A, I + 1 == sizeof...(A)>::from(args[I])...};      // every call's last argument is its stream
        return unlocked([&] { return f(std::get<I>(a)...); });
    });
}
template <class... A>
PyObject *call(const char *name, int (*f)(A...), PyObject *const *args, Py_ssize_t n)
{
    if (!f) {
        PyErr_Format(PyExc_RuntimeError, "%s is not bound", name);
        return nullptr;
    }
    if (!counted(name, n, sizeof...(A))) return nullptr;
    return invoke(f, args, std::index_sequence_for<A...>());
}

#define CALLS(X)                                                                                                          \
    X(moe_route) X(moe_route_topk) X(sru_predict) X(replica_plan) X(moe_dispatch) X(moe_dispatch_static) X(moe_dispatch_topk)  \
    X(moe_plan_dispatch) X(moe_pack_weights) X(moe_expert_ffn) X(moe_expert_ffn_rows) X(moe_combine) X(moe_combine_topk)

#define DECLARE(NAME)                                                                                                     \
    decltype(&NAME) bound_##NAME = nullptr;                                                                               \
    PyObject *py_##NAME(PyObject *, PyObject *const *args, Py_ssize_t n) { return call(#NAME, bound_##NAME, args, n); }
CALLS(DECLARE)
#undef DECLARE

// The fields of moe_layer_args one by one in their order, then the stream.
decltype(&moe_layer_forward) bound_moe_layer_forward = nullptr;
constexpr int LAYER_POINTERS = 25, LAYER_SIZES = 3, LAYER_INTS = 16;
static_assert(sizeof(moe_layer_args) == LAYER_POINTERS * sizeof(void *) + LAYER_SIZES * sizeof(size_t) + LAYER_INTS * sizeof(int),
              "no padding: the fields are filled one after another");
PyObject *py_moe_layer_forward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (!bound_moe_layer_forward) {
        PyErr_SetString(PyExc_RuntimeError, "moe_layer_forward is not bound");
        return nullptr;
    }
    if (!counted("moe_layer_forward", n, LAYER_POINTERS + LAYER_SIZES + LAYER_INTS + 1)) return nullptr;
    return guarded([&] {
        struct {
            void *pointers[LAYER_POINTERS];
            size_t sizes[LAYER_SIZES];
            int ints[LAYER_INTS];
        } fields;
        PyObject *const *at = args;
        for (void *&p : fields.pointers) p = pointer_of(*at++);
        for (size_t &s : fields.sizes) fit(*at++, s);
        for (int &i : fields.ints) fit(*at++, i);
        moe_layer_args layer;
        memcpy(&layer, &fields, sizeof layer);
        void *stream = address_of(*at);
        return unlocked([&] { return bound_moe_layer_forward(&layer, stream); });
    });
}

// bind(name, address)
PyObject *py_bind(PyObject *, PyObject *args)
{
    const char *name;
    unsigned long long address;
    if (!PyArg_ParseTuple(args, "sK", &name, &address)) return nullptr;
#define BIND(NAME)                                                            \
    if (!strcmp(name, #NAME)) {                                               \
        bound_##NAME = reinterpret_cast<decltype(&NAME)>(address);            \
        Py_RETURN_NONE;                                                       \
    }
    CALLS(BIND)
    BIND(moe_layer_forward)
#undef BIND
    PyErr_Format(PyExc_ValueError, "no call named %s", name);
    return nullptr;
}

PyMethodDef methods[] = {
#define METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))py_##NAME, METH_FASTCALL, nullptr},
    CALLS(METHOD) METHOD(moe_layer_forward)
#undef METHOD
    {"bind", py_bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void)
{
    PyObject *m = PyModule_Create(&module);
    if (m && (PyModule_AddStringConstant(m, "build_id", MOE_BUILD_ID) < 0 || PyModule_AddStringConstant(m, "built_for", MOE_BUILT_FOR) < 0)) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
