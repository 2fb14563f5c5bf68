// CPython extension behind the functions of binding.py: turns torch tensors, numbers and descriptors into the arguments of
// the C ABI.  Nothing of the method is here.
//
// An eager pass over a small cache is bound by its calls (4 of them: 20 us of host time against 14 us on the GPU), and a
// call's time went into ctypes and some 80 attribute lookups on tensors.  A call whose arguments are all of the ordinary kind
// - exact torch tensors on the GPU and contiguous, plain ints and floats, the binding's own structures - is made
// here; any other returns None, with nothing launched, and binding.py takes its general path, which converts or refuses it
// as ever.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <array>
#include <cstdint>
#include <tuple>
#include <type_traits>
#include <utility>

#include "pikv.h"

namespace {

// The classes of binding.py's ctypes structures; set once by setup(), which the binding calls when it loads the library.
PyTypeObject *desc_type = nullptr, *policy_type = nullptr, *feedback_type = nullptr;

// Addresses of the library's functions, in the order of `Functions`.
enum Function {
    kRoute, kAttn, kAttnNoalloc, kUtility, kUtilityTracked, kEvict, kAppend, kStep, kStepPolicy, kCompress, kStamp, kPolicyUtility,
    kPolicyCompact, kPenalty, kFunctions
};
void *addresses[kFunctions] = {};

// Buffers of the ctypes structures, released when the call is over.
struct Buffers {
    Py_buffer view[3];
    int n = 0;
    void *get(PyObject *o) {
        if (PyObject_GetBuffer(o, &view[n], PyBUF_SIMPLE) != 0) {
            PyErr_Clear();
            return nullptr;
        }
        return view[n++].buf;
    }
    ~Buffers() {
        for (int i = 0; i < n; ++i) PyBuffer_Release(&view[i]);
    }
};

struct Args {
    PyObject *const *at;
    PyObject *const *begin;
    Buffers buffers;
    const at::Tensor *last = nullptr;    // the last tensor taken
    const at::Tensor *first = nullptr;
    bool usual = true;                   // every argument so far was of the ordinary kind (no exception: one costs as much as a call)

    template <typename T>
    T unusual() {
        usual = false;
        return T{};
    }
    const at::Tensor *tensor(PyObject *o) {
        if (o == Py_None) return nullptr;
        if (!THPVariable_CheckExact(o)) return unusual<const at::Tensor *>();
        const at::Tensor &t = THPVariable_Unpack(o);
        return t.is_cuda() && t.is_contiguous() ? &t : unusual<const at::Tensor *>();
    }
    template <typename T>
    T buffer(PyObject *o) {
        void *p = buffers.get(o);
        return p != nullptr ? static_cast<T>(p) : unusual<T>();
    }
};

// What a parameter of the C function is made of.
struct Stream {};      // void *: the caller's, as an integer, or None - torch's current one
struct Bytes {};       // size_t: of the tensor before it; takes no argument
struct Dtype {};       // int32_t: of the first argument, a tensor; takes none itself

template <typename T, typename Kind>
struct Take {
    static T from(Args &a) {
        PyObject *o = *a.at++;
        if constexpr (std::is_same_v<T, const pikv_desc *>) {
            return Py_TYPE(o) == desc_type ? a.template buffer<T>(o) : a.template unusual<T>();
        } else if constexpr (std::is_same_v<T, const pikv_policy_args *> || std::is_same_v<T, const pikv_router_feedback *>) {
            if (o == Py_None) return nullptr;
            const bool mine = Py_TYPE(o) == (std::is_same_v<T, const pikv_policy_args *> ? policy_type : feedback_type);
            return mine ? a.template buffer<T>(o) : a.template unusual<T>();
        } else if constexpr (std::is_pointer_v<T>) {
            const at::Tensor *t = a.tensor(o);
            a.last = t;
            if (a.first == nullptr) a.first = t;
            return t == nullptr ? nullptr : static_cast<T>(t->data_ptr());
        } else if constexpr (std::is_floating_point_v<T>) {
            if (PyFloat_CheckExact(o)) return static_cast<T>(PyFloat_AS_DOUBLE(o));
            if (!PyLong_CheckExact(o)) return a.template unusual<T>();
            int overflow = 0;
            const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
            return overflow == 0 ? static_cast<T>(static_cast<double>(v)) : a.template unusual<T>();
        } else {
            if (!PyLong_CheckExact(o) && !PyBool_Check(o)) return a.template unusual<T>();
            int overflow = 0;
            const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
            return overflow == 0 && v >= INT32_MIN && v <= INT32_MAX ? static_cast<T>(v) : a.template unusual<T>();
        }
    }
};
template <typename T>
struct Take<T, Stream> {
    static T from(Args &a) {
        PyObject *o = *a.at++;
        if (o == Py_None) {
            if (a.first == nullptr) return a.template unusual<T>();     // (a tensor on the GPU: the device is initialised)
            return c10::hip::getCurrentHIPStream().stream();
        }
        if (!PyLong_CheckExact(o)) return a.template unusual<T>();
        void *p = PyLong_AsVoidPtr(o);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            return a.template unusual<T>();
        }
        return p;
    }
};
template <typename T>
struct Take<T, Bytes> {
    static T from(Args &a) {
        return a.last != nullptr ? a.last->nbytes() : a.template unusual<T>();
    }
};
template <typename T>
struct Take<T, Dtype> {
    static T from(Args &a) {
        if (*a.begin == Py_None || a.first == nullptr) return a.template unusual<T>();
        const auto t = a.first->scalar_type();
        if (t == at::kFloat) return PIKV_F32;
        if (t == at::kBFloat16) return PIKV_BF16;
        return a.template unusual<T>();
    }
};

struct Plain {};
// The kind of parameter I: KINDS lists (index, kind) pairs for those that are not plain.
template <int INDEX, typename KIND>
struct At {};
template <int I, typename... KINDS>
struct KindOf {
    typedef Plain type;
};
template <int I, int INDEX, typename KIND, typename... REST>
struct KindOf<I, At<INDEX, KIND>, REST...> {
    typedef std::conditional_t<I == INDEX, KIND, typename KindOf<I, REST...>::type> type;
};
template <typename KIND>
constexpr int takes = std::is_same_v<KIND, Bytes> || std::is_same_v<KIND, Dtype> ? 0 : 1;

template <Function F, typename FN, typename... KINDS>
struct Caller;
template <Function F, typename... A, typename... KINDS>
struct Caller<F, int (*)(A...), KINDS...> {
    template <size_t... I>
    static PyObject *run(PyObject *const *args, Py_ssize_t n, std::index_sequence<I...>) {
        constexpr int wanted = (0 + ... + takes<typename KindOf<(int)I, KINDS...>::type>);
        if (n != wanted || addresses[F] == nullptr || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
        try {
            Args a{args, args};
            // (braces: the arguments are taken from left to right)
            const std::tuple<A...> values{Take<A, typename KindOf<(int)I, KINDS...>::type>::from(a)...};
            if (!a.usual || a.first == nullptr) Py_RETURN_NONE;
            auto call = [&]() noexcept { return std::apply(reinterpret_cast<int (*)(A...)>(addresses[F]), values); };
            int status;
            Py_BEGIN_ALLOW_THREADS
            status = call();
            Py_END_ALLOW_THREADS
            return PyLong_FromLong(status);
        } catch (...) {                  // torch's own refusal: the general path reports it
            PyErr_Clear();
            Py_RETURN_NONE;
        }
    }
    static PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n) {
        return run(args, n, std::index_sequence_for<A...>{});
    }
};

template <Function F, typename FN, typename... KINDS>
PyMethodDef method(const char *name) {
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(&Caller<F, FN, KINDS...>::call)), METH_FASTCALL, nullptr};
}

// setup(descriptor class, policy class, feedback class, {name: address})
PyObject *setup(PyObject *, PyObject *args);

PyMethodDef methods[] = {
    {"setup", setup, METH_VARARGS, nullptr},
    method<kRoute, decltype(&pikv_route), At<7, Dtype>, At<11, Stream>>("pikv_route"),
    method<kAttn, decltype(&pikv_sharded_attn), At<18, Bytes>, At<19, Stream>>("pikv_sharded_attn"),
    method<kAttnNoalloc, decltype(&pikv_sharded_attn_noalloc), At<17, Stream>>("pikv_sharded_attn_noalloc"),
    method<kUtility, decltype(&pikv_update_utility), At<8, Stream>>("pikv_update_utility"),
    method<kUtilityTracked, decltype(&pikv_update_utility_tracked), At<12, Stream>>("pikv_update_utility_tracked"),
    method<kEvict, decltype(&pikv_evict), At<12, Stream>>("pikv_evict"),
    method<kAppend, decltype(&pikv_append), At<12, Stream>>("pikv_append"),
    method<kStep, decltype(&pikv_decode_step), At<26, Bytes>, At<27, Stream>>("pikv_decode_step"),
    method<kStepPolicy, decltype(&pikv_decode_step_policy), At<26, Bytes>, At<27, Stream>>("pikv_decode_step_policy"),
    method<kCompress, decltype(&pikv_compress), At<7, Stream>>("pikv_compress"),
    method<kStamp, decltype(&pikv_policy_stamp), At<11, Stream>>("pikv_policy_stamp"),
    method<kPolicyUtility, decltype(&pikv_policy_utility), At<12, Stream>>("pikv_policy_utility"),
    method<kPolicyCompact, decltype(&pikv_policy_compact), At<8, Stream>>("pikv_policy_compact"),
    method<kPenalty, decltype(&pikv_router_penalty), At<9, Stream>>("pikv_router_penalty"),
    {nullptr, nullptr, 0, nullptr},
};

PyObject *setup(PyObject *, PyObject *args) {
    PyObject *desc, *policy, *feedback, *table;
    if (!PyArg_ParseTuple(args, "O!O!O!O!", &PyType_Type, &desc, &PyType_Type, &policy, &PyType_Type, &feedback, &PyDict_Type, &table))
        return nullptr;
    for (int f = 0; f < kFunctions; ++f) {
        PyObject *address = PyDict_GetItemString(table, methods[f + 1].ml_name);
        if (address == nullptr) return PyErr_Format(PyExc_KeyError, "%s", methods[f + 1].ml_name);
        addresses[f] = PyLong_AsVoidPtr(address);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_INCREF(desc), Py_INCREF(policy), Py_INCREF(feedback);     // for the life of the process
    desc_type = reinterpret_cast<PyTypeObject *>(desc);
    policy_type = reinterpret_cast<PyTypeObject *>(policy);
    feedback_type = reinterpret_cast<PyTypeObject *>(feedback);
    Py_RETURN_NONE;
}

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pikv_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pikv_native(void) { return PyModule_Create(&module); }
