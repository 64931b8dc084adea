// Python binding of the C ABI's launching calls: every function takes the arguments of its C counterpart in order.
//
// A call through ctypes cost the host 1.3 to 2.9 us for its arguments beside the 2.7 us of a kernel launch, which is what
// bounds operators of a few thousand elements; here it is 0.2 to 0.4 us.  Arguments: a pointer parameter takes a tensor (or what
// else has a data_ptr()) or None -- a pointer to host sizes an address or None --, an integer parameter whatever has an index.  A dtype takes
// the tensor passed just in front of it once more, a workspace size the tensor or None likewise.  The last parameter, the
// stream, takes a torch stream, a handle, or None for torch's current stream.  A status other than QSYNC_OK raises what
// `set_error` was given.  The GIL is released around the call.
#include <Python.h>

#include <pthread.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>
#include <stdexcept>
#include <string>
#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/qsync.h"

namespace {

PyObject* g_error          = nullptr;      // called with the status, returns the exception
PyObject* g_is_initialized = nullptr;      // torch.cuda.is_initialized
PyObject* g_current_stream = nullptr;      // torch.cuda.current_stream
// torch has initialised the device, which stays so (read and written under the GIL) -- but not in a process forked from this one,
// where torch refuses the device's use
bool g_device_ready = false;

struct PythonError : std::exception {};      // a Python error is set

const at::Tensor* as_tensor(PyObject* o) { return THPVariable_Check(o) ? &THPVariable_Unpack(o) : nullptr; }

uint64_t integer(PyObject* o)      // modulo 2^64, as ctypes takes them: of an int, or of what answers as one (numpy's integers)
{
    if(!PyIndex_Check(o))
    {
        PyErr_Format(PyExc_TypeError, "an integer is required (got type %s)", Py_TYPE(o)->tp_name);
        throw PythonError();
    }
    const uint64_t v = PyLong_AsUnsignedLongLongMask(o);
    if(v == static_cast<uint64_t>(-1) && PyErr_Occurred()) throw PythonError();
    return v;
}

uint64_t answer(PyObject* o, const char* method)
{
    PyObject* r = PyObject_CallMethod(o, method, nullptr);
    if(!r) throw PythonError();
    const uint64_t v = PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    if(PyErr_Occurred()) throw PythonError();
    return v;
}

void* pointer(PyObject* o)
{
    if(o == Py_None) return nullptr;
    if(THPVariable_CheckExact(o)) return THPVariable_Unpack(o).data_ptr();
    return reinterpret_cast<void*>(answer(o, "data_ptr"));      // (subclasses answer for themselves; a number has none)
}

int dtype_code(PyObject* o, at::ScalarType type)
{
    switch(type)
    {
    case at::kFloat: return QSYNC_F32;
    case at::kHalf: return QSYNC_F16;
    case at::kChar: return QSYNC_I8;
    case at::kInt: return QSYNC_I32;
    default: break;
    }
    PyObject* dt = PyObject_GetAttrString(o, "dtype");
    if(dt) { PyErr_SetObject(PyExc_KeyError, dt); Py_DECREF(dt); }
    throw PythonError();
}

// ... of what is no tensor but has a dtype
int dtype_code(PyObject* o)
{
    PyObject* dt = PyObject_GetAttrString(o, "dtype");
    if(!dt) throw PythonError();
    const bool known = THPDtype_Check(dt);
    if(!known) PyErr_SetObject(PyExc_KeyError, dt);
    const at::ScalarType type = known ? reinterpret_cast<THPDtype*>(dt)->scalar_type : at::ScalarType::Undefined;
    Py_DECREF(dt);
    if(!known) throw PythonError();
    return dtype_code(o, type);
}

void* stream_handle(PyObject* o)
{
    if(o == Py_None)
    {
        if(!g_device_ready)
        {
            PyObject* r = PyObject_CallNoArgs(g_is_initialized);
            if(!r) throw PythonError();
            const bool up = r == Py_True;
            Py_DECREF(r);
            if(!up)
            {   // the first use of the device initialises it, or says that there is none
                PyObject* s = PyObject_CallNoArgs(g_current_stream);
                if(!s) throw PythonError();
                Py_DECREF(s);
            }
            g_device_ready = true;
        }
        return c10::hip::getCurrentHIPStream().stream();
    }
    if(PyLong_Check(o)) return reinterpret_cast<void*>(integer(o));
    PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
    if(!h)
    {
        PyErr_Clear();
        h = PyNumber_Long(o);
        if(!h) throw PythonError();
    }
    const uint64_t v = PyLong_AsUnsignedLongLongMask(h);
    Py_DECREF(h);
    if(PyErr_Occurred()) throw PythonError();
    return reinterpret_cast<void*>(v);
}

template <typename T> T argument(PyObject* const* args, size_t i, bool last)
{
    PyObject* const o        = args[i];
    const bool      repeated = i > 0 && args[i - 1] == o;
    if constexpr(std::is_same<T, size_t*>::value)      // (an array of the host's)
        return o == Py_None ? nullptr : reinterpret_cast<T>(integer(o));
    else if constexpr(std::is_pointer<T>::value)
        return reinterpret_cast<T>(last ? stream_handle(o) : pointer(o));
    else if constexpr(std::is_floating_point<T>::value)
    {
        const double v = PyFloat_AsDouble(o);
        if(v == -1.0 && PyErr_Occurred()) throw PythonError();
        return static_cast<T>(v);
    }
    else if constexpr(std::is_same<T, int>::value)
    {
        if(const at::Tensor* t = repeated ? as_tensor(o) : nullptr) return dtype_code(o, t->scalar_type());
        return repeated && o != Py_None && !PyIndex_Check(o) ? dtype_code(o) : static_cast<int>(integer(o));
    }
    else if constexpr(std::is_same<T, size_t>::value)
    {
        if(repeated && o == Py_None) return 0;
        if(const at::Tensor* t = repeated ? as_tensor(o) : nullptr) return t->nbytes();
        return repeated && !PyIndex_Check(o) ? answer(o, "numel") * answer(o, "element_size") : integer(o);
    }
    else
        return static_cast<T>(integer(o));
}

template <auto F> struct Call;
template <typename... A, int (*F)(A...)> struct Call<F>
{
    static constexpr size_t N = sizeof...(A);
    template <size_t... I> static int run(PyObject* const* args, std::index_sequence<I...>)
    {
        std::tuple<A...> a{argument<A>(args, I, I + 1 == N)...};
        int              rc;
        Py_BEGIN_ALLOW_THREADS
        rc = std::apply(F, a);
        Py_END_ALLOW_THREADS
        return rc;
    }
    static PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n)
    {
        if(n != static_cast<Py_ssize_t>(N))
            return PyErr_Format(PyExc_TypeError, "%zu arguments expected, %zd given", N, n);
        try
        {
            const int rc = run(args, std::make_index_sequence<N>{});
            if(rc == QSYNC_OK) Py_RETURN_NONE;
            PyObject* e = PyObject_CallFunction(g_error, "i", rc);
            if(e) { PyErr_SetObject(reinterpret_cast<PyObject*>(Py_TYPE(e)), e); Py_DECREF(e); }
        }
        catch(const PythonError&) {}
        catch(const std::exception& e) { PyErr_SetString(PyExc_RuntimeError, e.what()); }
        catch(...) { PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception"); }
        return nullptr;
    }
};

PyObject* set_error(PyObject*, PyObject* f)
{
    Py_INCREF(f);
    Py_XSETREF(g_error, f);
    Py_RETURN_NONE;
}

#define ENTRY(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&Call<name>::call)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"set_error", set_error, METH_O, nullptr},
    ENTRY(qsync_absmax_scale), ENTRY(qsync_absmax_scale_static), ENTRY(qsync_quantize), ENTRY(qsync_absmax_quantize),
    ENTRY(qsync_gradient_quantize), ENTRY(qsync_convert_operands), ENTRY(qsync_qlinear_fwd), ENTRY(qsync_qlinear_fwd_amax),
    ENTRY(qsync_qlinear_fwd_codes), ENTRY(qsync_transpose_i8), ENTRY(qsync_scale_from_amax), ENTRY(qsync_qlinear_bwd),
    ENTRY(qsync_qlinear_bwd_rm), ENTRY(qsync_qlinear_backward), ENTRY(qsync_qlinear_bwd_fp16_of_int8), ENTRY(qsync_conv3x3_fwd), ENTRY(qsync_conv3x3_fwd_amax),
    ENTRY(qsync_conv3x3_wgrad), ENTRY(qsync_conv3x3_prepare_weights), ENTRY(qsync_conv3x3_wflip), ENTRY(qsync_im2col3x3_i8),
    ENTRY(qsync_prepare_weights), ENTRY(qsync_dequantize), {nullptr, nullptr, 0, nullptr}};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    PyObject* cuda = PyImport_ImportModule("torch.cuda");
    if(!cuda) return nullptr;
    g_is_initialized = PyObject_GetAttrString(cuda, "is_initialized");
    g_current_stream = PyObject_GetAttrString(cuda, "current_stream");
    Py_DECREF(cuda);
    if(!g_is_initialized || !g_current_stream) return nullptr;
    g_error = reinterpret_cast<PyObject*>(PyExc_RuntimeError);
    Py_INCREF(g_error);
    if(pthread_atfork(nullptr, nullptr, [] { g_device_ready = false; }) != 0) return PyErr_NoMemory();
    return PyModule_Create(&module_def);
}
