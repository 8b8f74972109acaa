// The calls of the Python binding that launch a kernel, as a CPython extension: the checks on the tensors, their addresses, the current
// stream and the C ABI call.  Host time of a call, in Python with ctypes / here, us (three processes of each, the least of 40 rounds of 300
// calls): run 4.2 / 2.9 (256^3 then takes the 3.9 of its kernel, launch after launch), quantise 4.9 / 3.4 - 3.9, decode (which makes its
// result) 5.8 - 6.0 / 3.7 - 4.3.
// The C ABI is reached through the addresses that the binding hands over, so this file links against torch only.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ops/empty.h>
#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>

#include <cstdint>

namespace {

// What a plan's operands are checked against; the binding fills it in as a ctypes structure of the same layout.
struct RunSpec {
    int (*run)(const void *, const void *, const void *, void *, void *);
    void *plan;
    int64_t a_bytes;
    int64_t b_bytes;           // B as a BFP16 buffer of this many bytes, or 0: bf16 of b_rows x b_cols
    int64_t b_rows, b_cols;
    int64_t c_bytes;           // C likewise
    int64_t c_rows, c_cols;
};

bool is_matrix(const at::Tensor &t, int64_t rows, int64_t cols)
{
    return t.scalar_type() == at::kBFloat16 && t.dim() == 2 && t.size(0) == rows && t.size(1) == cols && t.is_contiguous();
}

bool is_buffer(const at::Tensor &t, int64_t bytes) { return t.scalar_type() == at::kByte && t.numel() == bytes && t.is_contiguous(); }

// Where a kernel can store: C may also be in pinned host memory.
bool on_device_or_pinned(const at::Tensor &t) { return t.is_cuda() || t.is_pinned(); }

PyObject *refuse()
{
    PyErr_SetNone(PyExc_AssertionError);
    return nullptr;
}

// hipStream_t of an int handle, by default of the current device's current stream
bool stream_of(PyObject *arg, void **out)
{
    if (arg == Py_None) {
        *out = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    *out = PyLong_AsVoidPtr(arg);
    return !PyErr_Occurred();
}

bool tensors(PyObject *const *args, int n)
{
    for (int i = 0; i < n; ++i)
        if (!THPVariable_Check(args[i])) {
            PyErr_SetString(PyExc_TypeError, "expected a torch.Tensor");
            return false;
        }
    return true;
}

// The interpreter lock given back for a scope, also where that is left by an exception.
struct WithoutLock {
    PyThreadState *state = PyEval_SaveThread();
    ~WithoutLock() { PyEval_RestoreThread(state); }
};

// run(address of a RunSpec, A, B, C, stream handle or None) -> status
PyObject *run(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 5) return PyErr_Format(PyExc_TypeError, "run takes 5 arguments");
    const RunSpec *s = static_cast<const RunSpec *>(PyLong_AsVoidPtr(args[0]));
    if (PyErr_Occurred() || !tensors(args + 1, 3)) return nullptr;
    HANDLE_TH_ERRORS                       // torch's exceptions keep their Python types (an allocation's torch.OutOfMemoryError)
    const at::Tensor &a = THPVariable_Unpack(args[1]), &b = THPVariable_Unpack(args[2]), &c = THPVariable_Unpack(args[3]);
    if (!a.is_cuda() || !is_buffer(a, s->a_bytes) || !b.is_cuda()) return refuse();
    if (!(s->b_bytes ? is_buffer(b, s->b_bytes) : is_matrix(b, s->b_rows, s->b_cols))) return refuse();
    if (!on_device_or_pinned(c) || !(s->c_bytes ? is_buffer(c, s->c_bytes) : is_matrix(c, s->c_rows, s->c_cols))) return refuse();
    const void *pa = a.data_ptr(), *pb = b.data_ptr();
    void *pc = c.data_ptr(), *stream = nullptr;
    if (!stream_of(args[4], &stream)) return nullptr;
    int st;
    {
        WithoutLock unlocked;
        st = s->run(s->plan, pa, pb, pc, stream);
    }
    return PyLong_FromLong(st);
    END_HANDLE_TH_ERRORS
}

// quantize(address of atb_bfp16_quantize, A, out, bytes of out, stream handle or None) -> status
PyObject *quantize(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    typedef int (*fn)(const float *, int64_t, void *, int64_t, int64_t, void *);
    if (n != 5) return PyErr_Format(PyExc_TypeError, "quantize takes 5 arguments");
    const fn call = reinterpret_cast<fn>(PyLong_AsVoidPtr(args[0]));
    const int64_t bytes = PyLong_AsLongLong(args[3]);
    if (PyErr_Occurred() || !tensors(args + 1, 2)) return nullptr;
    HANDLE_TH_ERRORS
    const at::Tensor &a = THPVariable_Unpack(args[1]), &out = THPVariable_Unpack(args[2]);
    if (!out.is_cuda() || !is_buffer(out, bytes)) return refuse();
    const int64_t rows = a.size(0), cols = a.size(1), lda = a.stride(0);
    const float *pa = static_cast<const float *>(a.data_ptr());
    void *po = out.data_ptr(), *stream = nullptr;
    if (!stream_of(args[4], &stream)) return nullptr;
    int st;
    {
        WithoutLock unlocked;
        st = call(pa, lda, po, rows, cols, stream);
    }
    return PyLong_FromLong(st);
    END_HANDLE_TH_ERRORS
}

// decode(address of atb_bfp16_decode, address of atb_bfp16_bytes, A, rows, columns, stream handle or None) -> the decoded matrix, or the
// status if that is not 0.  A is read as bytes, whatever its type, and may be longer.
PyObject *decode(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    typedef int (*fn)(const void *, void *, int64_t, int64_t, void *);
    if (n != 6) return PyErr_Format(PyExc_TypeError, "decode takes 6 arguments");
    typedef size_t (*size_fn)(int64_t, int64_t);
    const fn call = reinterpret_cast<fn>(PyLong_AsVoidPtr(args[0]));
    const size_fn size = reinterpret_cast<size_fn>(PyLong_AsVoidPtr(args[1]));
    if (PyErr_Occurred()) return nullptr;
    const int64_t rows = PyLong_AsLongLong(args[3]), cols = PyLong_AsLongLong(args[4]);
    if (PyErr_Occurred() || !tensors(args + 2, 1)) return nullptr;
    HANDLE_TH_ERRORS
    const at::Tensor &a = THPVariable_Unpack(args[2]);
    if (!a.is_cuda() || !a.is_contiguous() || a.nbytes() < size(rows, cols)) return refuse();     // (a size of 0: the call below says why)
    at::Tensor out;
    {
        WithoutLock unlocked;              // an allocation may wait for the device
        out = at::empty({rows, cols}, at::TensorOptions().dtype(at::kBFloat16).device(a.device()));
    }
    const void *pa = a.data_ptr();
    void *po = out.data_ptr(), *stream = nullptr;
    if (!stream_of(args[5], &stream)) return nullptr;
    int st;
    {
        WithoutLock unlocked;
        st = call(pa, po, rows, cols, stream);
    }
    return st == 0 ? THPVariable_Wrap(out) : PyLong_FromLong(st);
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {{"run", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(run)), METH_FASTCALL, nullptr},
                         {"quantize", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(quantize)), METH_FASTCALL, nullptr},
                         {"decode", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_launch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__launch() { return PyModule_Create(&module); }
