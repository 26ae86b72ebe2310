// The host side of a call from Python, in C++: what binding.py does around the C functions, for the calls that are made most.
//
// A call of a small layer is five microseconds on the device, and a launch by itself two on the host; checking nine tensors,
// marshalling a dozen pointers, making the output and looking its stream up took six more in Python.  Here they take two (64 -> 64 on
// 1 x 56 x 56, mask given: 8.4 -> 4.6 us of the host's time a call, 8.8 -> 5.6 a call one after another; a prepared pyramid 4.5 -> 3.5).
// Only plain calls are taken: tensors of torch's own class, on the device, contiguous, with nothing that watches tensor
// operations, on the current stream.  Everything else, and every error in the arguments, is left to the Python code, which
// treats them as it always did: `call` returns None for those.
#include <Python.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <hip/hip_runtime_api.h>
#include <pybind11/gil.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include "focused_conv.h"

namespace {

struct Functions {
    decltype(&fc_focused_conv2d) conv2d;
    decltype(&fc_focused_gconv2d) gconv2d;
    decltype(&fc_focused_dwconv2d) dwconv2d;
    decltype(&fc_mask_pyramid) pyramid;
    decltype(&fc_mask_pyramid_packed) pyramid_packed;
    decltype(&fc_out_dims) out_dims;
    decltype(&fc_workspace_bytes) workspace_bytes;
} fn;
PyObject *kept;             // binding's thread-local workspaces
PyObject *dict_name;        // "__dict__"
size_t most_kept;

// A tensor that binding.py would take and that nothing stands in for.
bool plain(PyObject *o)
{
    if (Py_TYPE(o) != reinterpret_cast<PyTypeObject *>(THPVariableClass)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    constexpr c10::DispatchKeySet watched({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                           c10::DispatchKey::Functionalize, c10::DispatchKey::Batched});
    return t.is_cuda() && t.layout() == c10::kStrided && t.unsafeGetTensorImpl()->has_storage() && !t.key_set().has_any(watched) &&
           t.is_contiguous();
}

void *address(PyObject *o) { return o == Py_None ? nullptr : THPVariable_Unpack(o).data_ptr(); }

// The workspace kept for this thread, stream and device if it is large enough, else NULL (a borrowed reference).
PyObject *kept_workspace(size_t need, const at::Tensor &x, void *stream)
{
    if (need > most_kept) return nullptr;
    hipStreamCaptureStatus status;
    if (hipStreamIsCapturing(static_cast<hipStream_t>(stream), &status) != hipSuccess || status != hipStreamCaptureStatusNone) return nullptr;
    PyObject *pool = PyObject_GetAttr(kept, dict_name);
    if (!pool) {
        PyErr_Clear();
        return nullptr;
    }
    PyObject *key = Py_BuildValue("(nn)", reinterpret_cast<Py_ssize_t>(stream), static_cast<Py_ssize_t>(x.device().index()));
    PyObject *ws = key ? PyDict_GetItem(pool, key) : nullptr;
    Py_XDECREF(key);
    Py_DECREF(pool);        // (the thread's dict stays)
    if (!ws || !plain(ws) || static_cast<size_t>(THPVariable_Unpack(ws).numel()) < need) return nullptr;
    return ws;
}

// call(desc, groups, x, w, bias, mask_in, mask_out, idx, count, out, workspace): the output; a status that is an error; or None:
// not a call for this function.  groups: 0 the full layer, -1 the depthwise one.
PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 11 || at::impl::torch_function_mode_enabled() || c10::impl::dispatch_mode_enabled()) Py_RETURN_NONE;
    const long groups = PyLong_AsLong(args[1]);
    if (groups < -1 || groups > INT32_MAX || (groups == -1 && PyErr_Occurred())) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    if (args[2] == Py_None || args[3] == Py_None) Py_RETURN_NONE;
    for (int i = 2; i < 11; ++i)
        if (args[i] != Py_None && !plain(args[i])) Py_RETURN_NONE;
    fc_conv_desc desc;
    Py_buffer view;
    if (PyObject_GetBuffer(args[0], &view, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const bool whole = view.len == sizeof desc;
    if (whole) memcpy(&desc, view.buf, sizeof desc);
    PyBuffer_Release(&view);
    int32_t ho, wo;
    size_t need;
    if (!whole || fn.out_dims(&desc, &ho, &wo) != FC_OK || fn.workspace_bytes(&desc, &need) != FC_OK) Py_RETURN_NONE;

    const at::Tensor &x = THPVariable_Unpack(args[2]);
    void *const stream = c10::hip::getCurrentHIPStream().stream();
    PyObject *scratch_in = args[10];
    if (scratch_in == Py_None && args[5] != Py_None && args[7] == Py_None && groups >= 0) {
        scratch_in = kept_workspace(need, x, stream);
        if (!scratch_in) Py_RETURN_NONE;    // (binding.py makes it, and keeps it where it may)
    }
    // (both are given back whatever the allocation throws; another thread may replace what is kept while the lock is not held)
    THPObjectPtr ws = THPObjectPtr::dup(scratch_in);
    THPObjectPtr out;
    if (args[9] == Py_None) {
        static constexpr c10::ScalarType types[] = {c10::kFloat, c10::kBFloat16, c10::kHalf, c10::ScalarType::Float8_e4m3fn};
        const int64_t shape[] = {desc.n, ho, wo, desc.c_out};
        const auto options = x.options().dtype(types[desc.out_dtype]).requires_grad(false);
        at::Tensor made;
        {
            const pybind11::gil_scoped_release unlocked;    // (an allocation may wait for the device)
            made = at::empty(shape, options);
        }
        out = THPVariable_Wrap(std::move(made));
        if (!out) return nullptr;
    } else {
        out = THPObjectPtr::dup(args[9]);
    }
    const size_t ws_bytes = ws.get() == Py_None ? 0 : THPVariable_Unpack(ws.get()).nbytes();
    const void *const xp = address(args[2]), *const w = address(args[3]);
    const float *const bias = static_cast<float *>(address(args[4]));
    const uint8_t *const mask_in = static_cast<uint8_t *>(address(args[5])), *const mask_out = static_cast<uint8_t *>(address(args[6]));
    const int32_t *const idx = static_cast<int32_t *>(address(args[7])), *const count = static_cast<int32_t *>(address(args[8]));
    void *const to = address(out.get()), *const scratch = address(ws.get());
    int32_t status;
    Py_BEGIN_ALLOW_THREADS
    status = groups < 0    ? fn.dwconv2d(&desc, xp, mask_in, w, bias, to, stream)
             : groups == 0 ? fn.conv2d(&desc, xp, mask_in, w, bias, mask_out, idx, count, to, scratch, ws_bytes, stream)
                           : fn.gconv2d(&desc, static_cast<int32_t>(groups), xp, mask_in, w, bias, mask_out, idx, count, to, scratch, ws_bytes, stream);
    Py_END_ALLOW_THREADS
    if (status == FC_OK) return out.release();
    return PyLong_FromLong(status);
    END_HANDLE_TH_ERRORS
}

// ---- Prepared(kind, arguments): a call whose arguments are numbers already; calling it with a raw stream, or with None for the
// current one, returns the status ----
enum { kConv = 0, kDepthwise = 1, kPyramid = 2, kPyramidPacked = 3 };
constexpr int kMostArgs = 13;
constexpr int kArgs[] = {11, 6, 11, 12};

struct Prepared {
    PyObject_HEAD
    int kind;
    uintptr_t a[kMostArgs];
};

int prepared_init(PyObject *self, PyObject *args, PyObject *)
{
    Prepared *p = reinterpret_cast<Prepared *>(self);
    PyObject *list;
    if (!PyArg_ParseTuple(args, "iO!", &p->kind, &PyTuple_Type, &list)) return -1;
    if (p->kind < 0 || p->kind > kPyramidPacked || PyTuple_GET_SIZE(list) != kArgs[p->kind]) {
        PyErr_SetString(PyExc_ValueError, "not a prepared call");
        return -1;
    }
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(list); ++i) {
        PyObject *v = PyTuple_GET_ITEM(list, i);
        p->a[i] = v == Py_None ? 0 : static_cast<uintptr_t>(PyLong_AsUnsignedLongLong(v));
        if (PyErr_Occurred()) return -1;
    }
    return 0;
}

PyObject *prepared_call(PyObject *self, PyObject *args, PyObject *)
{
    HANDLE_TH_ERRORS
    const Prepared *p = reinterpret_cast<Prepared *>(self);
    PyObject *raw;
    if (!PyArg_UnpackTuple(args, "Prepared", 1, 1, &raw)) return nullptr;
    void *stream;
    if (raw == Py_None) {
        stream = c10::hip::getCurrentHIPStream().stream();
    } else {
        stream = reinterpret_cast<void *>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLong(raw)));
        if (PyErr_Occurred()) return nullptr;
    }
    const uintptr_t *const a = p->a;
    auto i32 = [&](int i) { return static_cast<int32_t>(a[i]); };
    auto at = [&](int i, auto type) { return reinterpret_cast<decltype(type)>(a[i]); };
    const void *const cv = nullptr;
    void *const v = nullptr;
    const uint8_t *const u8 = nullptr;
    const float *const f32 = nullptr;
    const int32_t *const list = nullptr;
    const fc_conv_desc *const desc = nullptr;
    const fc_mask_step *const steps = nullptr;
    uint8_t *const *const masks = nullptr;
    uint64_t *const *const bits = nullptr;
    int32_t *const *const lists = nullptr;
    int32_t status = FC_OK;
    Py_BEGIN_ALLOW_THREADS
    switch (p->kind) {
    case kConv:
        status = fn.conv2d(at(0, desc), at(1, cv), at(2, u8), at(3, cv), at(4, f32), at(5, u8), at(6, list), at(7, list), at(8, v), at(9, v), a[10],
                           stream);
        break;
    case kDepthwise:
        status = fn.dwconv2d(at(0, desc), at(1, cv), at(2, u8), at(3, cv), at(4, f32), at(5, v), stream);
        break;
    case kPyramid:
        status = fn.pyramid(at(0, u8), i32(1), i32(2), i32(3), i32(4), at(5, steps), at(6, masks), at(7, lists), at(8, lists), at(9, v), a[10], stream);
        break;
    case kPyramidPacked:
        status = fn.pyramid_packed(at(0, cv), i32(1), i32(2), i32(3), i32(4), i32(5), at(6, steps), at(7, bits), at(8, lists), at(9, lists),
                                   at(10, v), a[11], stream);
        break;
    }
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
    END_HANDLE_TH_ERRORS
}

PyTypeObject prepared_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// bind(addresses of the C functions, the thread-local workspaces, the largest workspace kept)
PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long a[7], most;
    PyObject *pool;
    if (!PyArg_ParseTuple(args, "(KKKKKKK)OK", &a[0], &a[1], &a[2], &a[3], &a[4], &a[5], &a[6], &pool, &most)) return nullptr;
    fn.conv2d = reinterpret_cast<decltype(fn.conv2d)>(a[0]);
    fn.gconv2d = reinterpret_cast<decltype(fn.gconv2d)>(a[1]);
    fn.dwconv2d = reinterpret_cast<decltype(fn.dwconv2d)>(a[2]);
    fn.pyramid = reinterpret_cast<decltype(fn.pyramid)>(a[3]);
    fn.pyramid_packed = reinterpret_cast<decltype(fn.pyramid_packed)>(a[4]);
    fn.out_dims = reinterpret_cast<decltype(fn.out_dims)>(a[5]);
    fn.workspace_bytes = reinterpret_cast<decltype(fn.workspace_bytes)>(a[6]);
    Py_INCREF(pool);
    Py_XDECREF(kept);
    kept = pool;
    most_kept = most;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call)), METH_FASTCALL, nullptr},
                         {"bind", bind, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__native()
{
    dict_name = PyUnicode_InternFromString("__dict__");
    prepared_type.tp_name = "paper_2207_10741_amd._native.Prepared";
    prepared_type.tp_basicsize = sizeof(Prepared);
    prepared_type.tp_flags = Py_TPFLAGS_DEFAULT;
    prepared_type.tp_new = PyType_GenericNew;
    prepared_type.tp_init = prepared_init;
    prepared_type.tp_call = prepared_call;
    if (!dict_name || PyType_Ready(&prepared_type) < 0) return nullptr;
    PyObject *m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&prepared_type);
    if (PyModule_AddObject(m, "Prepared", reinterpret_cast<PyObject *>(&prepared_type)) < 0) {
        Py_DECREF(&prepared_type);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
