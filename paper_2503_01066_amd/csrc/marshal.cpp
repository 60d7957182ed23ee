// alch_capture_pack for Python: reads its tensors, makes the three small outputs and calls the library, in one call from Python.
// A short prompt's capture is 4 us on the GPU; from Python, seven attributes of each of its 14 tensors, three allocations and a
// ctypes call of eleven arguments took twice as long (one prompt of 317 tokens, six streams: 10.9 us a pass, with this 7.0).
#include <Python.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>

#include "alch.h"

namespace {

typedef int (*PackFn)(const alch_batch*, const uint8_t*, int32_t, const alch_stream*, int64_t, int32_t*, int32_t*, int32_t*, void*, size_t,
                      void*);
constexpr Py_ssize_t kMost = 64;  // streams of a call that this takes

// A plain tensor in device memory, as strided storage; null: something else, which is the caller's own business.
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.layout() == at::kStrided && t.is_cuda() && !t.is_quantized() ? &t : nullptr;
}

// (function, batch, mask, streams, dsts, capacity, sequences, workspace, stream) -> (status, kept_index, cu_kept, n_kept_and_status),
// or None for arguments that it leaves to the caller: other kinds of sequences and tensors, and whatever an error is due for.
PyObject* capture_pack(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TORCH_CHECK_TYPE(n == 9, "capture_pack takes nine arguments");
    const at::Tensor *mask = plain(a[2]), *ws = plain(a[7]);
    const bool lists = (PyList_CheckExact(a[3]) || PyTuple_CheckExact(a[3])) && (PyList_CheckExact(a[4]) || PyTuple_CheckExact(a[4]));
    const Py_ssize_t count = lists ? PySequence_Fast_GET_SIZE(a[3]) : 0;
    if (!mask || !ws || !lists || count > kMost || PySequence_Fast_GET_SIZE(a[4]) < count) Py_RETURN_NONE;
    alch_stream words[kMost];
    for (Py_ssize_t k = 0; k < count; ++k) {
        const at::Tensor *s = plain(PySequence_Fast_GET_ITEM(a[3], k)), *d = plain(PySequence_Fast_GET_ITEM(a[4], k));
        if (!s || !d || s->dim() != 2 || s->numel() == 0 || s->stride(1) != 1 || s->stride(0) < 0 || !d->is_contiguous()) Py_RETURN_NONE;
        const size_t size = s->element_size();
        words[k] = alch_stream{s->data_ptr(), d->data_ptr(), (size_t)s->size(1) * size, (size_t)s->stride(0) * size};
    }
    const PackFn fn = reinterpret_cast<PackFn>(PyLong_AsVoidPtr(a[0]));
    const alch_batch* batch = static_cast<const alch_batch*>(PyLong_AsVoidPtr(a[1]));
    const long long capacity = PyLong_AsLongLong(a[5]), n_seqs = PyLong_AsLongLong(a[6]);
    void* stream = PyLong_AsVoidPtr(a[8]);
    if (PyErr_Occurred()) return nullptr;
    const at::TensorOptions ints = at::TensorOptions().dtype(at::kInt).device(mask->device());
    const at::Tensor kept = at::empty({capacity > 1 ? capacity : 1}, ints), cu = at::empty({n_seqs + 1}, ints), status = at::empty({2}, ints);
    const void* m = mask->data_ptr();
    void *p[4] = {kept.data_ptr(), cu.data_ptr(), status.data_ptr(), ws->data_ptr()};
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(batch, static_cast<const uint8_t*>(m), (int32_t)count, words, capacity, static_cast<int32_t*>(p[0]), static_cast<int32_t*>(p[1]),
            static_cast<int32_t*>(p[2]), p[3], (size_t)ws->numel(), stream);
    Py_END_ALLOW_THREADS
    PyObject* out = PyTuple_New(4);
    if (!out) return nullptr;
    PyTuple_SET_ITEM(out, 0, PyLong_FromLong(rc));
    PyTuple_SET_ITEM(out, 1, THPVariable_Wrap(kept));
    PyTuple_SET_ITEM(out, 2, THPVariable_Wrap(cu));
    PyTuple_SET_ITEM(out, 3, THPVariable_Wrap(status));
    return out;
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {{"capture_pack", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(capture_pack)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// The layout of at::Tensor is compiled in, and another torch may export the same names: the binding compares torch_build with its own.
PyMODINIT_FUNC PyInit__marshal(void) {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_build", ALCH_TORCH_BUILD) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
