// ckpt_py.cpp -- CPython module _ckpt_py: the argument marshalling of
// ckpt_pack_noalloc for lists of torch tensors.  A call of 64 fragments spent
// 25 us of its 41 reading the tensors' attributes one Python call at a time.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <vector>

#include "../../include/ckpt.h"

namespace {

using PackFn = ckpt_status (*)(const ckpt_tensor*, uint32_t, uint64_t, uint32_t, int32_t, void*, uint64_t, uint64_t*,
                               uint64_t, void*, uint64_t*, uint64_t*);

// Read one tensor's address and bytes.  False for whatever the Python path
// answers better: other types and subclasses (their attributes may be
// overridden), tensors without plain storage, and those it refuses.
bool read(PyObject* o, bool contiguous, void** ptr, uint64_t* nbytes)
{
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || (contiguous && !t.is_contiguous())) return false;
    *nbytes = (uint64_t)t.numel() * t.element_size();
    *ptr = t.data_ptr();
    return true;
}

// pack_noalloc(function address, tensors, image, sums, chunk_bytes,
// align_bytes, device, stream handle) -> (status, image bytes, chunks), or
// None when an argument needs the Python path.
PyObject* pack_noalloc(PyObject*, PyObject* const* args, Py_ssize_t n_args)
{
    if (n_args != 8) {
        PyErr_SetString(PyExc_TypeError, "pack_noalloc takes 8 arguments");
        return nullptr;
    }
    if (!PyList_CheckExact(args[1]) && !PyTuple_CheckExact(args[1])) Py_RETURN_NONE;
    const unsigned long long fn = PyLong_AsUnsignedLongLong(args[0]), chunk = PyLong_AsUnsignedLongLong(args[4]);
    const unsigned long long align = PyLong_AsUnsignedLongLong(args[5]), stream = PyLong_AsUnsignedLongLong(args[7]);
    const long device = PyLong_AsLong(args[6]);
    if (PyErr_Occurred() || align > UINT32_MAX || device < INT32_MIN || device > INT32_MAX) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(args[1]);
    PyObject* const* items = PySequence_Fast_ITEMS(args[1]);
    uint64_t image_cap = 0, sums_cap = 0, image_bytes = 0, n_chunks = 0;
    void *image = nullptr, *sums = nullptr;
    std::vector<ckpt_tensor> t;
    if (n == 0 || (uint64_t)n > UINT32_MAX) Py_RETURN_NONE;
    try {
        t.resize((size_t)n);
        for (Py_ssize_t k = 0; k < n; ++k) {
            void* p = nullptr;
            if (!read(items[k], true, &p, &t[k].nbytes)) Py_RETURN_NONE;
            t[k].dev_ptr = t[k].nbytes ? p : nullptr;
            t[k].dtype = t[k].cls = 0;
        }
        if (!read(args[2], false, &image, &image_cap) || !read(args[3], false, &sums, &sums_cap)) Py_RETURN_NONE;
    } catch (...) { // no storage behind the tensor, out of memory: the Python path raises its own error
        Py_RETURN_NONE;
    }
    ckpt_status rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = ((PackFn)(uintptr_t)fn)(t.data(), (uint32_t)n, chunk, (uint32_t)align, (int32_t)device, image, image_cap,
                                 (uint64_t*)sums, sums_cap / 8, (void*)(uintptr_t)stream, &image_bytes, &n_chunks);
    Py_END_ALLOW_THREADS;
    return Py_BuildValue("iKK", (int)rc, (unsigned long long)image_bytes, (unsigned long long)n_chunks);
}

PyMethodDef methods[] = {{"pack_noalloc", (PyCFunction)(void (*)(void))pack_noalloc, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ckpt_py", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

// torch_version: what it was compiled against; another torch lays tensors out
// differently.
PyMODINIT_FUNC PyInit__ckpt_py()
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) != 0) Py_CLEAR(m);
    return m;
}
