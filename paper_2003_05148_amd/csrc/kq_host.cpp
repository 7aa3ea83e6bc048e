// Host side of the Python binding: the argument checks and descriptor arrays of calls that take
// many tensors.  In Python each tensor costs 1 to 2 us of attribute look-ups, so a decoding
// call on 13 layers spent 35 us on the host for 16 us of GPU work.
//
// recon_args(layers): the kq_recon_layer array (include/kq.h) of a list of dicts as
// kq_reconstruct_stack takes them.  Returns (array as bytes, list of W_hat tensors, device index,
// whether any layer asks for its squared error), or None when a layer is anything but the plain
// case (plain contiguous tensors of the right types and shapes on one GPU, the outputs given): the
// caller then goes through its own checks, which convert, allocate or raise.
#define PY_SSIZE_T_CLEAN
#include <torch/csrc/autograd/python_variable.h>

#include <string>
#include <vector>

#include "kq.h"

namespace {

// the item of a dict as a plain GPU tensor: 1 yes, 0 absent or None, -1 anything else
int tensor_item(PyObject* dict, const char* key, c10::ScalarType type, at::Tensor& out) {
    PyObject* const o = PyDict_GetItemString(dict, key);  // borrowed
    if (o == nullptr || o == Py_None) return 0;
    if (!THPVariable_CheckExact(o)) return -1;
    out = THPVariable_Unpack(o);
    return out.is_cuda() && out.scalar_type() == type && out.layout() == c10::kStrided && out.is_contiguous() ? 1 : -1;
}

bool rows9(const at::Tensor& t) { return t.dim() == 2 && t.size(1) == KQ_DIM; }

bool int_item(PyObject* dict, const char* key, bool required, int64_t& v) {
    PyObject* const o = PyDict_GetItemString(dict, key);
    if (o == nullptr) return !required;
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}

// one layer's descriptor and output; false: not the plain case
bool recon_layer(PyObject* d, kq_recon_layer& r, at::Tensor& W, c10::Device& dev, bool first, bool& any_sq) {
    if (!PyDict_CheckExact(d)) return false;
    at::Tensor C, idx, packed, ref, sq;
    int64_t n = 0, bits = 0;
    if (tensor_item(d, "C", at::kFloat, C) != 1 || !rows9(C)) return false;
    if (!int_item(d, "n", true, n) || !int_item(d, "bits", false, bits)) return false;
    if (n < 1 || n > INT32_MAX || bits < 0 || bits > 16 || C.size(0) > INT32_MAX) return false;
    if (first) dev = C.device();
    const int hi = tensor_item(d, "idx", at::kInt, idx);
    if (hi < 0 || (hi == 1 && (idx.dim() != 1 || idx.size(0) != n))) return false;
    if (hi == 0 && tensor_item(d, "packed", at::kByte, packed) != 1) return false;
    if (tensor_item(d, "W_hat", at::kFloat, W) != 1 || !rows9(W) || W.size(0) != n) return false;
    const int hr = tensor_item(d, "W_ref", at::kFloat, ref), hs = tensor_item(d, "sq_error", at::kDouble, sq);
    if (hr < 0 || hs < 0 || (hr == 1 && !rows9(ref))) return false;
    if (C.device() != dev || W.device() != dev) return false;
    r.idx = hi ? (const int32_t*)idx.data_ptr() : nullptr;
    r.packed = hi ? nullptr : (const uint8_t*)packed.data_ptr();
    r.bits = (int32_t)bits;
    r.k = (int32_t)C.size(0);
    r.n = n;
    r.C = (const float*)C.data_ptr();
    r.W_hat = (float*)W.data_ptr();
    r.W_ref = hr ? (const float*)ref.data_ptr() : nullptr;
    r.sq_error = hs ? (double*)sq.data_ptr() : nullptr;
    any_sq |= hs == 1;
    return true;
}

PyObject* recon_args(PyObject*, PyObject* layers) {
    try {
        if (!PyList_CheckExact(layers)) Py_RETURN_NONE;
        const Py_ssize_t m = PyList_GET_SIZE(layers);
        if (m < 1 || m > KQ_MAX_STACK) Py_RETURN_NONE;
        kq_recon_layer arr[KQ_MAX_STACK] = {};
        std::vector<at::Tensor> W((size_t)m);
        c10::Device dev(c10::kCPU);
        bool any_sq = false;
        for (Py_ssize_t q = 0; q < m; ++q)
            if (!recon_layer(PyList_GET_ITEM(layers, q), arr[q], W[(size_t)q], dev, q == 0, any_sq)) Py_RETURN_NONE;
        PyObject* const outs = PyList_New(m);
        if (outs == nullptr) return nullptr;
        for (Py_ssize_t q = 0; q < m; ++q) {
            PyObject* const o = THPVariable_Wrap(W[(size_t)q]);
            if (o == nullptr) {
                Py_DECREF(outs);
                return nullptr;
            }
            PyList_SET_ITEM(outs, q, o);
        }
        return Py_BuildValue("(y#NiO)", (const char*)arr, (Py_ssize_t)(sizeof(kq_recon_layer) * (size_t)m), outs,
                             (int)dev.index(), any_sq ? Py_True : Py_False);
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

PyMethodDef methods[] = {{"recon_args", recon_args, METH_O, "descriptor array of kq_reconstruct_stack, or None"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_kqhost", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__kqhost(void) { return PyModule_Create(&module); }
