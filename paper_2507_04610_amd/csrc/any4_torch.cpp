// The GEMM entry points of binding.py for the ordinary, valid call, in native code.
//
// A decode-size GEMM takes the GPU 5 - 10 us; checking shapes and types, asking for the workspace size,
// allocating the output and calling through ctypes took the host 13 us in Python, so that one call after
// another was bound by the host (1 x 1024 x 1024: 13.2 us a call, 4.7 us of it on the GPU).  gemm() does
// the same checks on the tensors themselves and calls the C ABI.  It only ever says yes: whatever is not a
// plain valid call (a wrong type, shape, device, layout, a combination that does not exist) returns None
// with nothing done, and binding.py goes through its own checks, which name the mistake.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include "any4.h"

namespace {

const at::Tensor* tensor(PyObject* o) {
    return THPVariable_Check(o) ? &THPVariable_Unpack(o) : nullptr;
}
bool plain(const at::Tensor& t, at::ScalarType ty) {
    return t.is_cuda() && t.scalar_type() == ty && t.is_contiguous() && t.layout() == at::kStrided;
}
bool shaped(const at::Tensor& t, int64_t a, int64_t b) { return t.dim() == 2 && t.size(0) == a && t.size(1) == b; }

const uint16_t* u16(const at::Tensor& t) { return static_cast<const uint16_t*>(t.data_ptr()); }

// gemm(x, codes, lut, scale, offset, bits, out, workspace, group, repacked)
//   -> the output tensor; None: not a plain valid call, nothing was done; an int: the runtime refused a launch
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS                                               // out of device memory and the like, as torch raises it
    if (n != 10) Py_RETURN_NONE;
    const at::Tensor *x = tensor(a[0]), *codes = tensor(a[1]), *scale = tensor(a[3]), *offset = tensor(a[4]);
    const bool has_lut = a[2] != Py_None, has_out = a[6] != Py_None, has_ws = a[7] != Py_None;
    const at::Tensor *lut = has_lut ? tensor(a[2]) : nullptr, *out = has_out ? tensor(a[6]) : nullptr,
                     *ws = has_ws ? tensor(a[7]) : nullptr;
    if (!x || !codes || !scale || !offset || (has_lut && !lut) || (has_out && !out) || (has_ws && !ws)) Py_RETURN_NONE;
    if (!PyLong_CheckExact(a[5]) || !PyLong_CheckExact(a[8])) Py_RETURN_NONE;
    const long bits = PyLong_AsLong(a[5]), group = PyLong_AsLong(a[8]);
    if (PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
    const bool repacked = a[9] == Py_True;
    if (x->dim() != 2 || codes->dim() < 1 || scale->dim() != 2) Py_RETURN_NONE;
    const int64_t M = x->size(0), K = x->size(1), N = repacked ? scale->size(0) : codes->size(0);
    const at::ScalarType ty = x->scalar_type();
    const bool f16 = ty == at::kHalf;
    if (!f16 && ty != at::kBFloat16) Py_RETURN_NONE;
    if (bits < 2 || bits > 4 || M < 1 || N < 1 || K < 1 || K % ANY4_GROUP || group < 1 || K % group) Py_RETURN_NONE;
    if (!plain(*x, ty) || !plain(*codes, at::kInt) || !plain(*scale, ty) || !plain(*offset, ty)) Py_RETURN_NONE;
    const int64_t words = K * bits / 32, L = (int64_t)1 << bits;
    if (repacked ? codes->numel() != (N + 15) / 16 * 16 * words : !shaped(*codes, N, words)) Py_RETURN_NONE;
    if (!shaped(*scale, N, K / group) || !shaped(*offset, N, K / group)) Py_RETURN_NONE;
    bool one_table = false;
    if (lut) {
        if (!plain(*lut, ty)) Py_RETURN_NONE;
        one_table = N != 1 && shaped(*lut, 1, L);
        if (!one_table && !shaped(*lut, N, L)) Py_RETURN_NONE;
    }
    if ((f16 || one_table || repacked) && group != ANY4_GROUP) Py_RETURN_NONE;
    if ((f16 && (one_table || repacked)) || (one_table && repacked)) Py_RETURN_NONE;
    if (out && !(plain(*out, ty) && shaped(*out, M, N))) Py_RETURN_NONE;
    // (of any type, but as much memory as it has elements, and on the device)
    if (ws && !(ws->layout() == at::kStrided && ws->device() == x->device() && ws->is_non_overlapping_and_dense())) Py_RETURN_NONE;

    at::Tensor y = out ? *out : at::empty({M, N}, x->options().requires_grad(false));
    at::Tensor scratch;
    void* wp = nullptr;
    size_t wbytes = 0;
    if (ws) {
        wp = ws->data_ptr();
        wbytes = (size_t)ws->numel() * ws->element_size();
    } else if (const size_t need = any4_gemm_workspace_bytes(M, N, K, (int)bits)) {
        scratch = at::empty({(int64_t)need}, x->options().dtype(at::kByte).requires_grad(false));
        wp = scratch.data_ptr();
        wbytes = need;
    }
    void* stream = c10::hip::getCurrentHIPStream().stream();
    const uint16_t *px = u16(*x), *pl = lut ? u16(*lut) : nullptr, *ps = u16(*scale), *po = u16(*offset);
    const uint32_t* pc = static_cast<const uint32_t*>(codes->data_ptr());
    uint16_t* py = static_cast<uint16_t*>(y.data_ptr());
    const int b = (int)bits;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    if (repacked) rc = any4_gemm_repacked(px, pc, pl, ps, po, M, N, K, b, py, wp, wbytes, stream);
    else if (f16) rc = any4_gemm_f16(px, pc, pl, ps, po, M, N, K, b, py, wp, wbytes, stream);
    else if (one_table) rc = any4_gemm_single_table(px, pc, pl, ps, po, M, N, K, b, py, wp, wbytes, stream);
    else if (group == ANY4_GROUP) rc = any4_gemm(px, pc, pl, ps, po, M, N, K, b, py, wp, wbytes, stream);
    else rc = any4_gemm_grouped(px, pc, pl, ps, po, M, N, K, b, (int)group, py, wp, wbytes, stream);
    Py_END_ALLOW_THREADS
    if (rc == ANY4_ERR_HIP) return PyLong_FromLong(rc);
    if (rc != ANY4_OK) Py_RETURN_NONE;                             // refused before any launch: binding.py names the call and the mistake
    if (out) { Py_INCREF(a[6]); return a[6]; }
    return THPVariable_Wrap(std::move(y));
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(gemm)), METH_FASTCALL,
     "gemm(x, codes, lut, scale, offset, bits, out, workspace, group, repacked)"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_any4_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__any4_torch(void) { return PyModule_Create(&module); }
