// Forward calls of api.py without Python's part of the argument marshalling (CPython extension _flashrnn_binding).
//
// A call of one time step takes the GPU 4 us; checking four tensors and filling in a descriptor from Python took the host 7.
// Here the same checks run on the tensors' C++ side.  A call that is anything but plain -- an argument of another type, a shape that does not fit, a
// buffer left out -- is handed back (kNotHandled) and goes the way through Python, which allocates, converts or raises.
// Nothing is kept from one call for the next but the library's entry points.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "flashrnn.h"

namespace {

constexpr long kNotHandled = 1;   // (status codes are zero or negative)

decltype(&flashrnn_fwd) p_fwd = nullptr;
decltype(&flashrnn_fwd_static_scratch) p_fwd_static = nullptr;
decltype(&flashrnn_num_states) p_num_states = nullptr;
decltype(&flashrnn_num_gates) p_num_gates = nullptr;

// bind(flashrnn_fwd, flashrnn_fwd_static_scratch, flashrnn_num_states, flashrnn_num_gates): addresses in the loaded library
PyObject* bind(PyObject*, PyObject* args) {
    unsigned long long a, b, c, d;
    if (!PyArg_ParseTuple(args, "KKKK", &a, &b, &c, &d)) return nullptr;
    p_fwd = (decltype(p_fwd))a;
    p_fwd_static = (decltype(p_fwd_static))b;
    p_num_states = (decltype(p_num_states))c;
    p_num_gates = (decltype(p_num_gates))d;
    Py_RETURN_NONE;
}

// a tensor proper (no subclass but Parameter, no wrapper of a transformation, memory of its own) on the GPU
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || !t.has_storage() || !t.is_contiguous()) return nullptr;
    const c10::DispatchKeySet ks = t.key_set();
    if (ks.has_any(c10::DispatchKeySet({c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize, c10::DispatchKey::Python})))
        return nullptr;
    return &t;
}
const at::Tensor* plain(PyObject* o, at::ScalarType dtype, std::initializer_list<int64_t> shape) {
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == dtype && t->sizes() == at::IntArrayRef(shape) ? t : nullptr;
}

// fwd(cell, Wx, R, b, states0 | None, save, workspace | None, states, gate_cache | None): workspace None = static scratch; the current stream
PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    auto handed_back = [] { return PyLong_FromLong(kNotHandled); };
    if (n != 9 || !p_fwd || !PyLong_CheckExact(a[0]) || !PyBool_Check(a[5])) return handed_back();
    long rc = kNotHandled;
    try {
        const long cell = PyLong_AsLong(a[0]);
        if (cell < 0 || cell > 1024) return PyErr_Clear(), handed_back();
        const int S = p_num_states((int)cell), G = p_num_gates((int)cell);
        const at::Tensor* Wx = plain(a[1]);
        if (S <= 0 || !Wx || Wx->dim() != 5) return handed_back();
        const at::ScalarType dt = Wx->scalar_type();
        if (dt != at::kBFloat16 && dt != at::kFloat) return handed_back();
        const int64_t T = Wx->size(0), B = Wx->size(1), NH = Wx->size(3), D = Wx->size(4);
        if (Wx->size(2) != G || T >= INT32_MAX || B >= INT32_MAX || NH >= INT32_MAX || D >= INT32_MAX) return handed_back();
        const at::Tensor *R = plain(a[2], dt, {NH, D, G, D}), *b = plain(a[3], dt, {NH, G, D});
        const at::Tensor* s0 = a[4] == Py_None ? nullptr : plain(a[4], at::kFloat, {S, B, NH, D});
        const at::Tensor* states = plain(a[7], at::kFloat, {T + 1, S, B, NH, D});
        const bool save = a[5] == Py_True;
        const at::Tensor *cache = save ? plain(a[8]) : nullptr, *ws = a[6] == Py_None ? nullptr : plain(a[6]);
        if (!R || !b || !states || (a[4] != Py_None && !s0) || (save && !cache) || (a[6] != Py_None && !ws)) return handed_back();
        flashrnn_desc_t d;
        d.cell = (int)cell; d.T = (int)T; d.B = (int)B; d.NH = (int)NH; d.D = (int)D;
        d.io_dtype = dt == at::kBFloat16 ? FLASHRNN_BF16 : FLASHRNN_F32;
        d.recurrent_grad_clip = 0.0f;
        void* stream = c10::hip::getCurrentHIPStream().stream();
        void* s0p = s0 ? s0->data_ptr() : nullptr;
        void* cp = cache ? cache->data_ptr() : nullptr;
        void *wxp = Wx->data_ptr(), *rp = R->data_ptr(), *bp = b->data_ptr(), *sp = states->data_ptr(), *wp = ws ? ws->data_ptr() : nullptr;
        Py_BEGIN_ALLOW_THREADS
        rc = ws ? p_fwd(&d, wxp, rp, bp, s0p, sp, cp, wp, stream) : p_fwd_static(&d, wxp, rp, bp, s0p, sp, cp, stream);
        Py_END_ALLOW_THREADS
    } catch (...) {   // (ahead of the call only: the library throws nothing)
        return handed_back();
    }
    return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr}, {"fwd", (PyCFunction)(void (*)(void))fwd, METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_flashrnn_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the Python and the torch whose headers this was compiled with.  The loader binds no other: a layout may change while every symbol still resolves.
PyMODINIT_FUNC PyInit__flashrnn_binding() {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", FLASHRNN_BUILT_FOR) < 0) Py_CLEAR(m);
    return m;
}
