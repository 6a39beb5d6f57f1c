// The two calls that a program makes at every decode step, cfgzip_decode_step and cfgzip_engine_step, as functions of
// a CPython extension: what the binding does for them in Python (a dozen attribute look-ups and checks of tensors, the
// conversion of as many arguments for ctypes) took 5 us of the 8 that a step on small logits takes, and the kernel 3.
//
// Marshalling only, and only of the plain case: exact torch.Tensor objects in GPU memory of the types and layouts the
// binding asks for, the current stream.  For anything else a function returns None and has done nothing; the binding then
// goes its general way, which also says what is wrong.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <limits>

namespace {

using DecodeStep = int (*)(void *, int32_t, int32_t, int32_t, int64_t, const int32_t *, const int32_t *, int32_t,
                           int32_t *, const int32_t *, const int32_t *, int32_t *, void *);
using EngineStep = int (*)(void *, int32_t, int32_t, int32_t, int64_t, const int32_t *, int32_t, int32_t,
                           const int32_t *, const uint16_t *, const int32_t *, const int32_t *, int32_t *, int32_t *,
                           void *);
DecodeStep g_decode_step = nullptr;
EngineStep g_engine_step = nullptr;

constexpr int64_t kMost = std::numeric_limits<int32_t>::max();

// The tensor in GPU memory that `o` is, nothing else around it, or null.  (A tensor that a transformation wraps has no
// storage.)
const at::Tensor *plain(PyObject *o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage()) return nullptr;
    return &t;
}
const at::Tensor *plain(PyObject *o, at::ScalarType type) {
    const at::Tensor *t = plain(o);
    return t && t->scalar_type() == type && t->is_contiguous() ? t : nullptr;
}
// The same where None stands for "none": false if it is something else.
template <typename T>
bool plain_or_none(PyObject *o, at::ScalarType type, T **out) {
    *out = nullptr;
    if (o == Py_None) return true;
    const at::Tensor *t = plain(o, type);
    if (!t) return false;
    *out = static_cast<T *>(t->data_ptr());
    return true;
}
// An exact int of 1 .. 2^31 - 1, or 0.
int64_t small_int(PyObject *o) {
    if (!PyLong_CheckExact(o)) return 0;
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow || v < 1 || v > kMost ? 0 : v;
}

struct Logits {
    void *data;
    int32_t type, B, V;
    int64_t stride;
};
bool logits_of(PyObject *o, PyObject *V, Logits *out) {
    const at::Tensor *t = plain(o);
    if (!t || t->dim() != 2 || t->stride(1) != 1) return false;
    if (t->scalar_type() == at::kFloat) out->type = 0;
    else if (t->scalar_type() == at::kBFloat16) out->type = 1;
    else return false;
    const int64_t columns = V == Py_None ? t->size(1) : small_int(V);
    if (columns < 1 || columns > kMost || t->size(0) > kMost) return false;
    out->data = t->data_ptr();
    out->B = (int32_t)t->size(0);
    out->V = (int32_t)columns;
    out->stride = t->stride(0);
    return true;
}

// What the call returns, made before the launch, behind which nothing can fail any more: the tensor handed in, or the new
// one around `made`.  Null: a Python error is set.
PyObject *result_of(PyObject *given, const at::Tensor &made) {
    if (given == Py_None) return THPVariable_Wrap(made);
    Py_INCREF(given);
    return given;
}
// The same, or the status of the launch if it is not 0.
PyObject *finish(int rc, PyObject *result) {
    if (rc == 0) return result;
    Py_DECREF(result);
    return PyLong_FromLong(rc);
}
// Nothing has been launched: the general way meets the same error (one that a dispatch mode raises is also set in the
// interpreter) and says so.
PyObject *leave_it() {
    PyErr_Clear();
    Py_RETURN_NONE;
}

// (logits, cls_bits, class_of_token, C, tok, rep_of_class, tok_bits_out, rep_out, V)
PyObject *decode_step(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 9 || !g_decode_step || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    Logits l;
    int32_t C = 0, *tok_bits = nullptr, *rep_out = nullptr;
    const int32_t *bits_p = nullptr, *cls_p = nullptr, *tok_p = nullptr, *rep_p = nullptr;
    void *stream = nullptr;
    PyObject *result = nullptr;
    try {
        if (!logits_of(args[0], args[8], &l)) Py_RETURN_NONE;
        C = (int32_t)small_int(args[3]);
        const at::Tensor *bits = plain(args[1], at::kInt), *cls = plain(args[2], at::kInt),
                         *tok = plain(args[4], at::kInt), *rep = plain(args[5], at::kInt);
        if (!C || !bits || !cls || !tok || !rep || !plain_or_none(args[6], at::kInt, &tok_bits) ||
            !plain_or_none(args[7], at::kInt, &rep_out))
            Py_RETURN_NONE;
        if (bits->dim() != 2 || bits->size(0) != l.B || bits->size(1) != ((int64_t)C + 31) / 32 || tok->numel() != l.B ||
            rep->numel() != C || cls->numel() != l.V)
            Py_RETURN_NONE;
        at::Tensor made;
        if (args[7] == Py_None) {
            made = tok->dim() == 1 ? at::empty_like(*tok) : at::empty({l.B}, tok->options());
            rep_out = static_cast<int32_t *>(made.data_ptr());
        }
        bits_p = static_cast<const int32_t *>(bits->data_ptr());
        cls_p = static_cast<const int32_t *>(cls->data_ptr());
        tok_p = static_cast<const int32_t *>(tok->data_ptr());
        rep_p = static_cast<const int32_t *>(rep->data_ptr());
        stream = c10::hip::getCurrentHIPStream().stream();
        result = result_of(args[7], made);
    } catch (...) {
    }
    if (!result) return leave_it();
    int rc = 0;
    Py_BEGIN_ALLOW_THREADS
    rc = g_decode_step(l.data, l.type, l.B, l.V, l.stride, bits_p, cls_p, C, tok_bits, tok_p, rep_p, rep_out, stream);
    Py_END_ALLOW_THREADS
    return finish(rc, result);
}

// (logits, state_mask, C, class_of_token, sig_rep, tok_prev, states_in, states_out, tok_bits_out, V)
PyObject *engine_step(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 10 || !g_engine_step || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    Logits l;
    int32_t S = 0, C = 0, *tok_prev = nullptr, *out = nullptr, *tok_bits = nullptr;
    uint16_t *sig_rep = nullptr;
    const int32_t *mask_p = nullptr, *cls_p = nullptr, *in_p = nullptr;
    void *stream = nullptr;
    PyObject *result = nullptr;
    try {
        if (!logits_of(args[0], args[9], &l)) Py_RETURN_NONE;
        C = (int32_t)small_int(args[2]);
        const at::Tensor *mask = plain(args[1], at::kInt), *cls = plain(args[3], at::kInt), *in = plain(args[6], at::kInt);
        if (!C || !mask || mask->dim() < 1 || mask->size(0) > kMost || !cls || !in ||
            !plain_or_none(args[4], at::kUInt16, &sig_rep) || !plain_or_none(args[5], at::kInt, &tok_prev) ||
            !plain_or_none(args[7], at::kInt, &out) || !plain_or_none(args[8], at::kInt, &tok_bits))
            Py_RETURN_NONE;
        at::Tensor made;
        if (args[7] == Py_None) {
            made = at::empty_like(*in);
            out = static_cast<int32_t *>(made.data_ptr());
        }
        mask_p = static_cast<const int32_t *>(mask->data_ptr());
        cls_p = static_cast<const int32_t *>(cls->data_ptr());
        in_p = static_cast<const int32_t *>(in->data_ptr());
        S = (int32_t)mask->size(0);
        stream = c10::hip::getCurrentHIPStream().stream();
        result = result_of(args[7], made);
    } catch (...) {
    }
    if (!result) return leave_it();
    int rc = 0;
    Py_BEGIN_ALLOW_THREADS
    rc = g_engine_step(l.data, l.type, l.B, l.V, l.stride, mask_p, S, C, cls_p, sig_rep, tok_prev, in_p, out, tok_bits, stream);
    Py_END_ALLOW_THREADS
    return finish(rc, result);
}

// (address of cfgzip_decode_step, address of cfgzip_engine_step), of the library that the binding has loaded
PyObject *connect(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "connect takes two addresses");
        return nullptr;
    }
    void *decode = PyLong_AsVoidPtr(args[0]), *engine = PyLong_AsVoidPtr(args[1]);
    if (PyErr_Occurred()) return nullptr;
    g_decode_step = reinterpret_cast<DecodeStep>(decode);
    g_engine_step = reinterpret_cast<EngineStep>(engine);
    Py_RETURN_NONE;
}

template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyCFunction fast() {
    return reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(F));
}
PyMethodDef g_methods[] = {{"decode_step", fast<decode_step>(), METH_FASTCALL, nullptr},
                           {"engine_step", fast<engine_step>(), METH_FASTCALL, nullptr},
                           {"connect", fast<connect>(), METH_FASTCALL, nullptr},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "cfgzip_stepcall", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

#define TEXT_OF(x) #x
#define TEXT(x) TEXT_OF(x)
// What this was built for, which the binding compares with what it runs in: torch's C++ layouts are those of one version.
PyMODINIT_FUNC PyInit_cfgzip_stepcall() {
    PyObject *m = PyModule_Create(&g_module);
    if (m && (PyModule_AddStringConstant(m, "python", TEXT(PY_MAJOR_VERSION) "." TEXT(PY_MINOR_VERSION)) < 0 ||
              PyModule_AddStringConstant(m, "torch", BUILT_FOR_TORCH) < 0)) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
