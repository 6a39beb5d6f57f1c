// The calls that a program makes at every decode step, cfgzip_decode_step and cfgzip_engine_step, and those of the
// pre-computation as functions of a CPython extension: what the binding does for them in Python (a dozen attribute look-ups
// and checks of tensors, the conversion of as many arguments for ctypes) took 5 us of the 8 that a step on small logits
// takes, and the kernel 3; and of the 44 us of signatures and classes of 4,096 tokens, 157 of displacements and classes of
// 32,000 and 165 of relations and classes of 32,000 it took 5, 6 and 4, as the GPU has nothing to do before the first launch.
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
using Signatures = int (*)(const uint8_t *, const int64_t *, int32_t, const uint16_t *, int32_t, uint16_t *, uint64_t *,
                           uint64_t, void *, size_t, void *);
using BuildClasses = int (*)(const uint8_t *, const int64_t *, int32_t, const uint16_t *, int32_t, const uint16_t *,
                             const uint64_t *, void *, int32_t *, int32_t *, int32_t *, int32_t *, int32_t *, void *,
                             size_t, void *);
using Displacements = int (*)(const uint8_t *, const int64_t *, int32_t, const uint16_t *, const uint8_t *, const int32_t *,
                              const uint16_t *, int32_t, int32_t, int32_t, uint16_t *, int32_t, uint64_t *, int32_t *,
                              uint64_t, void *, size_t, void *);
using NfaSignatures = int (*)(const uint8_t *, const int64_t *, int32_t, const int32_t *, int32_t, int32_t *, uint64_t *,
                              uint64_t, void *);
DecodeStep g_decode_step = nullptr;
EngineStep g_engine_step = nullptr;
Signatures g_signatures = nullptr;
BuildClasses g_build_classes = nullptr;
Displacements g_displacements = nullptr;
NfaSignatures g_nfa_signatures = nullptr;

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

// A vocabulary as every call of the pre-computation takes it.
struct Vocabulary {
    const uint8_t *bytes;  // null where every token is empty
    const int64_t *off;
    int32_t V;
    const at::Tensor *off_tensor;
};
bool vocabulary_of(PyObject *bytes, PyObject *off, Vocabulary *out) {
    const at::Tensor *b = plain(bytes, at::kByte), *o = plain(off, at::kLong);
    if (!b || !o || o->numel() < 2 || o->numel() - 1 > kMost) return false;
    out->bytes = b->numel() ? static_cast<const uint8_t *>(b->data_ptr()) : nullptr;
    out->off = static_cast<const int64_t *>(o->data_ptr());
    out->V = (int32_t)(o->numel() - 1);
    out->off_tensor = o;
    return true;
}
bool seed_of(PyObject *o, uint64_t *out) {
    if (!PyLong_CheckExact(o)) return false;
    *out = PyLong_AsUnsignedLongLongMask(o);
    return !PyErr_Occurred();
}
bool bool_of(PyObject *o, bool *out) {
    *out = o == Py_True;
    return o == Py_True || o == Py_False;
}
at::Tensor new_tensor(at::IntArrayRef sizes, at::ScalarType type, const Vocabulary &v) {
    return at::empty(sizes, v.off_tensor->options().dtype(type));
}
// The tensor that a result is: the one handed in, else a new one.  False: not a plain one.
template <typename T>
bool result_in(PyObject *given, at::IntArrayRef sizes, at::ScalarType type, const Vocabulary &v, at::Tensor *made, T **data) {
    if (!plain_or_none(given, type, data)) return false;
    if (given == Py_None) {
        *made = new_tensor(sizes, type, v);
        *data = static_cast<T *>(made->data_ptr());
    }
    return true;
}
// References that are given up unless they are handed on.
struct Held {
    PyObject *o = nullptr;
    explicit Held(PyObject *x) : o(x) {}
    Held(const Held &) = delete;
    Held &operator=(const Held &) = delete;
    ~Held() { Py_XDECREF(o); }
};

// (tok_bytes, tok_off, table, want_sig, want_hash, hash_seed, sig_out, hash_out, workspace)
PyObject *signatures(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 9 || !g_signatures || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    Vocabulary v;
    bool want_sig = false, want_hash = false;
    uint64_t seed = 0, *hash = nullptr;
    uint16_t *sig = nullptr;
    const uint16_t *table_p = nullptr;
    void *ws = nullptr, *stream = nullptr;
    int64_t S = 0, ws_bytes = 0;
    PyObject *result = nullptr;
    try {
        const at::Tensor *table = plain(args[2], at::kUInt16), *workspace = plain(args[8]);
        if (!vocabulary_of(args[0], args[1], &v) || !table || table->dim() < 1 || table->size(0) < 1 || table->size(0) > kMost ||
            !bool_of(args[3], &want_sig) || !bool_of(args[4], &want_hash) || !seed_of(args[5], &seed) || !workspace)
            return leave_it();
        S = table->size(0);
        at::Tensor made_sig, made_hash;
        if (want_sig ? !result_in(args[6], {v.V, S}, at::kUInt16, v, &made_sig, &sig) : !plain_or_none(args[6], at::kUInt16, &sig))
            Py_RETURN_NONE;
        if (want_hash ? !result_in(args[7], {v.V}, at::kLong, v, &made_hash, &hash) : !plain_or_none(args[7], at::kLong, &hash))
            Py_RETURN_NONE;
        table_p = static_cast<const uint16_t *>(table->data_ptr());
        ws = workspace->data_ptr();
        ws_bytes = workspace->numel();
        stream = c10::hip::getCurrentHIPStream().stream();
        const Held a(made_sig.defined() ? THPVariable_Wrap(made_sig) : Py_NewRef(args[6]));
        const Held b(made_hash.defined() ? THPVariable_Wrap(made_hash) : Py_NewRef(args[7]));
        if (a.o && b.o) result = PyTuple_Pack(2, a.o, b.o);
    } catch (...) {
    }
    if (!result) return leave_it();
    int rc = 0;
    Py_BEGIN_ALLOW_THREADS
    rc = g_signatures(v.bytes, v.off, v.V, table_p, (int32_t)S, sig, hash, seed, ws, (size_t)ws_bytes, stream);
    Py_END_ALLOW_THREADS
    return finish(rc, result);
}

// (tok_bytes, tok_off, table, sig, hash, class_of_token, rep_of_class, workspace, signatures_workspace): a tuple of the
// first two results, whole, and the two counts
PyObject *build_classes(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 9 || !g_build_classes || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    Vocabulary v;
    uint16_t *table = nullptr, *sig = nullptr;
    uint8_t *sig_ws = nullptr;
    int32_t *cls = nullptr, *rep = nullptr;
    const uint64_t *hash = nullptr;
    void *ws = nullptr, *stream = nullptr;
    int64_t S = 0, ws_bytes = 0;
    PyObject *first = nullptr, *second = nullptr;
    try {
        const at::Tensor *h = plain(args[4], at::kLong), *workspace = plain(args[7]);
        if (!vocabulary_of(args[0], args[1], &v) || !plain_or_none(args[2], at::kUInt16, &table) ||
            !plain_or_none(args[3], at::kUInt16, &sig) || !h || !workspace || !plain_or_none(args[8], at::kByte, &sig_ws))
            Py_RETURN_NONE;
        if (args[2] != Py_None) {
            const at::Tensor &t = THPVariable_Unpack(args[2]);
            S = t.dim() >= 1 ? t.size(0) : 0;
        } else if (args[3] != Py_None) {
            const at::Tensor &t = THPVariable_Unpack(args[3]);
            S = t.dim() >= 2 ? t.size(1) : 0;
        }
        if (S < 1 || S > kMost) Py_RETURN_NONE;
        at::Tensor made_cls, made_rep;
        if (!result_in(args[5], {v.V}, at::kInt, v, &made_cls, &cls) || !result_in(args[6], {v.V}, at::kInt, v, &made_rep, &rep))
            Py_RETURN_NONE;
        hash = static_cast<const uint64_t *>(h->data_ptr());
        ws = workspace->data_ptr();
        ws_bytes = workspace->numel();
        stream = c10::hip::getCurrentHIPStream().stream();
        first = made_cls.defined() ? THPVariable_Wrap(made_cls) : Py_NewRef(args[5]);
        second = made_rep.defined() ? THPVariable_Wrap(made_rep) : Py_NewRef(args[6]);
    } catch (...) {
    }
    if (!first || !second) {
        Py_XDECREF(first);
        Py_XDECREF(second);
        return leave_it();
    }
    int rc = 0;
    int32_t C = 0, collisions = 0;
    Py_BEGIN_ALLOW_THREADS
    rc = g_build_classes(v.bytes, v.off, v.V, table, (int32_t)S, sig, hash, sig_ws, cls, rep, nullptr, &C, &collisions, ws,
                         (size_t)ws_bytes, stream);
    Py_END_ALLOW_THREADS
    if (rc != 0) {
        Py_DECREF(first);
        Py_DECREF(second);
        return PyLong_FromLong(rc);
    }
    return Py_BuildValue("(NNii)", first, second, (int)C, (int)collisions);
}

// (tok_bytes, tok_off, prod_head, prod_byte, prod_body_off, prod_body, N, row_len, hash_seed, workspace)
PyObject *displacements(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 10 || !g_displacements || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    Vocabulary v;
    uint64_t seed = 0, *hash = nullptr;
    const uint16_t *head_p = nullptr, *body_p = nullptr;
    const uint8_t *byte_p = nullptr;
    const int32_t *off_p = nullptr;
    uint16_t *rows = nullptr;
    int32_t *status = nullptr;
    void *ws = nullptr, *stream = nullptr;
    int64_t P = 0, total = 0, N = 0, row_len = 0, ws_bytes = 0;
    PyObject *result = nullptr;
    try {
        const at::Tensor *head = plain(args[2], at::kUInt16), *byte = plain(args[3], at::kByte), *off = plain(args[4], at::kInt),
                         *body = plain(args[5], at::kUInt16), *workspace = plain(args[9]);
        N = small_int(args[6]);
        row_len = small_int(args[7]);
        if (!vocabulary_of(args[0], args[1], &v) || !head || !byte || !off || !body || !workspace || !N || !row_len ||
            !seed_of(args[8], &seed) || head->numel() < 1 || head->numel() >= kMost || off->numel() != head->numel() + 1 ||
            body->numel() > kMost)
            return leave_it();
        P = head->numel();
        total = body->numel();
        const at::Tensor made_rows = new_tensor({v.V, row_len}, at::kUInt16, v), made_hash = new_tensor({v.V}, at::kLong, v),
                         made_status = new_tensor({v.V}, at::kInt, v);
        rows = static_cast<uint16_t *>(made_rows.data_ptr());
        hash = static_cast<uint64_t *>(made_hash.data_ptr());
        status = static_cast<int32_t *>(made_status.data_ptr());
        head_p = static_cast<const uint16_t *>(head->data_ptr());
        byte_p = static_cast<const uint8_t *>(byte->data_ptr());
        off_p = static_cast<const int32_t *>(off->data_ptr());
        body_p = total ? static_cast<const uint16_t *>(body->data_ptr()) : nullptr;
        ws = workspace->data_ptr();
        ws_bytes = workspace->numel();
        stream = c10::hip::getCurrentHIPStream().stream();
        const Held a(THPVariable_Wrap(made_rows)), b(THPVariable_Wrap(made_hash)), c(THPVariable_Wrap(made_status));
        if (a.o && b.o && c.o) result = PyTuple_Pack(3, a.o, b.o, c.o);
    } catch (...) {
    }
    if (!result) return leave_it();
    int rc = 0;
    Py_BEGIN_ALLOW_THREADS
    rc = g_displacements(v.bytes, v.off, v.V, head_p, byte_p, off_p, body_p, (int32_t)total, (int32_t)P, (int32_t)N, rows,
                         (int32_t)row_len, hash, status, seed, ws, (size_t)ws_bytes, stream);
    Py_END_ALLOW_THREADS
    return finish(rc, result);
}

// (tok_bytes, tok_off, nfa, want_hash, hash_seed)
PyObject *nfa_signatures(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 5 || !g_nfa_signatures || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    Vocabulary v;
    bool want_hash = false;
    uint64_t seed = 0, *hash = nullptr;
    const int32_t *nfa_p = nullptr;
    int32_t *rel = nullptr;
    void *stream = nullptr;
    int64_t S = 0;
    PyObject *result = nullptr;
    try {
        const at::Tensor *nfa = plain(args[2], at::kInt);
        if (!vocabulary_of(args[0], args[1], &v) || !nfa || nfa->dim() != 3 || nfa->size(0) != 256 || nfa->size(1) < 1 ||
            nfa->size(1) > kMost - 31 || nfa->size(2) != (nfa->size(1) + 31) / 32 || !bool_of(args[3], &want_hash) ||
            !seed_of(args[4], &seed))
            return leave_it();
        S = nfa->size(1);
        const at::Tensor made_rel = new_tensor({v.V, S, nfa->size(2)}, at::kInt, v);
        const at::Tensor made_hash = want_hash ? new_tensor({v.V}, at::kLong, v) : at::Tensor();
        rel = static_cast<int32_t *>(made_rel.data_ptr());
        if (want_hash) hash = static_cast<uint64_t *>(made_hash.data_ptr());
        nfa_p = static_cast<const int32_t *>(nfa->data_ptr());
        stream = c10::hip::getCurrentHIPStream().stream();
        const Held a(THPVariable_Wrap(made_rel)), b(want_hash ? THPVariable_Wrap(made_hash) : Py_NewRef(Py_None));
        if (a.o && b.o) result = PyTuple_Pack(2, a.o, b.o);
    } catch (...) {
    }
    if (!result) return leave_it();
    int rc = 0;
    Py_BEGIN_ALLOW_THREADS
    rc = g_nfa_signatures(v.bytes, v.off, v.V, nfa_p, (int32_t)S, rel, hash, seed, stream);
    Py_END_ALLOW_THREADS
    return finish(rc, result);
}

// The addresses of cfgzip_decode_step, cfgzip_engine_step, cfgzip_signatures, cfgzip_build_classes, cfgzip_displacements and
// cfgzip_nfa_signatures, of the library that the binding has loaded
PyObject *connect(PyObject *, PyObject *const *args, Py_ssize_t n) {
    void *at[6];
    if (n != 6) {
        PyErr_SetString(PyExc_TypeError, "connect takes six addresses");
        return nullptr;
    }
    for (int i = 0; i < 6; ++i) at[i] = PyLong_AsVoidPtr(args[i]);
    if (PyErr_Occurred()) return nullptr;
    g_decode_step = reinterpret_cast<DecodeStep>(at[0]);
    g_engine_step = reinterpret_cast<EngineStep>(at[1]);
    g_signatures = reinterpret_cast<Signatures>(at[2]);
    g_build_classes = reinterpret_cast<BuildClasses>(at[3]);
    g_displacements = reinterpret_cast<Displacements>(at[4]);
    g_nfa_signatures = reinterpret_cast<NfaSignatures>(at[5]);
    Py_RETURN_NONE;
}

template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyCFunction fast() {
    return reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(F));
}
PyMethodDef g_methods[] = {{"decode_step", fast<decode_step>(), METH_FASTCALL, nullptr},
                           {"engine_step", fast<engine_step>(), METH_FASTCALL, nullptr},
                           {"signatures", fast<signatures>(), METH_FASTCALL, nullptr},
                           {"build_classes", fast<build_classes>(), METH_FASTCALL, nullptr},
                           {"displacements", fast<displacements>(), METH_FASTCALL, nullptr},
                           {"nfa_signatures", fast<nfa_signatures>(), METH_FASTCALL, nullptr},
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
