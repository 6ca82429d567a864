// The per-step tensor helpers of binding.py as native functions: the same arguments, defaults, results and
// errors, without the interpreter's share of a call.  What the host spends on a call decides how long the
// small ones take: of the 5.7 us of a linear of 2 tokens 2.4 us were the checks, addresses and the conversion
// of 16 arguments in Python, 3.2 us the launch itself.
//
// A helper here takes the ordinary call: plain tensors that pass the helper's checks, workspace and output
// given, known names.  Anything else - an argument that is missing, wrong, of another type, a tensor subclass, a
// mode that intercepts tensor methods, a tensor without memory - goes with the same arguments to
// the Python helper, which allocates, raises and dispatches as it does without this module.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "qc.h"

namespace {

enum Helper { kLinear, kAsym, kTensor, kDelta, kSimilarity, kGradient, kVariation, kHelpers };
constexpr int kArgsMost = 9;
const char *const kNames[kHelpers][kArgsMost] = {
    {"X", "pw", "bias", "epi", "out", "workspace", "Y", "act_bits", "rot_block"},
    {"X", "pw", "row_sums", "bias", "epi", "out", "workspace", "Y", "act_bits"},
    {"X", "pw", "bias", "epi", "out", "workspace", "Y", "act_bits"},
    {"cur", "prev", "workspace", "out3"},
    {"a", "b", "workspace", "out4"},
    {"m", "workspace", "out2"},
    {"cur", "prevs", "workspace", "out"},
};
PyObject *names[kHelpers][kArgsMost];   // interned, made once, kept
PyObject *attr_blob, *attr_scale, *attr_N, *attr_K, *attr_bits;

// what one import of the module holds; the C entries are asked for on the first call
struct State {
    PyObject *resolve, *check, *fallback[kHelpers];
    void *entry[kHelpers + 1];   // the last one: qc_qlinear_rot
    bool resolved;
};
State *state_of(PyObject *module) { return static_cast<State *>(PyModule_GetState(module)); }

bool resolve_entries(State *s) {
    if (s->resolved) return true;
    PyObject *addresses = s->resolve ? PyObject_CallNoArgs(s->resolve) : nullptr;
    if (!addresses) return false;
    bool ok = PyTuple_Check(addresses) && PyTuple_GET_SIZE(addresses) == kHelpers + 1;
    for (int i = 0; ok && i <= kHelpers; ++i) {
        s->entry[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i));
        ok = s->entry[i] != nullptr;
    }
    Py_DECREF(addresses);
    s->resolved = ok;
    return ok;
}

// arguments by position and name into out[0 .. count); false for what the Python helper should sort out
bool gather(Helper which, int count, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames, PyObject **out) {
    if (nargs > count) return false;
    for (int i = 0; i < count; ++i) out[i] = i < nargs ? args[i] : nullptr;
    const Py_ssize_t kw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < kw; ++k) {
        PyObject *const name = PyTuple_GET_ITEM(kwnames, k);
        int i = 0;
        while (i < count && names[which][i] != name) ++i;
        if (i == count || out[i]) return false;
        out[i] = args[nargs + k];
    }
    return true;
}

const at::Tensor *tensor(PyObject *o) { return o && THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

bool whole_number(PyObject *o, long absent, long &value) {
    if (!o) { value = absent; return true; }
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    value = PyLong_AsLongAndOverflow(o, &over);
    return over == 0;
}

// index of a text among `count`; absent: the first one
bool choice(PyObject *o, const char *const *texts, int count, int &index) {
    if (!o) { index = 0; return true; }
    if (!PyUnicode_CheckExact(o)) return false;
    for (index = 0; index < count; ++index)
        if (PyUnicode_CompareWithASCIIString(o, texts[index]) == 0) return true;
    return false;
}

bool data_type(const at::Tensor &t, qc_dtype &dt) {
    const auto s = t.scalar_type();
    dt = s == at::kBFloat16 ? QC_BF16 : QC_F32;
    return s == at::kBFloat16 || s == at::kFloat;
}

void *current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// the attributes a linear reads from a PackedWeight
struct Weight {
    const void *blob = nullptr;
    const float *scale = nullptr;
    long N = 0, K = 0, bits = 0;
    bool read(PyObject *pw) {
        if (!pw) return false;
        PyObject *const b = PyObject_GetAttr(pw, attr_blob), *const s = b ? PyObject_GetAttr(pw, attr_scale) : nullptr;
        bool ok = b && s;
        if (ok) {
            const at::Tensor *const tb = tensor(b), *const ts = tensor(s);
            ok = tb && ts;
            if (ok) {
                try {
                    blob = tb->data_ptr();
                    scale = static_cast<const float *>(ts->data_ptr());
                } catch (...) {
                    ok = false;
                }
            }
        }
        Py_XDECREF(b);
        Py_XDECREF(s);
        return ok && number(pw, attr_N, N) && number(pw, attr_K, K) && number(pw, attr_bits, bits);
    }
    static bool number(PyObject *pw, PyObject *attr, long &value) {
        PyObject *const o = PyObject_GetAttr(pw, attr);
        const bool ok = o && whole_number(o, 0, value);
        Py_XDECREF(o);
        return ok;
    }
};

struct Call {
    State *s;
    Helper which;
    PyObject *const *args;
    Py_ssize_t nargs;
    PyObject *kwnames;
    PyObject *a[kArgsMost];

    PyObject *python() const {
        PyErr_Clear();
        return PyObject_Vectorcall(s->fallback[which], args, (size_t)nargs, kwnames);
    }
    // the helper's result, or the error that the Python helper raises for this status
    PyObject *finish(int status, const char *where, PyObject *result) const {
        if (status == QC_OK) {
            Py_INCREF(result);
            return result;
        }
        PyObject *const none = PyObject_CallFunction(s->check, "is", status, where);
        if (!none) return nullptr;
        Py_DECREF(none);
        Py_INCREF(result);
        return result;
    }
};

// body(call): the result, or null without an error set for the Python helper's turn
template <Helper W, int COUNT, typename F>
PyObject *helper(PyObject *module, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames, F body) {
    Call c{state_of(module), W, args, nargs, kwnames, {}};
    if (!c.s->fallback[W]) {
        PyErr_SetString(PyExc_RuntimeError, "setup() has not been called");
        return nullptr;
    }
    if (!gather(W, COUNT, args, nargs, kwnames, c.a) || at::impl::torch_function_mode_enabled()) return c.python();
    if (!resolve_entries(c.s)) return c.python();
    PyObject *result = nullptr;
    bool done = false;
    try {
        done = body(c, result);
    } catch (...) {   // a tensor without memory, without a shape
        if (!done) result = nullptr;
    }
    if (result || (done && PyErr_Occurred())) return result;
    return c.python();
}

const char *const kEpilogues[] = {"none", "gelu_tanh", "gelu_erf"};
const qc_epilogue kEpilogueOf[] = {QC_EPI_NONE, QC_EPI_GELU_TANH, QC_EPI_GELU_ERF};
const char *const kOuts[] = {"bf16", "f32", "i32"};
const qc_out kOutOf[] = {QC_OUT_BF16, QC_OUT_F32, QC_OUT_I32_ACC};

// the three linears; at: where their common arguments from `bias` on begin
bool linear(const Call &c, int at, PyObject *rot, PyObject *row_sums, PyObject *&result) {
    const at::Tensor *const X = tensor(c.a[0]), *const ws = tensor(c.a[at + 3]), *const Y = tensor(c.a[at + 4]);
    PyObject *const bias_object = c.a[at] ? c.a[at] : Py_None;
    const at::Tensor *const bias = bias_object == Py_None ? nullptr : tensor(bias_object);
    const at::Tensor *const sums = row_sums ? tensor(row_sums) : nullptr;
    if (!X || !ws || !Y || (bias_object != Py_None && !bias) || (c.which == kAsym && !sums)) return false;
    int epi, out;
    long act_bits, rot_block;
    qc_dtype xdt;
    Weight w;
    if (!choice(c.a[at + 1], kEpilogues, 3, epi) || !choice(c.a[at + 2], kOuts, 3, out) || !whole_number(c.a[at + 5], 8, act_bits) ||
        !whole_number(rot, 0, rot_block) || !data_type(*X, xdt) || !w.read(c.a[1]))
        return false;
    if (!X->is_cuda() || !X->is_contiguous() || X->dim() != 2 || X->size(1) != w.K) return false;
    const int64_t M = X->size(0), K = w.K, N = w.N;
    const void *const x = X->data_ptr();
    const float *const b = bias ? static_cast<const float *>(bias->data_ptr()) : nullptr;
    const int32_t *const rs = sums ? static_cast<const int32_t *>(sums->data_ptr()) : nullptr;
    void *const y = Y->data_ptr(), *const space = ws->data_ptr(), *const stream = current_stream();
    const size_t bytes = (size_t)ws->numel();
    const qc_epilogue e = kEpilogueOf[epi];
    const qc_out o = kOutOf[out];
    const char *where;
    int status;
    Py_BEGIN_ALLOW_THREADS
    if (c.which == kAsym) {
        where = "qc_qlinear_asym";
        status = reinterpret_cast<decltype(&qc_qlinear_asym)>(c.s->entry[kAsym])(
            x, xdt, M, K, (int)act_bits, w.blob, w.scale, rs, (int)w.bits, N, b, e, y, o, space, bytes, stream);
    } else if (c.which == kTensor) {
        where = "qc_qlinear_tensor";
        status = reinterpret_cast<decltype(&qc_qlinear_tensor)>(c.s->entry[kTensor])(
            x, xdt, M, K, (int)act_bits, w.blob, w.scale, (int)w.bits, N, b, e, y, o, space, bytes, stream);
    } else if (rot_block) {
        where = "qc_qlinear_rot";
        status = reinterpret_cast<decltype(&qc_qlinear_rot)>(c.s->entry[kHelpers])(
            x, xdt, M, K, (int)act_bits, (int)rot_block, w.blob, w.scale, (int)w.bits, N, b, e, y, o, space, bytes, stream);
    } else {
        where = "qc_qlinear_act_bits";
        status = reinterpret_cast<decltype(&qc_qlinear_act_bits)>(c.s->entry[kLinear])(
            x, xdt, M, K, (int)act_bits, w.blob, w.scale, (int)w.bits, N, b, e, y, o, space, bytes, stream);
    }
    Py_END_ALLOW_THREADS
    result = c.finish(status, where, c.a[at + 4]);
    return true;
}

PyObject *qlinear_t(PyObject *m, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    return helper<kLinear, 9>(m, args, n, kw, [](const Call &c, PyObject *&r) { return linear(c, 2, c.a[8], nullptr, r); });
}
PyObject *qlinear_asym_t(PyObject *m, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    return helper<kAsym, 9>(m, args, n, kw, [](const Call &c, PyObject *&r) { return linear(c, 3, nullptr, c.a[2], r); });
}
PyObject *qlinear_tensor_t(PyObject *m, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    return helper<kTensor, 8>(m, args, n, kw, [](const Call &c, PyObject *&r) { return linear(c, 2, nullptr, nullptr, r); });
}

bool is_input(const at::Tensor &t) { return t.is_cuda() && t.is_contiguous(); }

PyObject *latent_delta_t(PyObject *m, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    return helper<kDelta, 4>(m, args, n, kw, [](const Call &c, PyObject *&r) {
        const at::Tensor *const cur = tensor(c.a[0]), *const prev = tensor(c.a[1]), *const ws = tensor(c.a[2]), *const out = tensor(c.a[3]);
        if (!cur || !prev || !ws || !out || !is_input(*cur) || cur->scalar_type() != at::kFloat || prev->sizes() != cur->sizes() ||
            prev->scalar_type() != at::kFloat || !prev->is_contiguous())
            return false;
        const float *const p = static_cast<const float *>(cur->data_ptr()), *const q = static_cast<const float *>(prev->data_ptr());
        float *const o = static_cast<float *>(out->data_ptr());
        void *const space = ws->data_ptr(), *const stream = current_stream();
        const int64_t count = cur->numel(), bytes = ws->numel();
        int status;
        Py_BEGIN_ALLOW_THREADS
        status = reinterpret_cast<decltype(&qc_latent_delta)>(c.s->entry[kDelta])(p, q, count, o, space, (size_t)bytes, stream);
        Py_END_ALLOW_THREADS
        r = c.finish(status, "qc_latent_delta", c.a[3]);
        return true;
    });
}

PyObject *layer_similarity_t(PyObject *m, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    return helper<kSimilarity, 4>(m, args, n, kw, [](const Call &c, PyObject *&r) {
        const at::Tensor *const a = tensor(c.a[0]), *const b = tensor(c.a[1]), *const ws = tensor(c.a[2]), *const out = tensor(c.a[3]);
        qc_dtype dt;
        if (!a || !b || !ws || !out || !is_input(*a) || !b->is_contiguous() || a->sizes() != b->sizes() ||
            a->scalar_type() != b->scalar_type() || !data_type(*a, dt))
            return false;
        const void *const p = a->data_ptr(), *const q = b->data_ptr();
        float *const o = static_cast<float *>(out->data_ptr());
        void *const space = ws->data_ptr(), *const stream = current_stream();
        const int64_t count = a->numel(), bytes = ws->numel();
        int status;
        Py_BEGIN_ALLOW_THREADS
        status = reinterpret_cast<decltype(&qc_layer_similarity)>(c.s->entry[kSimilarity])(p, q, dt, count, o, space, (size_t)bytes, stream);
        Py_END_ALLOW_THREADS
        r = c.finish(status, "qc_layer_similarity", c.a[3]);
        return true;
    });
}

PyObject *frame_gradient_norm_t(PyObject *m, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    return helper<kGradient, 3>(m, args, n, kw, [](const Call &c, PyObject *&r) {
        const at::Tensor *const t = tensor(c.a[0]), *const ws = tensor(c.a[1]), *const out = tensor(c.a[2]);
        qc_dtype dt;
        if (!t || !ws || !out || !is_input(*t) || t->dim() < 2 || t->size(0) < 1 || !data_type(*t, dt)) return false;
        const int64_t frames = t->size(0), inner = t->numel() / frames, bytes = ws->numel();
        const void *const p = t->data_ptr();
        float *const o = static_cast<float *>(out->data_ptr());
        void *const space = ws->data_ptr(), *const stream = current_stream();
        int status;
        Py_BEGIN_ALLOW_THREADS
        status = reinterpret_cast<decltype(&qc_frame_gradient_norm)>(c.s->entry[kGradient])(p, dt, frames, inner, o, space, (size_t)bytes, stream);
        Py_END_ALLOW_THREADS
        r = c.finish(status, "qc_frame_gradient_norm", c.a[2]);
        return true;
    });
}

PyObject *cumulative_variation_t(PyObject *m, PyObject *const *args, Py_ssize_t n, PyObject *kw) {
    return helper<kVariation, 4>(m, args, n, kw, [](const Call &c, PyObject *&r) {
        const at::Tensor *const cur = tensor(c.a[0]), *const ws = tensor(c.a[2]), *const out = tensor(c.a[3]);
        PyObject *const list = c.a[1];
        if (!cur || !ws || !out || !list || !PyList_CheckExact(list) || PyList_GET_SIZE(list) < 1 || PyList_GET_SIZE(list) > QC_MAX_PREV ||
            !is_input(*cur) || cur->scalar_type() != at::kFloat)
            return false;
        const int count = (int)PyList_GET_SIZE(list);
        const int64_t elements = cur->numel(), bytes = ws->numel();
        const float *prevs[QC_MAX_PREV];
        for (int i = 0; i < count; ++i) {
            const at::Tensor *const p = tensor(PyList_GET_ITEM(list, i));
            if (!p || !is_input(*p) || p->scalar_type() != at::kFloat || p->numel() != elements) return false;
            prevs[i] = static_cast<const float *>(p->data_ptr());
        }
        const float *const p = static_cast<const float *>(cur->data_ptr());
        float *const o = static_cast<float *>(out->data_ptr());
        void *const space = ws->data_ptr(), *const stream = current_stream();
        int status;
        Py_BEGIN_ALLOW_THREADS
        status = reinterpret_cast<decltype(&qc_cumulative_variation)>(c.s->entry[kVariation])(p, prevs, count, elements, o, space, (size_t)bytes, stream);
        Py_END_ALLOW_THREADS
        r = c.finish(status, "qc_cumulative_variation", c.a[3]);
        return true;
    });
}

// setup(resolve, check, (the Python helpers, in the order of Helper)).  resolve() -> the addresses of the C entries, in
// that order and qc_qlinear_rot last; check(status, where) raises.
PyObject *setup(PyObject *module, PyObject *args) {
    PyObject *resolve, *check, *helpers;
    if (!PyArg_ParseTuple(args, "OOO!", &resolve, &check, &PyTuple_Type, &helpers)) return nullptr;
    if (PyTuple_GET_SIZE(helpers) != kHelpers) {
        PyErr_SetString(PyExc_ValueError, "one Python helper for each native one");
        return nullptr;
    }
    State *const s = state_of(module);
    Py_INCREF(resolve);
    Py_XSETREF(s->resolve, resolve);
    Py_INCREF(check);
    Py_XSETREF(s->check, check);
    for (int i = 0; i < kHelpers; ++i) {
        PyObject *const f = PyTuple_GET_ITEM(helpers, i);
        Py_INCREF(f);
        Py_XSETREF(s->fallback[i], f);
    }
    s->resolved = false;
    Py_RETURN_NONE;
}

#define QC_METHOD(name, signature, ...) \
    {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL | METH_KEYWORDS, #name signature "\n--\n\n" __VA_ARGS__}
PyMethodDef methods[] = {
    QC_METHOD(qlinear_t, "($module, X, pw, bias=None, epi='none', out='bf16', workspace=None, Y=None, act_bits=8, rot_block=0)"),
    QC_METHOD(qlinear_asym_t, "($module, X, pw, row_sums, bias=None, epi='none', out='bf16', workspace=None, Y=None, act_bits=8)"),
    QC_METHOD(qlinear_tensor_t, "($module, X, pw, bias=None, epi='none', out='bf16', workspace=None, Y=None, act_bits=8)"),
    QC_METHOD(latent_delta_t, "($module, cur, prev, workspace=None, out3=None)"),
    QC_METHOD(layer_similarity_t, "($module, a, b, workspace=None, out4=None)"),
    QC_METHOD(frame_gradient_norm_t, "($module, m, workspace=None, out2=None)",
              "m: [frames, ...] float32 or bfloat16, contiguous -> device float [2]."),
    QC_METHOD(cumulative_variation_t, "($module, cur, prevs, workspace=None, out=None)",
              "cur float32 [n], prevs a list of float32 tensors of the same size -> device float\n[len(prevs) + 1]."),
    {"setup", setup, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

int traverse(PyObject *module, visitproc visit, void *arg) {
    if (State *const s = state_of(module)) {
        Py_VISIT(s->resolve);
        Py_VISIT(s->check);
        for (PyObject *f : s->fallback) Py_VISIT(f);
    }
    return 0;
}
int clear(PyObject *module) {
    if (State *const s = state_of(module)) {
        Py_CLEAR(s->resolve);
        Py_CLEAR(s->check);
        for (PyObject *&f : s->fallback) Py_CLEAR(f);
    }
    return 0;
}
void release(void *module) { clear(static_cast<PyObject *>(module)); }

int execute(PyObject *) {
    for (int w = 0; w < kHelpers; ++w)
        for (int i = 0; i < kArgsMost && kNames[w][i]; ++i)
            if (!names[w][i] && !(names[w][i] = PyUnicode_InternFromString(kNames[w][i]))) return -1;
    PyObject **const attrs[] = {&attr_blob, &attr_scale, &attr_N, &attr_K, &attr_bits};
    const char *const texts[] = {"blob", "scale", "N", "K", "bits"};
    for (int i = 0; i < 5; ++i)
        if (!*attrs[i] && !(*attrs[i] = PyUnicode_InternFromString(texts[i]))) return -1;
    return 0;
}

// a state per import: two copies of the binding in one process do not share their C entries
PyModuleDef_Slot slots[] = {{Py_mod_exec, (void *)execute}, {0, nullptr}};
PyModuleDef definition = {PyModuleDef_HEAD_INIT, "_qc_torch", nullptr, sizeof(State), methods, slots, traverse, clear, release};

}  // namespace

PyMODINIT_FUNC PyInit__qc_torch(void) { return PyModuleDef_Init(&definition); }
