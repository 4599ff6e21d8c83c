// The compute entry points as Python calls them: torch tensors to device pointers, outputs that the caller did not pass
// allocated, the status checked.  No computation.
//
// A step of a small model is bound by the host: two calls whose four kernels take less time than it takes to issue them.
// Through ctypes the step's two calls cost 23.7 microseconds (one sequence, 4 heads, 8 rounds): 11.0 in the library,
// nearly all of it the launches, 8.6 for the six output tensors (torch.empty from Python takes 1.4 each) and 4 of argument
// marshalling.  Here an output costs what the allocator costs and the arguments are read directly: 24.7 -> 19.9 microseconds
// a pass on one GPU.
//
// The library is not linked: its functions arrive as addresses (setup), from whichever build of it was loaded.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <cmath>
#include <cstring>

#include "round_attention.h"

namespace {

struct Functions {
    decltype(&ra_round_scores) scores;
    decltype(&ra_round_scores_select) scores_select;
    decltype(&ra_round_scores_accumulate) scores_accumulate;
    decltype(&ra_selection_coverage) coverage;
    decltype(&ra_round_sparse_attn_decode) decode;
    decltype(&ra_watershed_attn_decode) watershed_decode;
    decltype(&ra_round_sparse_attn_prefill) prefill;
    decltype(&ra_watershed_attn_prefill) watershed_prefill;
} fn;
PyObject* on_error = nullptr;  // called with a status that is not RA_OK; raises
PyObject* name_c = nullptr;    // "c"
// What an argument may be is ctypes' rule, as for every other call of the package: structures by their type (only a
// c_void_p is read as a handle, only a ra_kv_view as a view, ...), and whatever is not of the usual type goes to ctypes itself,
// which converts or refuses it.
PyObject *handle_type = nullptr, *view_type = nullptr, *params_type = nullptr;  // c_void_p, ra_kv_view, ra_select_params
PyObject *to_handle = nullptr, *to_float = nullptr;                             // object -> int, object -> float by ctypes
PyObject *wrong_type = nullptr, *not_a_tensor = nullptr;                        // exceptions

// A Python error is set: leave the entry point.
struct PythonError {};

// A ctypes object's memory, if it is of `type`.
template <typename T>
T* address_of(PyObject* o, PyObject* type, const char* what) {
    if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(type))) {
        PyErr_Format(wrong_type, "%s: %s expected, not %s", what, reinterpret_cast<PyTypeObject*>(type)->tp_name, Py_TYPE(o)->tp_name);
        throw PythonError();
    }
    Py_buffer buf;
    if (PyObject_GetBuffer(o, &buf, PyBUF_SIMPLE) != 0) throw PythonError();
    T* p = static_cast<T*>(buf.buf);
    PyBuffer_Release(&buf);  // the object itself is kept by the caller's reference
    return p;
}

void* handle(PyObject* o) {
    if (o == Py_None) return nullptr;
    if (PyLong_Check(o)) return reinterpret_cast<void*>(PyLong_AsUnsignedLongMask(o));
    if (PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(handle_type))) return *address_of<void*>(o, handle_type, "handle");
    PyObject* r = PyObject_CallOneArg(to_handle, o);
    if (!r) throw PythonError();
    void* p = r == Py_None ? nullptr : PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    if (PyErr_Occurred()) throw PythonError();
    return p;
}
ra_ctx* context(PyObject* o) { return static_cast<ra_ctx*>(handle(o)); }

// The C view of a KVView; holds a reference to the structure while the call lasts.
struct View {
    PyObject* c;
    const ra_kv_view* p;
    explicit View(PyObject* view) : c(PyObject_GetAttr(view, name_c)), p(nullptr) {
        if (!c) throw PythonError();
        try {
            p = address_of<ra_kv_view>(c, view_type, "view");
        } catch (...) {
            Py_DECREF(c);
            throw;
        }
    }
    View(const View&) = delete;
    View& operator=(const View&) = delete;
    ~View() { Py_DECREF(c); }
    const ra_kv_view* operator->() const { return p; }
};

const at::Tensor* tensor_or_null(PyObject* o) {
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) {
        PyErr_Format(not_a_tensor, "expected a torch.Tensor, not %s", Py_TYPE(o)->tp_name);
        throw PythonError();
    }
    return &THPVariable_Unpack(o);
}
const at::Tensor& tensor(PyObject* o) {
    const at::Tensor* t = tensor_or_null(o);
    if (!t) {
        PyErr_SetString(PyExc_AttributeError, "expected a torch.Tensor, not None");
        throw PythonError();
    }
    return *t;
}
void* data(const at::Tensor& t) {
    if (!t.is_contiguous()) {
        PyErr_SetString(PyExc_AssertionError, "tensors handed to the library must be contiguous");
        throw PythonError();
    }
    return t.data_ptr();
}
template <typename T = void>
T* data(PyObject* o) {
    const at::Tensor* t = tensor_or_null(o);
    return t ? static_cast<T*>(data(*t)) : nullptr;
}
void want_dims(const at::Tensor& t, int64_t dims) {
    if (t.dim() == dims) return;
    PyErr_Format(PyExc_ValueError, "a tensor of %d dimensions is needed here, this one has %d", (int)dims, (int)t.dim());
    throw PythonError();
}
int second_size(PyObject* o) {  // tokens of the current round; 0 without one
    const at::Tensor* t = tensor_or_null(o);
    return t ? (int)t->size(1) : 0;
}
float scale_of(PyObject* o, int64_t d) {
    if (o == Py_None) {
        if (d == 0) {
            PyErr_SetString(PyExc_ZeroDivisionError, "no default scale without channels");
            throw PythonError();
        }
        return (float)std::pow((double)d, -0.5);
    }
    if (PyFloat_Check(o)) return (float)PyFloat_AS_DOUBLE(o);
    PyObject* r = PyObject_CallOneArg(to_float, o);
    if (!r) throw PythonError();
    const double v = PyFloat_AsDouble(r);
    Py_DECREF(r);
    if (v == -1.0 && PyErr_Occurred()) throw PythonError();
    return (float)v;
}

// An output: the caller's tensor, or a new one, which allocate() gets.
template <typename T>
struct Output {
    PyObject* given;  // None: a new one
    T* p;
    at::DimVector shape;
    at::TensorOptions options;
    at::Tensor made;
    Output(PyObject* o, at::IntArrayRef dims, const at::Tensor& like)
        : given(o), p(data<T>(o)), shape(dims.begin(), dims.end()),
          options(at::TensorOptions().dtype(c10::CppTypeToScalarType<T>::value).device(like.device())) {}
    void allocate() {
        if (given != Py_None) return;
        made = at::empty(shape, options);
        p = static_cast<T*>(made.data_ptr());
    }
    PyObject* object() {  // a new reference
        if (given == Py_None) return THPVariable_Wrap(made);
        Py_INCREF(given);
        return given;
    }
};

template <typename T>
PyObject* results(Output<T>& out) { return out.object(); }
template <typename... Outputs>
PyObject* results(Outputs&... outs) {
    PyObject* tuple = PyTuple_New((Py_ssize_t)sizeof...(Outputs));
    if (!tuple) return nullptr;
    Py_ssize_t i = 0;
    const auto add = [&](PyObject* o) {
        if (o) PyTuple_SET_ITEM(tuple, i++, o);
        return o != nullptr;
    };
    if ((add(outs.object()) && ...)) return tuple;
    Py_DECREF(tuple);
    return nullptr;
}

// The interpreter, given to the other threads until the end of the block, also by an exception.
struct Released {
    PyThreadState* state = PyEval_SaveThread();
    Released() = default;
    Released(const Released&) = delete;
    Released& operator=(const Released&) = delete;
    ~Released() { PyEval_RestoreThread(state); }
};

// New outputs and the library call, with the interpreter released: an allocation may have to get memory from the device, or
// wait for it.  A status that is not RA_OK is raised.
template <typename Call, typename... Outputs>
PyObject* checked(Call call, Outputs&... outs) {
    int rc;
    {
        const Released released;
        (outs.allocate(), ...);
        rc = call();
    }
    if (rc == RA_OK) return results(outs...);
    PyObject* r = PyObject_CallFunction(on_error, "i", rc);
    if (r) {
        Py_DECREF(r);
        PyErr_SetString(PyExc_SystemError, "the status handler did not raise");
    }
    throw PythonError();
}

// (ctx, stream, q, view, cur_k, scale, scores_head, scores)
PyObject* scores(PyObject* const* a) {
    const at::Tensor& q = tensor(a[2]);
    want_dims(q, 4);
    const View view(a[3]);
    const int64_t B = q.size(0), q_len = q.size(1), Hq = q.size(2), R = view->R_max;
    Output<float> ph(a[6], {B, Hq, R}, q), p(a[7], {B, R}, q);
    ra_ctx* ctx = context(a[0]);
    void *st = handle(a[1]), *qp = data(q), *ck = data(a[4]);
    const int cur = second_size(a[4]);
    const float scale = scale_of(a[5], q.size(3));
    return checked([&] { return fn.scores(ctx, st, qp, (int)q_len, (int)Hq, view.p, ck, cur, scale, ph.p, p.p); }, ph, p);
}

// (ctx, stream, q, view, params, cur_k, scale, scores_head, scores, sel_idx, n_sel)
PyObject* scores_select(PyObject* const* a) {
    const at::Tensor& q = tensor(a[2]);
    want_dims(q, 4);
    const View view(a[3]);
    const int64_t B = q.size(0), q_len = q.size(1), Hq = q.size(2), R = view->R_max;
    Output<float> ph(a[7], {B, Hq, R}, q), p(a[8], {B, R}, q);
    Output<int32_t> sel(a[9], {B, R}, q), n(a[10], {B}, q);
    ra_ctx* ctx = context(a[0]);
    const ra_select_params* params = address_of<ra_select_params>(a[4], params_type, "params");
    void *st = handle(a[1]), *qp = data(q), *ck = data(a[5]);
    const int cur = second_size(a[5]);
    const float scale = scale_of(a[6], q.size(3));
    return checked(
        [&] { return fn.scores_select(ctx, st, qp, (int)q_len, (int)Hq, view.p, ck, cur, scale, params, ph.p, p.p, sel.p,
                                      n.p); },
        ph, p, sel, n);
}

// (ctx, stream, q, view, acc, cur_k, scale, scores_head, scores)
PyObject* scores_accumulate(PyObject* const* a) {
    const at::Tensor& q = tensor(a[2]);
    want_dims(q, 4);
    const View view(a[3]);
    const int64_t B = q.size(0), q_len = q.size(1), Hq = q.size(2), R = view->R_max;
    if (a[4] != Py_None && !THPVariable_Check(a[4])) {
        PyErr_SetString(PyExc_AssertionError, "acc must be a tensor");
        throw PythonError();
    }
    const at::Tensor& acc = tensor(a[4]);
    if (acc.scalar_type() != at::kFloat || acc.sizes() != at::IntArrayRef({B, Hq, R})) {
        PyErr_SetString(PyExc_AssertionError, "acc must be float32 [B, Hq, R_max]");
        throw PythonError();
    }
    Output<float> ph(a[7], {B, Hq, R}, q), p(a[8], {B, R}, q);
    ra_ctx* ctx = context(a[0]);
    void *st = handle(a[1]), *qp = data(q), *ck = data(a[5]);
    float* ap = static_cast<float*>(data(acc));
    const int cur = second_size(a[5]);
    const float scale = scale_of(a[6], q.size(3));
    return checked(
        [&] { return fn.scores_accumulate(ctx, st, qp, (int)q_len, (int)Hq, view.p, ck, cur, scale, ap, ph.p, p.p); },
        ph, p);
}

// (ctx, stream, scores, sel_idx, n_sel)
PyObject* coverage(PyObject* const* a) {
    const at::Tensor& s = tensor(a[2]);
    want_dims(s, 2);
    const int64_t B = s.size(0), R = s.size(1);
    Output<float> cov(Py_None, {B}, s);
    ra_ctx* ctx = context(a[0]);
    void* st = handle(a[1]);
    const float* sp = static_cast<float*>(data(s));
    const int32_t *sel = data<int32_t>(a[3]), *n = data<int32_t>(a[4]);
    return checked([&] { return fn.coverage(ctx, st, sp, sel, n, (int)B, (int)R, cov.p); }, cov);
}

// (ctx, stream, q, view, sel_idx, n_sel, cur_k, cur_v, cur_len, scale, out, lse)
PyObject* decode(PyObject* const* a) {
    const at::Tensor& q = tensor(a[2]);
    want_dims(q, 3);
    const View view(a[3]);
    const int64_t B = q.size(0), Hq = q.size(1), d = q.size(2);
    Output<float> out(a[10], {B, Hq, d}, q), lse(a[11], {B, Hq}, q);
    ra_ctx* ctx = context(a[0]);
    void *st = handle(a[1]), *qp = data(q), *ck = data(a[6]), *cv = data(a[7]);
    const int32_t *sel = data<int32_t>(a[4]), *n = data<int32_t>(a[5]), *cl = data<int32_t>(a[8]);
    const int cap = second_size(a[6]);
    const float scale = scale_of(a[9], d);
    return checked(
        [&] { return fn.decode(ctx, st, qp, (int)Hq, view.p, sel, n, ck, cv, cl, cap, scale, out.p, lse.p); },
        out, lse);
}

// (ctx, stream, q, view, cur_k, cur_v, cur_len, scale, out, lse, scores_head, scores)
PyObject* watershed_decode(PyObject* const* a) {
    const at::Tensor& q = tensor(a[2]);
    want_dims(q, 3);
    const View view(a[3]);
    const int64_t B = q.size(0), Hq = q.size(1), d = q.size(2), R = view->R_max;
    Output<float> out(a[8], {B, Hq, d}, q), lse(a[9], {B, Hq}, q);
    Output<float> ph(a[10], {B, Hq, R}, q), p(a[11], {B, R}, q);
    ra_ctx* ctx = context(a[0]);
    void *st = handle(a[1]), *qp = data(q), *ck = data(a[4]), *cv = data(a[5]);
    const int32_t* cl = data<int32_t>(a[6]);
    const int cap = second_size(a[4]);
    const float scale = scale_of(a[7], d);
    return checked(
        [&] { return fn.watershed_decode(ctx, st, qp, (int)Hq, view.p, ck, cv, cl, cap, scale, out.p, lse.p, ph.p,
                                         p.p); },
        out, lse, ph, p);
}

// (ctx, stream, q, view, sel_idx, n_sel, cur_k, cur_v, scale, out, lse)
PyObject* prefill(PyObject* const* a) {
    const at::Tensor& q = tensor(a[2]);
    want_dims(q, 4);
    const View view(a[3]);
    const int64_t B = q.size(0), q_len = q.size(1), Hq = q.size(2), d = q.size(3);
    Output<float> out(a[9], {B, q_len, Hq, d}, q), lse(a[10], {B, q_len, Hq}, q);
    ra_ctx* ctx = context(a[0]);
    void *st = handle(a[1]), *qp = data(q), *ck = data(a[6]), *cv = data(a[7]);
    const int32_t *sel = data<int32_t>(a[4]), *n = data<int32_t>(a[5]);
    const int cur = second_size(a[6]);
    const float scale = scale_of(a[8], d);
    return checked(
        [&] { return fn.prefill(ctx, st, qp, (int)q_len, (int)Hq, view.p, sel, n, ck, cv, cur, scale, out.p, lse.p); },
        out, lse);
}

// (ctx, stream, q, view, cur_k, cur_v, scale, out, lse, scores_head, scores)
PyObject* watershed_prefill(PyObject* const* a) {
    const at::Tensor& q = tensor(a[2]);
    want_dims(q, 4);
    const View view(a[3]);
    const int64_t B = q.size(0), q_len = q.size(1), Hq = q.size(2), d = q.size(3), R = view->R_max;
    Output<float> out(a[7], {B, q_len, Hq, d}, q), lse(a[8], {B, q_len, Hq}, q);
    Output<float> ph(a[9], {B, Hq, R}, q), p(a[10], {B, R}, q);
    ra_ctx* ctx = context(a[0]);
    void *st = handle(a[1]), *qp = data(q), *ck = data(a[4]), *cv = data(a[5]);
    const int cur = second_size(a[4]);
    const float scale = scale_of(a[6], d);
    return checked(
        [&] { return fn.watershed_prefill(ctx, st, qp, (int)q_len, (int)Hq, view.p, ck, cv, cur, scale, out.p, lse.p,
                                          ph.p, p.p); },
        out, lse, ph, p);
}

// The Python function: argument count, C++ exceptions (an allocation that fails among them) turned into Python's.
template <PyObject* (*F)(PyObject* const*), Py_ssize_t N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != N) {
        PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", N, nargs);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const PythonError&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// setup(status handler, c_void_p, ra_kv_view, ra_select_params, to_handle, to_float, wrong_type, not_a_tensor, addresses in the
// order of Functions)
PyObject** const kObjects[] = {&on_error, &handle_type, &view_type, &params_type, &to_handle, &to_float, &wrong_type, &not_a_tensor};
constexpr Py_ssize_t kNumObjects = sizeof(kObjects) / sizeof(kObjects[0]), kNumFunctions = sizeof(Functions) / sizeof(void*);
PyObject* setup(PyObject* const* a) {
    void* p[kNumFunctions];
    for (Py_ssize_t i = 0; i < kNumFunctions; ++i) {
        p[i] = PyLong_AsVoidPtr(a[kNumObjects + i]);
        if (PyErr_Occurred()) throw PythonError();
    }
    for (Py_ssize_t i = 1; i <= 3; ++i)
        if (!PyType_Check(a[i])) {
            PyErr_SetString(PyExc_TypeError, "setup: a type is expected");
            throw PythonError();
        }
    std::memcpy(&fn, p, sizeof(fn));
    for (Py_ssize_t i = 0; i < kNumObjects; ++i) {
        Py_INCREF(a[i]);
        Py_XSETREF(*kObjects[i], a[i]);
    }
    Py_RETURN_NONE;
}

// What ctypes calls to convert an argument for us: the value comes back as it arrives.
void* same_handle(void* p) { return p; }
float same_float(float v) { return v; }
PyObject* conversions(PyObject* const*) {
    return Py_BuildValue("(NN)", PyLong_FromVoidPtr(reinterpret_cast<void*>(same_handle)),
                         PyLong_FromVoidPtr(reinterpret_cast<void*>(same_float)));
}

#define RA_METHOD(NAME, N) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<NAME, N>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    RA_METHOD(setup, kNumObjects + kNumFunctions),
    RA_METHOD(conversions, 0),
    RA_METHOD(scores, 8),
    RA_METHOD(scores_select, 11),
    RA_METHOD(scores_accumulate, 9),
    RA_METHOD(coverage, 5),
    RA_METHOD(decode, 12),
    RA_METHOD(watershed_decode, 12),
    RA_METHOD(prefill, 11),
    RA_METHOD(watershed_prefill, 11),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
    name_c = PyUnicode_InternFromString("c");
    return name_c ? PyModule_Create(&module) : nullptr;
}
