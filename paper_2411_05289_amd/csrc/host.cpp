// The per-call work of binding.py's draft and verify functions in native code: looking the tensors over,
// filling the C structures, allocating the outputs and making the call.  In Python these cost more than
// the kernels of a small batch (config 1, 4096 trees: spechub_draft and spechub_verify 37 us of host time a
// pair for 12 us of kernels; here 15).
//
// draft() and verify() take what the Python functions were given and return the outputs, or an MDSD_E_*
// code (a negative int) for the caller to raise, or None for anything out of the ordinary (a tensor
// subclass, a wrong shape, type or layout): the caller then goes its own way, which raises the error.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/autograd/python_variable.h>

#include <utility>

#include "mdsd.h"

namespace {

// what a call is about, from the first arguments of draft() and verify()
struct Rows {
    mdsd_problem pb;
    int64_t B, N, V;
    at::Tensor draft;
};

const at::Tensor* tensor_of(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

bool is_rows(const at::Tensor& t)
{
    return t.is_cuda() && t.dim() == 3 && t.stride(2) == 1 && t.stride(0) == t.size(1) * t.stride(1) &&
           (t.scalar_type() == at::kFloat || t.scalar_type() == at::kBFloat16);
}

// a contiguous device tensor of this type and shape
const at::Tensor* plain(PyObject* o, at::ScalarType type, at::IntArrayRef shape)
{
    const at::Tensor* t = tensor_of(o);
    return t && t->is_cuda() && t->scalar_type() == type && t->is_contiguous() && t->sizes() == shape ? t : nullptr;
}

bool number(PyObject* o, int32_t& v)
{
    if (!PyLong_CheckExact(o)) return false;
    const long l = PyLong_AsLong(o);
    if ((l == -1 && PyErr_Occurred()) || l != (int32_t)l) {
        PyErr_Clear();
        return false;
    }
    v = (int32_t)l;
    return true;
}
bool number(PyObject* o, float& v)
{
    if (!PyFloat_CheckExact(o)) return false;  // (an integer temperature goes the other way)
    v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}

// args: target or None, draft, kind, k, depth, temp_target, temp_draft, first_child or None, draft_stats or None
constexpr int kRowArgs = 9;
bool rows_of(PyObject* const* a, Rows& r)
{
    mdsd_problem& p = r.pb;
    p = mdsd_problem{};
    const at::Tensor* draft = tensor_of(a[1]);
    if (!draft || !is_rows(*draft)) return false;
    r.draft = *draft;
    r.B = draft->size(0);
    r.N = draft->size(1);
    r.V = draft->size(2);
    if (r.B > INT32_MAX || r.N > INT32_MAX || r.V > INT32_MAX) return false;
    p.ld_t = draft->stride(1);
    if (a[0] != Py_None) {
        const at::Tensor* target = tensor_of(a[0]);
        if (!target || !is_rows(*target) || target->sizes() != draft->sizes() ||
            target->scalar_type() != draft->scalar_type())
            return false;
        p.target = target->data_ptr();
        p.ld_t = target->stride(1);
    }
    p.draft = draft->data_ptr();
    p.ld_d = draft->stride(1);
    p.dtype = draft->scalar_type() == at::kFloat ? MDSD_FP32 : MDSD_BF16;
    p.B = (int32_t)r.B;
    p.N = (int32_t)r.N;
    p.V = (int32_t)r.V;
    if (!number(a[2], p.kind) || !number(a[3], p.k) || !number(a[4], p.depth) || !number(a[5], p.temp_target) ||
        !number(a[6], p.temp_draft))
        return false;
    if (a[7] != Py_None) {
        const at::Tensor* t = plain(a[7], at::kInt, {r.N});
        if (!t) return false;
        p.first_child = (const int32_t*)t->data_ptr();
    }
    if (a[8] != Py_None) {
        const at::Tensor* t = plain(a[8], at::kFloat, {r.B, r.N, 4});
        if (!t) return false;
        p.draft_stats = (mdsd_row_stats*)t->data_ptr();
    }
    return true;
}

bool stream_of(PyObject* o, void*& stream)
{
    stream = PyLong_AsVoidPtr(o);
    if (!PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}

// the outputs of a call; given up with everything in it wherever the call does not come to its end
struct Outputs {
    PyObject* dict = PyDict_New();
    Outputs()
    {
        if (!dict) throw std::bad_alloc();
    }
    Outputs(const Outputs&) = delete;
    ~Outputs() { Py_XDECREF(dict); }

    // a new output under `name`; its data pointer
    void* add(const char* name, at::IntArrayRef shape, const at::TensorOptions& options)
    {
        at::Tensor t = at::empty(shape, options);
        void* data = t.data_ptr();
        PyObject* o = THPVariable_Wrap(std::move(t));
        const bool ok = o && PyDict_SetItemString(dict, name, o) == 0;
        Py_XDECREF(o);
        if (!ok) throw std::bad_alloc();
        return data;
    }
    // what a call that the library answered with `rc` returns
    PyObject* answer(int rc)
    {
        return rc == MDSD_OK ? std::exchange(dict, nullptr) : PyLong_FromLong(rc);
    }
};

template <class F>
PyObject* guarded(F f)
{
    try {
        return f();
    } catch (const std::exception&) {  // an allocation that failed: torch reports it on the other way
        if (PyErr_Occurred()) return nullptr;
        Py_RETURN_NONE;
    }
}

// draft(method, stream, <rows>, u)
PyObject* draft(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        int32_t method;
        void* stream;
        Rows r;
        if (n != 2 + kRowArgs + 1 || !number(a[0], method) || !stream_of(a[1], stream) || !rows_of(a + 2, r))
            Py_RETURN_NONE;
        const at::Tensor* u = plain(a[2 + kRowArgs], at::kFloat, {r.B, r.N, r.pb.k});
        if (!u) Py_RETURN_NONE;
        Outputs out;
        const at::TensorOptions ints = r.draft.options().dtype(at::kInt);
        int32_t* tokens = (int32_t*)out.add("tokens", {r.B, r.N}, ints);
        int32_t* flags = (int32_t*)out.add("flags", {r.B, r.N}, ints);
        int32_t* hub = method == 0 ? (int32_t*)out.add("hub", {r.B, r.N}, ints) : nullptr;
        const float* up = (const float*)u->data_ptr();
        int rc;
        Py_BEGIN_ALLOW_THREADS;
        rc = method == 0   ? spechub_draft(&r.pb, up, tokens, hub, flags, nullptr, 0, stream)
             : method == 1 ? rrs_draft(&r.pb, up, tokens, flags, nullptr, 0, stream)
                           : rrsw_draft(&r.pb, up, tokens, flags, nullptr, 0, stream);
        Py_END_ALLOW_THREADS;
        return out.answer(rc);
    });
}

// verify(method, stream, <rows>, tokens, u, resid_mass, flags, resid_prob, walk)
PyObject* verify(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        int32_t method;
        void* stream;
        Rows r;
        if (n != 2 + kRowArgs + 6 || !number(a[0], method) || !stream_of(a[1], stream) || a[2] == Py_None ||
            !rows_of(a + 2, r))
            Py_RETURN_NONE;
        a += 2 + kRowArgs;
        const at::Tensor *tokens = plain(a[0], at::kInt, {r.B, r.N}),
                         *u = plain(a[1], at::kFloat, {r.B, r.N, (int64_t)r.pb.k + 1});
        if (!tokens || !u || r.pb.depth < 0) Py_RETURN_NONE;
        for (int i = 2; i < 6; ++i)
            if (!PyBool_Check(a[i])) Py_RETURN_NONE;
        Outputs out;
        mdsd_result res = {};
        const at::TensorOptions ints = r.draft.options().dtype(at::kInt), floats = ints.dtype(at::kFloat);
        res.outcome = (int32_t*)out.add("outcome", {r.B, r.N}, ints);
        res.token = (int32_t*)out.add("token", {r.B, r.N}, ints);
        if (a[2] == Py_True) res.resid_mass = (float*)out.add("resid_mass", {r.B, r.N}, floats);
        if (a[3] == Py_True) res.flags = (int32_t*)out.add("flags", {r.B, r.N}, ints);
        if (a[4] == Py_True) res.resid_prob = (float*)out.add("resid_prob", {r.B, r.N, r.V}, floats);
        if (a[5] == Py_True) {
            res.accept_depth = (int32_t*)out.add("accept_depth", {r.B}, ints);
            res.emitted = (int32_t*)out.add("emitted", {r.B, r.pb.depth}, ints);
        }
        const int32_t* tp = (const int32_t*)tokens->data_ptr();
        const float* up = (const float*)u->data_ptr();
        decltype(&spechub_verify) call[] = {spechub_verify,      rrs_verify,      rrsw_verify,
                                            spechub_verify_path, rrs_verify_path, rrsw_verify_path};
        if (method < 0 || method > 5) Py_RETURN_NONE;
        int rc;
        Py_BEGIN_ALLOW_THREADS;
        rc = call[method](&r.pb, tp, up, &res, nullptr, 0, stream);
        Py_END_ALLOW_THREADS;
        return out.answer(rc);
    });
}

PyMethodDef methods[] = {
    {"draft", (PyCFunction)(void (*)(void))draft, METH_FASTCALL, nullptr},
    {"verify", (PyCFunction)(void (*)(void))verify, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host(void) { return PyModule_Create(&module); }
