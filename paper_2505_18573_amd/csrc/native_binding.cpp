// The binding's hot calls without Python between the tensors and libe3.so.  A call of a few microseconds on the GPU took as
// long in Python: about 0.7 us per checked tensor, 0.8 to 1.4 us per foreign call, 1.1 us per allocated output.
// One pass among others, in Python / here: 64 x 8 advantages 5.7 / 3.6 us (the kernel 2.9), the objective of 512
// rollouts 11.6 / 9.4 us (its kernels 8.9), a step of 512 rows, whose host work lies between two launches, 72.9 / 69.8 us,
// log-probs with the measured gap of 1 row x 1000 16.5 / 10.9.
//
// Every function takes the arguments of the Python function it serves, and does what that does when they are ordinary: plain
// torch tensors of the right type, size and device, Python ints and floats.  It returns the outputs; or the
// library's status if that is not E3_OK; or None, with nothing done, for arguments that are not ordinary, which
// binding.py then treats itself: errors are found and worded in one place.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/util/Exception.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/e3.h"

namespace {

// Entry points of the library that binding.py has loaded, and torch's handle of the current stream.
decltype(&e3_grpo_advantages) p_advantages;
decltype(&e3_grpo_objective) p_objective;
decltype(&e3_workspace_bytes) p_workspace_bytes;
decltype(&e3_sample_entropy) p_sample;
decltype(&e3_restricted_workspace_bytes) p_restricted_bytes;
decltype(&e3_sample_restricted_ws) p_restricted;
decltype(&e3_logprob_entropy_advantages) p_logprob;
decltype(&e3_logprob_entropy_gap) p_gap;
decltype(&e3_temperature_update) p_temperature;
PyObject* raw_stream = nullptr;

// A call's arguments as they are read: `ok` falls at the first one that is not ordinary.
struct Reader {
    bool ok = true;
    at::Device dev = at::Device(at::kCPU);

    const at::Tensor* plain(PyObject* o)
    {
        if (!ok || !THPVariable_CheckExact(o)) { ok = false; return nullptr; }
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.defined() || t.layout() != at::kStrided || !t.has_storage() || t.is_neg()
            || t.key_set().has(c10::DispatchKey::Python)) { ok = false; return nullptr; }
        return &t;
    }
    // the vector that names the device
    const at::Tensor* first(PyObject* o)
    {
        const at::Tensor* t = plain(o);
        if (t == nullptr || !t->is_cuda()) { ok = false; return nullptr; }
        dev = t->device();
        return t;
    }
    // a vector of n elements, or None
    void* vector(PyObject* o, at::ScalarType type, int64_t n)
    {
        if (o == Py_None) return nullptr;
        const at::Tensor* t = plain(o);
        if (t == nullptr || t->scalar_type() != type || t->dim() != 1 || t->size(0) != n || !t->is_contiguous()
            || t->device() != dev) { ok = false; return nullptr; }
        return t->data_ptr();
    }
    // one element, also in pinned host memory
    void* scalar(PyObject* o, at::ScalarType type)
    {
        if (o == Py_None) return nullptr;
        const at::Tensor* t = plain(o);
        if (t == nullptr || t->scalar_type() != type || t->dim() != 1 || t->size(0) != 1
            || (t->device() != dev && !(t->is_cpu() && t->is_pinned()))) { ok = false; return nullptr; }
        return t->data_ptr();
    }
    int64_t integer(PyObject* o)
    {
        if (!PyLong_CheckExact(o)) { ok = false; return 0; }
        int overflow = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
        if (overflow != 0) ok = false;
        return v;
    }
    int32_t integer32(PyObject* o)
    {
        const int64_t v = integer(o);
        if (v != (int32_t)v) ok = false;
        return (int32_t)v;
    }
    uint64_t word(PyObject* o)                                    // modulo 2^64
    {
        if (!PyLong_CheckExact(o)) { ok = false; return 0; }
        return PyLong_AsUnsignedLongLongMask(o);
    }
    double number(PyObject* o)
    {
        if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
        return (double)integer(o);
    }
    void* stream()
    {
        PyObject* index = PyLong_FromLong(dev.index());
        PyObject* s = index ? PyObject_CallOneArg(raw_stream, index) : nullptr;
        Py_XDECREF(index);
        void* p = s ? PyLong_AsVoidPtr(s) : nullptr;
        Py_XDECREF(s);
        if (PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return p;
    }
};

struct Logits {
    const void* p = nullptr;
    int dtype = 0;
    int64_t rows = 0, V = 0, pitch = 0;
    Logits(Reader& r, PyObject* o)
    {
        const at::Tensor* t = r.first(o);
        if (t == nullptr || t->dim() != 2) { r.ok = false; return; }
        if (t->scalar_type() == at::kBFloat16) dtype = E3_BF16;
        else if (t->scalar_type() == at::kFloat) dtype = E3_F32;
        else { r.ok = false; return; }
        rows = t->size(0); V = t->size(1);
        if (V > 1 && t->stride(1) != 1) { r.ok = false; return; }
        pitch = rows > 1 ? t->stride(0) : std::max(V, t->stride(0));
        p = t->data_ptr();
    }
};

// An output: the caller's tensor, or one of n elements.
struct Output {
    PyObject* object = nullptr;
    void* p = nullptr;
    Output() = default;
    Output(const Output&) = delete;
    ~Output() { Py_XDECREF(object); }
    void make(Reader& r, at::ScalarType type, int64_t n)
    {
        if (!r.ok) return;
        const at::Tensor t = at::empty({n}, at::TensorOptions().dtype(type).device(r.dev));
        p = t.data_ptr();
        object = THPVariable_Wrap(t);
        if (object == nullptr) { PyErr_Clear(); r.ok = false; }
    }
    void take(PyObject* given) { Py_INCREF(given); object = given; }
    void take_or_make(Reader& r, PyObject* given, at::ScalarType type, int64_t n)
    {
        if (given == Py_None) return make(r, type, n);
        p = r.vector(given, type, n);
        take(given);
    }
    PyObject* release() { PyObject* o = object; object = nullptr; return o; }
};

// The vocabulary pass's workspace argument: a tensor, None (allocate what is needed) or False (none).
struct Workspace {
    at::Tensor own;
    void* p = nullptr;
    size_t bytes = 0;
    void make(Reader& r, size_t need)
    {
        if (!r.ok || need == 0) return;
        own = at::empty({(int64_t)need}, at::TensorOptions().dtype(at::kByte).device(r.dev));
        p = own.data_ptr();
        bytes = need;
    }
    Workspace(Reader& r, PyObject* o, int64_t rows, int64_t V)
    {
        if (o == Py_False) return;
        if (o == Py_None) { make(r, p_workspace_bytes(rows, V)); return; }
        const at::Tensor* t = r.plain(o);
        if (t == nullptr) return;
        p = t->data_ptr();
        bytes = (size_t)t->numel() * t->element_size();
    }
    // The restricted sampler's: None allocates what is needed where `may_allocate`, and goes without where the memory is not there.
    Workspace(Reader& r, PyObject* o, size_t need, bool may_allocate)
    {
        if (o == Py_False) return;
        if (o == Py_None) {
            if (!may_allocate) return;
            try { make(r, need); } catch (const c10::OutOfMemoryError&) { own = at::Tensor(); p = nullptr; bytes = 0; }
            return;
        }
        const at::Tensor* t = r.plain(o);
        if (t == nullptr || t->device() != r.dev || !t->is_contiguous()) { r.ok = false; return; }
        p = t->data_ptr();
        bytes = (size_t)t->numel() * t->element_size();
    }
};

PyObject* unusual() { Py_RETURN_NONE; }

template <typename Call, typename Done>
PyObject* run(Reader& r, Call&& call, Done&& done)
{
    void* const stream = r.ok ? r.stream() : nullptr;
    if (!r.ok) return unusual();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call(stream);
    Py_END_ALLOW_THREADS
    return rc == E3_OK ? done() : PyLong_FromLong(rc);
}

// C++ errors (an allocation that fails) leave the call to binding.py, which meets them again and reports them.
template <typename F>
PyObject* guarded(F&& f)
{
    try { return f(); } catch (...) { PyErr_Clear(); return unusual(); }
}

// rewards, group_offsets, ddof, eps, adv_out
PyObject* advantages(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    if (n_args != 5) return unusual();
    return guarded([&]() -> PyObject* {
        Reader r;
        const at::Tensor* rewards = r.first(a[0]);
        const at::Tensor* offsets = r.ok ? r.plain(a[1]) : nullptr;
        if (!r.ok || rewards->dim() != 1 || offsets->dim() != 1) return unusual();
        const int64_t n = rewards->size(0), groups = offsets->size(0) - 1;
        const void* pr = r.vector(a[0], at::kFloat, n);
        const void* po = r.vector(a[1], at::kInt, groups + 1);
        const int32_t ddof = r.integer32(a[2]);
        const double eps = r.number(a[3]);
        if (groups != (int32_t)groups) return unusual();
        Output adv;
        adv.take_or_make(r, a[4], at::kFloat, n);
        return run(r, [&](void* s) { return p_advantages((const float*)pr, (const int32_t*)po, (int32_t)groups, ddof, (float)eps, (float*)adv.p, s); },
                   [&] { return adv.release(); });
    });
}

// logp_new, logp_old, seq_offsets, adv, group_offsets, clip_eps, want_token_terms
PyObject* objective(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    if (n_args != 7 || !PyBool_Check(a[6])) return unusual();
    return guarded([&]() -> PyObject* {
        Reader r;
        const at::Tensor* logp = r.first(a[0]);
        const at::Tensor* adv = r.ok ? r.plain(a[3]) : nullptr;
        const at::Tensor* groups = r.ok ? r.plain(a[4]) : nullptr;
        if (!r.ok || logp->dim() != 1 || adv->dim() != 1 || groups->dim() != 1) return unusual();
        const int64_t T = logp->size(0), N = adv->size(0), B = groups->size(0) - 1;
        if (N != (int32_t)N || B != (int32_t)B) return unusual();
        const void* p_new = r.vector(a[0], at::kFloat, T);
        const void* p_old = a[1] == Py_None ? (r.ok = false, nullptr) : r.vector(a[1], at::kFloat, T);
        const void* p_seq = a[2] == Py_None ? (r.ok = false, nullptr) : r.vector(a[2], at::kInt, N + 1);
        const void* p_adv = r.vector(a[3], at::kFloat, N);
        const void* p_grp = r.vector(a[4], at::kInt, B + 1);
        const double clip = r.number(a[5]);
        Output J, mean, terms;
        if (a[6] == Py_True) terms.make(r, at::kFloat, T);
        else terms.take(Py_None);
        mean.make(r, at::kDouble, N);
        J.make(r, at::kDouble, 1);
        return run(r, [&](void* s) {
                       return p_objective((const float*)p_new, (const float*)p_old, (const int32_t*)p_seq, (const float*)p_adv, (int32_t)N,
                                          (const int32_t*)p_grp, (int32_t)B, (float)clip, (float*)terms.p, (double*)mean.p, (double*)J.p, s);
                   },
                   [&] { return PyTuple_Pack(3, J.object, mean.object, terms.object); });
    });
}

// logits, tau_rows, tau_scalar, seed, row_base, token_out, logp_out, entropy_out, workspace
PyObject* sample(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    if (n_args != 9) return unusual();
    return guarded([&]() -> PyObject* {
        Reader r;
        const Logits l(r, a[0]);
        const void* tau = r.vector(a[1], at::kFloat, l.rows);
        const double tau_scalar = r.number(a[2]);
        const uint64_t seed = r.word(a[3]), row_base = r.word(a[4]);
        if (!r.ok) return unusual();
        Output token, logp, entropy;
        token.take_or_make(r, a[5], at::kInt, l.rows);
        logp.take_or_make(r, a[6], at::kFloat, l.rows);
        entropy.take_or_make(r, a[7], at::kFloat, l.rows);
        const Workspace ws(r, a[8], l.rows, l.V);
        return run(r, [&](void* s) {
                       return p_sample(l.p, l.dtype, l.rows, l.V, l.pitch, (const float*)tau, (float)tau_scalar, seed, row_base,
                                       (int32_t*)token.p, (float*)logp.p, (float*)entropy.p, ws.p, ws.bytes, s);
                   },
                   [&] { return PyTuple_Pack(3, token.object, logp.object, entropy.object); });
    });
}

// logits, tau_rows, tau_scalar, top_k, top_p, seed, row_base, token_out, logp_out, kept_out, workspace
PyObject* restricted(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    if (n_args != 11) return unusual();
    return guarded([&]() -> PyObject* {
        Reader r;
        const Logits l(r, a[0]);
        const void* tau = r.vector(a[1], at::kFloat, l.rows);
        const double tau_scalar = r.number(a[2]);
        const int32_t top_k = r.integer32(a[3]);
        const double top_p = r.number(a[4]);
        const uint64_t seed = r.word(a[5]), row_base = r.word(a[6]);
        if (!r.ok) return unusual();
        Output token, logp, kept;
        token.take_or_make(r, a[7], at::kInt, l.rows);
        logp.take_or_make(r, a[8], at::kFloat, l.rows);
        kept.take_or_make(r, a[9], at::kInt, l.rows);
        const bool may_allocate = a[7] == Py_None || a[8] == Py_None || a[9] == Py_None;
        const Workspace ws(r, a[10], p_restricted_bytes(l.dtype, l.rows, l.V, top_k), may_allocate);
        return run(r, [&](void* s) {
                       return p_restricted(l.p, l.dtype, l.rows, l.V, l.pitch, (const float*)tau, (float)tau_scalar, top_k, (float)top_p, seed,
                                           row_base, (int32_t*)token.p, (float*)logp.p, (int32_t*)kept.p, ws.p, ws.bytes, s);
                   },
                   [&] { return PyTuple_Pack(3, token.object, logp.object, kept.object); });
    });
}

// logits, target_ids, row_mask, tau_rows, tau_scalar, rewards, group_offsets, ddof, eps, logp_out, entropy_out,
// entropy_sum_out, entropy_count_out, adv_out, workspace, want_sum; rewards None: no advantages
PyObject* logprob(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    if (n_args != 16 || !PyBool_Check(a[15])) return unusual();
    return guarded([&]() -> PyObject* {
        Reader r;
        const Logits l(r, a[0]);
        const void* target = r.vector(a[1], at::kInt, l.rows);
        const void* mask = r.vector(a[2], at::kByte, l.rows);
        const void* tau = r.vector(a[3], at::kFloat, l.rows);
        const double tau_scalar = r.number(a[4]);
        if (!r.ok) return unusual();
        int64_t n = 0, groups = 0;
        const bool with_groups = a[5] != Py_None;
        const void *rewards = nullptr, *offsets = nullptr;
        if (with_groups) {
            const at::Tensor *tr = r.plain(a[5]), *to = r.ok ? r.plain(a[6]) : nullptr;
            if (!r.ok || tr->dim() != 1 || to->dim() != 1) return unusual();
            n = tr->size(0); groups = to->size(0) - 1;
            rewards = r.vector(a[5], at::kFloat, n);
            offsets = r.vector(a[6], at::kInt, groups + 1);
            if (groups != (int32_t)groups) return unusual();
        }
        const int32_t ddof = r.integer32(a[7]);
        const double eps = r.number(a[8]);
        Output logp, entropy, sum, count, adv;
        if (a[9] == Py_None && a[1] == Py_None) logp.take(Py_None);
        else logp.take_or_make(r, a[9], at::kFloat, l.rows);
        entropy.take_or_make(r, a[10], at::kFloat, l.rows);
        const bool want_sum = a[15] == Py_True;
        auto sum_out = [&](Output& o, PyObject* given, at::ScalarType type) {
            if (given == Py_None && want_sum) return o.make(r, type, 1);
            o.p = r.scalar(given, type);
            o.take(given);
        };
        sum_out(sum, a[11], at::kDouble);
        sum_out(count, a[12], at::kLong);
        if (with_groups) adv.take_or_make(r, a[13], at::kFloat, n);
        const Workspace ws(r, a[14], l.rows, l.V);
        return run(r, [&](void* s) {
                       return p_logprob(l.p, l.dtype, l.rows, l.V, l.pitch, (const int32_t*)target, (const uint8_t*)mask, (const float*)tau,
                                        (float)tau_scalar, (float*)logp.p, (float*)entropy.p, (double*)sum.p, (int64_t*)count.p,
                                        (const float*)rewards, (const int32_t*)offsets, (int32_t)groups, ddof, (float)eps, (float*)adv.p,
                                        ws.p, ws.bytes, s);
                   },
                   [&] {
                       return with_groups ? PyTuple_Pack(5, logp.object, entropy.object, sum.object, count.object, adv.object)
                                          : PyTuple_Pack(4, logp.object, entropy.object, sum.object, count.object);
                   });
    });
}

// logits, target_ids, row_mask, tau_rows, tau_scalar, workspace
PyObject* logprob_gap(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    if (n_args != 6) return unusual();
    return guarded([&]() -> PyObject* {
        Reader r;
        const Logits l(r, a[0]);
        const void* target = r.vector(a[1], at::kInt, l.rows);
        const void* mask = r.vector(a[2], at::kByte, l.rows);
        const void* tau = r.vector(a[3], at::kFloat, l.rows);
        const double tau_scalar = r.number(a[4]);
        if (!r.ok) return unusual();
        Output logp, entropy, gap, sum, gap_sum, count;
        if (a[1] == Py_None) logp.take(Py_None);
        else logp.make(r, at::kFloat, l.rows);
        entropy.make(r, at::kFloat, l.rows);
        gap.make(r, at::kFloat, l.rows);
        sum.make(r, at::kDouble, 1);
        gap_sum.make(r, at::kDouble, 1);
        count.make(r, at::kLong, 1);
        const Workspace ws(r, a[5], l.rows, l.V);
        return run(r, [&](void* s) {
                       return p_gap(l.p, l.dtype, l.rows, l.V, l.pitch, (const int32_t*)target, (const uint8_t*)mask, (const float*)tau,
                                    (float)tau_scalar, (float*)logp.p, (float*)entropy.p, (float*)gap.p, (double*)sum.p, (double*)gap_sum.p,
                                    (int64_t*)count.p, ws.p, ws.bytes, s);
                   },
                   [&] { return PyTuple_Pack(6, logp.object, entropy.object, gap.object, sum.object, gap_sum.object, count.object); });
    });
}

// tau_t, H_t, H_init, vocab, t, t_anneal, t_max, eta, tau_min, tau_max
PyObject* temperature(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    if (n_args != 10) return unusual();
    Reader r;
    const double tau = r.number(a[0]), H = r.number(a[1]), H0 = r.number(a[2]);
    const int64_t vocab = r.integer(a[3]), t = r.integer(a[4]), t_anneal = r.integer(a[5]), t_max = r.integer(a[6]);
    const double eta = r.number(a[7]), lo = r.number(a[8]), hi = r.number(a[9]);
    if (!r.ok) return unusual();
    double next = 0.0, target = 0.0;
    const int rc = p_temperature(tau, H, H0, vocab, t, t_anneal, t_max, eta, lo, hi, &next, &target);
    return rc == E3_OK ? Py_BuildValue("dd", next, target) : PyLong_FromLong(rc);
}

// The library's entry points by name (a dict of addresses), and torch's handle of the current stream.
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    if (n_args != 2 || !PyDict_Check(a[0]) || !PyCallable_Check(a[1])) {
        PyErr_SetString(PyExc_TypeError, "bind(addresses, current_raw_stream)");
        return nullptr;
    }
    bool all = true;
    auto get = [&](const char* name, auto& to) {
        PyObject* v = PyDict_GetItemString(a[0], name);
        void* p = v && PyLong_Check(v) ? PyLong_AsVoidPtr(v) : nullptr;
        if (p == nullptr) all = false;
        to = reinterpret_cast<std::remove_reference_t<decltype(to)>>(p);
    };
    get("e3_grpo_advantages", p_advantages);
    get("e3_grpo_objective", p_objective);
    get("e3_workspace_bytes", p_workspace_bytes);
    get("e3_sample_entropy", p_sample);
    get("e3_restricted_workspace_bytes", p_restricted_bytes);
    get("e3_sample_restricted_ws", p_restricted);
    get("e3_logprob_entropy_advantages", p_logprob);
    get("e3_logprob_entropy_gap", p_gap);
    get("e3_temperature_update", p_temperature);
    if (!all) { PyErr_SetString(PyExc_ValueError, "an entry point is missing"); return nullptr; }
    Py_INCREF(a[1]);
    Py_XSETREF(raw_stream, a[1]);
    Py_RETURN_NONE;
}

template <typename F>
constexpr PyCFunction fast(F* f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }

PyMethodDef methods[] = {
    {"bind", fast(bind), METH_FASTCALL, nullptr},
    {"advantages", fast(advantages), METH_FASTCALL, nullptr},
    {"objective", fast(objective), METH_FASTCALL, nullptr},
    {"sample", fast(sample), METH_FASTCALL, nullptr},
    {"restricted", fast(restricted), METH_FASTCALL, nullptr},
    {"logprob", fast(logprob), METH_FASTCALL, nullptr},
    {"logprob_advantages", fast(logprob), METH_FASTCALL, nullptr},
    {"logprob_gap", fast(logprob_gap), METH_FASTCALL, nullptr},
    {"temperature", fast(temperature), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
