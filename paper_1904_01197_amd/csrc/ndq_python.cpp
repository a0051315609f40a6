// Native half of the Python binding: argument marshalling between torch tensors and the
// C ABI (include/ndq.h).  A call made through ctypes costs 7 us of host time before its
// first launch plus 2.5 us per worker it names (2.4 us is a launch); reading the tensors
// here costs a few tens of nanoseconds each.
//
// The functions check what the binding promises (contiguous device tensors, types, sizes),
// call the library on torch's current stream and return its status; ndq.py turns a status
// into an exception.  The library's entry points arrive as addresses (bind()), so that
// whatever build ndq.py has loaded is the one that is called.  Nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <memory>

#include "ndq.h"

namespace {

struct Library {
    decltype(&ndq_code_bits) code_bits;
    decltype(&ndq_packed_bytes) packed_bytes;
    decltype(&ndq_num_buckets) num_buckets;
    decltype(&ndq_absmax) absmax;
    decltype(&ndq_dq_encode) dq_encode;
    decltype(&ndq_dq_encode_with_step) dq_encode_with_step;
    decltype(&ndq_nested_encode) nested_encode;
    decltype(&ndq_nested_encode_with_step) nested_encode_with_step;
    decltype(&ndq_encode_workers) encode_workers;
    decltype(&ndq_encode_check) encode_check;
    decltype(&ndq_dq_decode) dq_decode;
    decltype(&ndq_dq_decode_half) dq_decode_half;
    decltype(&ndq_nested_decode) nested_decode;
    decltype(&ndq_aggregate) aggregate;
    decltype(&ndq_decode_chain) decode_chain;
    decltype(&ndq_decode_mean) decode_mean;
    decltype(&ndq_code_entropy) code_entropy;
    decltype(&ndq_dense_pack) dense_pack;
    decltype(&ndq_dense_unpack) dense_unpack;
    decltype(&ndq_dense_bytes) dense_bytes;
    decltype(&ndq_sqdiff) sqdiff;
    decltype(&ndq_sqdiff_static) sqdiff_static;
};
Library lib = {};
PyObject* dither_type = nullptr;       // ctypes mirror of ndq_dither
PyObject* get_device = nullptr;        // torch's current device, and its current stream there
PyObject* get_raw_stream = nullptr;

struct Failed {};      // a Python exception is set

[[noreturn]] void fail(PyObject* type, const char* text)
{
    PyErr_SetString(type, text);
    throw Failed();
}

const at::Tensor& tensor(PyObject* o, const char* what)
{
    if (THPVariable_Check(o)) {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (t.is_cuda() && t.is_contiguous()) return t;
    }
    PyErr_Format(PyExc_TypeError, "%s must be a contiguous CUDA tensor", what);
    throw Failed();
}
void* address(const at::Tensor& t) { return t.data_ptr(); }
size_t count(const at::Tensor& t) { return (size_t)t.numel(); }
bool is_f32(const at::Tensor& t) { return t.scalar_type() == at::kFloat; }
bool is_f64(const at::Tensor& t) { return t.scalar_type() == at::kDouble; }

int gradient_type(const at::Tensor& t)
{
    if (t.scalar_type() == at::kFloat) return NDQ_F32;
    if (t.scalar_type() == at::kBFloat16) return NDQ_BF16;
    fail(PyExc_TypeError, "gradient must be float32 or bfloat16");
}

uint64_t integer(PyObject* o)
{
    PyObject* i = PyNumber_Index(o);
    if (!i) throw Failed();
    const uint64_t v = PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    if (v == (uint64_t)-1 && PyErr_Occurred()) throw Failed();
    return v;
}
float real(PyObject* o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Failed();
    return (float)v;
}
bool truth(PyObject* o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Failed();
    return v != 0;
}
ndq_dither dither(PyObject* o)
{
    ndq_dither d;
    Py_buffer view;
    const int is = PyObject_IsInstance(o, dither_type);
    if (is < 0) throw Failed();
    if (!is) fail(PyExc_TypeError, "expected an ndq_dither");
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Failed();
    const bool fits = (size_t)view.len == sizeof(d);
    if (fits) memcpy(&d, view.buf, sizeof(d));
    PyBuffer_Release(&view);
    if (!fits) fail(PyExc_TypeError, "expected an ndq_dither");
    return d;
}

// A worker's message may also carry its dither as a tuple of the fields (missing ones are 0).
ndq_dither dither_or_fields(PyObject* o)
{
    if (!PyTuple_Check(o)) return dither(o);
    PyObject* made = PyObject_Call(dither_type, o, nullptr);
    if (!made) throw Failed();
    ndq_dither d;
    try {
        d = dither(made);
    } catch (...) {
        Py_DECREF(made);
        throw;
    }
    Py_DECREF(made);
    return d;
}

void* current_stream()
{
    PyObject* device = PyObject_CallNoArgs(get_device);
    if (!device) throw Failed();
    PyObject* stream = PyObject_CallOneArg(get_raw_stream, device);
    Py_DECREF(device);
    if (!stream) throw Failed();
    void* s = PyLong_AsVoidPtr(stream);
    Py_DECREF(stream);
    if (!s && PyErr_Occurred()) throw Failed();
    return s;
}

// a sequence argument held as a fast sequence
class Sequence {
public:
    explicit Sequence(PyObject* o) : seq_(PySequence_Fast(o, "expected a sequence"))
    {
        if (!seq_) throw Failed();
    }
    ~Sequence() { Py_XDECREF(seq_); }
    Sequence(const Sequence&) = delete;
    Sequence& operator=(const Sequence&) = delete;
    size_t size() const { return (size_t)PySequence_Fast_GET_SIZE(seq_); }
    PyObject* operator[](size_t i) const { return PySequence_Fast_GET_ITEM(seq_, i); }
private:
    PyObject* seq_;
};

// up to N entries on the stack, more on the heap
template <class T, size_t N> class Few {
public:
    explicit Few(size_t n) : data_(here_)
    {
        if (n > N) { heap_.reset(new T[n]); data_ = heap_.get(); }
    }
    T& operator[](size_t i) { return data_[i]; }
    T* data() { return data_; }
private:
    T here_[N];
    std::unique_ptr<T[]> heap_;
    T* data_;
};

void check_outputs(size_t n, uint32_t bits, uint32_t bucket, const at::Tensor& codes, const at::Tensor& steps)
{
    if (codes.nbytes() < lib.packed_bytes(n, bits)) fail(PyExc_ValueError, "codes_out too small");
    if (count(steps) < lib.num_buckets(n, bucket)) fail(PyExc_ValueError, "steps_out too small");
}

// A worker's message must be as large as the call will read.
void check_message(const at::Tensor& codes, const at::Tensor& steps, size_t n, uint32_t bits, uint32_t bucket)
{
    if (codes.nbytes() < lib.packed_bytes(n, bits))
        fail(PyExc_ValueError, "codes hold fewer than ndq_packed_bytes(n, bits) bytes");
    if (!is_f32(steps) || count(steps) < lib.num_buckets(n, bucket))
        fail(PyExc_ValueError, "steps must hold ndq_num_buckets(n, bucket) float32");
}

const float* one_step(PyObject* o)
{
    const at::Tensor& t = tensor(o, "step_in");
    if (!is_f32(t) || count(t) < 1u) fail(PyExc_ValueError, "step_in must hold one float32");
    return (const float*)address(t);
}

void check_values(const at::Tensor& out, size_t n, const char* text)
{
    if (!is_f32(out) || count(out) < n) fail(PyExc_ValueError, text);
}

// The GIL is released while the library enqueues, as ctypes does.  Only the library's C function
// may run here: whatever can throw (reading a tensor's address does, for a tensor without
// storage) belongs before it, and is done while the GIL is held.
class WithoutGil {
public:
    WithoutGil() : state_(PyEval_SaveThread()) {}
    ~WithoutGil() { PyEval_RestoreThread(state_); }
    WithoutGil(const WithoutGil&) = delete;
    WithoutGil& operator=(const WithoutGil&) = delete;
private:
    PyThreadState* state_;
};
template <class R, class... P, class... A> PyObject* status(R (*function)(P...), A... arguments)
{
    R rc;
    {
        WithoutGil released;
        rc = function(arguments...);
    }
    return PyLong_FromLong(rc);
}

template <class F> PyObject* guarded(F body)
{
    if (!lib.absmax) {
        PyErr_SetString(PyExc_RuntimeError, "the library is not loaded");
        return nullptr;
    }
    try {
        return body();
    } catch (const Failed&) {
        return nullptr;
    } catch (...) {
        torch::translate_exception_to_python(std::current_exception());    // as torch's own functions do
        return nullptr;
    }
}

#define NDQ_METHOD(name, arity)                                                          \
    PyObject* name##_body(PyObject* const* v);                                           \
    PyObject* name(PyObject*, PyObject* const* v, Py_ssize_t n)                          \
    {                                                                                    \
        if (n != (arity)) {                                                              \
            PyErr_Format(PyExc_TypeError, #name " takes %d arguments", (int)(arity));   \
            return nullptr;                                                              \
        }                                                                                \
        return guarded([&] { return name##_body(v); });                                  \
    }                                                                                    \
    PyObject* name##_body(PyObject* const* v)

// g, bucket, kappa_out
NDQ_METHOD(absmax, 3)
{
    const at::Tensor &g = tensor(v[0], "g"), &out = tensor(v[2], "kappa_out");
    const int dt = gradient_type(g);
    const size_t n = count(g);
    const uint32_t bucket = (uint32_t)integer(v[1]);
    void* s = current_stream();
    return status(lib.absmax, address(g), dt, n, bucket, (float*)address(out), s);
}

// g, delta, levels, bucket, d, codes_out, steps_out
NDQ_METHOD(dq_encode, 7)
{
    const at::Tensor &g = tensor(v[0], "g"), &codes = tensor(v[5], "codes_out"), &steps = tensor(v[6], "steps_out");
    const int dt = gradient_type(g);
    const size_t n = count(g);
    const float delta = real(v[1]);
    const uint32_t levels = (uint32_t)integer(v[2]), bucket = (uint32_t)integer(v[3]);
    const ndq_dither d = dither(v[4]);
    check_outputs(n, lib.code_bits(levels), bucket, codes, steps);
    void* s = current_stream();
    return status(lib.dq_encode, address(g), dt, n, delta, levels, bucket, &d, address(codes),
                  (float*)address(steps), s);
}

// g, step_in, levels, d, codes_out, steps_out
NDQ_METHOD(dq_encode_with_step, 6)
{
    const at::Tensor &g = tensor(v[0], "g"), &codes = tensor(v[4], "codes_out"), &steps = tensor(v[5], "steps_out");
    const int dt = gradient_type(g);
    const size_t n = count(g);
    const float* step_in = one_step(v[1]);
    const uint32_t levels = (uint32_t)integer(v[2]);
    const ndq_dither d = dither(v[3]);
    check_outputs(n, lib.code_bits(levels), 0u, codes, steps);
    void* s = current_stream();
    return status(lib.dq_encode_with_step, address(g), dt, n, step_in, levels, &d, address(codes),
                  (float*)address(steps), s);
}

// g, delta, levels, M, alpha, bucket, d, codes_out, steps_out
NDQ_METHOD(nested_encode, 9)
{
    const at::Tensor &g = tensor(v[0], "g"), &codes = tensor(v[7], "codes_out"), &steps = tensor(v[8], "steps_out");
    const int dt = gradient_type(g);
    const size_t n = count(g);
    const float delta = real(v[1]), alpha = real(v[4]);
    const uint32_t levels = (uint32_t)integer(v[2]), M = (uint32_t)integer(v[3]), bucket = (uint32_t)integer(v[5]);
    const ndq_dither d = dither(v[6]);
    check_outputs(n, lib.code_bits(M), bucket, codes, steps);
    void* s = current_stream();
    return status(lib.nested_encode, address(g), dt, n, delta, levels, M, alpha, bucket, &d, address(codes),
                  (float*)address(steps), s);
}

// g, step_in, M, alpha, d, codes_out, steps_out
NDQ_METHOD(nested_encode_with_step, 7)
{
    const at::Tensor &g = tensor(v[0], "g"), &codes = tensor(v[5], "codes_out"), &steps = tensor(v[6], "steps_out");
    const int dt = gradient_type(g);
    const size_t n = count(g);
    const float* step_in = one_step(v[1]);
    const uint32_t M = (uint32_t)integer(v[2]);
    const float alpha = real(v[3]);
    const ndq_dither d = dither(v[4]);
    check_outputs(n, lib.code_bits(M), 0u, codes, steps);
    void* s = current_stream();
    return status(lib.nested_encode_with_step, address(g), dt, n, step_in, M, alpha, &d, address(codes),
                  (float*)address(steps), s);
}

// jobs of (g, kind, levels, M, alpha, d, codes_out, steps_out, step_in or None), delta, bucket.
// A library call takes vectors of one length and type, and a handed-over step belongs to the
// whole vector whatever the bucket: consecutive jobs that agree in these share a call.
struct EncodeCall { size_t first, jobs, n; int dt; uint32_t bucket; };
int encode_calls(const ndq_encode_job* jobs, const EncodeCall* calls, size_t num_calls, float delta, void* s)
{
    int rc = NDQ_OK;
    // a call checks its own jobs before it enqueues; several have to be checked before the first does
    for (size_t c = 0; c < num_calls && rc == NDQ_OK && num_calls > 1u; ++c)
        rc = lib.encode_check(jobs + calls[c].first, (uint32_t)calls[c].jobs, calls[c].dt, calls[c].n, delta,
                              calls[c].bucket);
    for (size_t c = 0; c < num_calls && rc == NDQ_OK; ++c)
        rc = lib.encode_workers(jobs + calls[c].first, (uint32_t)calls[c].jobs, calls[c].dt, calls[c].n, delta,
                                calls[c].bucket, s);
    return rc;
}
NDQ_METHOD(encode_workers, 3)
{
    Sequence jobs(v[0]);
    const size_t W = jobs.size();
    if (W == 0u) fail(PyExc_ValueError, "no jobs");
    const float delta = real(v[1]);
    const uint32_t bucket = (uint32_t)integer(v[2]);
    Few<ndq_encode_job, 32> list(W);
    Few<EncodeCall, 4> calls(W);
    size_t num_calls = 0;
    constexpr size_t kMaxJobs = 1024;      // of the library call
    for (size_t w = 0; w < W; ++w) {
        Sequence f(jobs[w]);
        if (f.size() != 9u) fail(PyExc_ValueError, "a job has nine entries");
        const at::Tensor &g = tensor(f[0], "g"), &codes = tensor(f[6], "codes_out"), &steps = tensor(f[7], "steps_out");
        ndq_encode_job& job = list[w];
        job.kind = (uint32_t)integer(f[1]);
        job.levels = (uint32_t)integer(f[2]);
        job.M = (uint32_t)integer(f[3]);
        job.alpha = real(f[4]);
        job.dither = dither(f[5]);
        job.g = address(g);
        job.codes_out = address(codes);
        job.steps_out = (float*)address(steps);
        job.step_in = f[8] == Py_None ? nullptr : one_step(f[8]);
        const size_t n = count(g);
        const int dt = gradient_type(g);
        const uint32_t job_bucket = job.step_in ? 0u : bucket;
        check_outputs(n, lib.code_bits(job.kind == NDQ_WORKER_NESTED ? job.M : job.levels), job_bucket, codes, steps);
        const EncodeCall* last = num_calls ? &calls[num_calls - 1u] : nullptr;
        if (!last || last->n != n || last->dt != dt || last->bucket != job_bucket || last->jobs == kMaxJobs)
            calls[num_calls++] = {w, 0u, n, dt, job_bucket};
        ++calls[num_calls - 1u].jobs;
    }
    void* s = current_stream();
    return status(encode_calls, list.data(), calls.data(), num_calls, delta, s);
}

// codes, n, levels, bucket, steps, d, out, accumulate
NDQ_METHOD(dq_decode, 8)
{
    const size_t n = integer(v[1]);
    const uint32_t levels = (uint32_t)integer(v[2]), bucket = (uint32_t)integer(v[3]);
    const at::Tensor &codes = tensor(v[0], "codes"), &steps = tensor(v[4], "steps"), &out = tensor(v[6], "out");
    const ndq_dither d = dither(v[5]);
    check_message(codes, steps, n, lib.code_bits(levels), bucket);
    check_values(out, n, "out must hold n float32");
    const int add = truth(v[7]);
    void* s = current_stream();
    return status(lib.dq_decode, address(codes), n, levels, bucket, (const float*)address(steps), &d,
                  (float*)address(out), add, s);
}

// codes, n, levels, bucket, steps, out, accumulate
NDQ_METHOD(dq_decode_half, 7)
{
    const size_t n = integer(v[1]);
    const uint32_t levels = (uint32_t)integer(v[2]), bucket = (uint32_t)integer(v[3]);
    const at::Tensor &codes = tensor(v[0], "codes"), &steps = tensor(v[4], "steps"), &out = tensor(v[5], "out");
    check_message(codes, steps, n, lib.code_bits(levels), bucket);
    check_values(out, n, "out must hold n float32");
    const int add = truth(v[6]);
    void* s = current_stream();
    return status(lib.dq_decode_half, address(codes), n, levels, bucket, (const float*)address(steps),
                  (float*)address(out), add, s);
}

// codes, n, M, alpha, bucket, steps, d, side, side_scale, out, accumulate
NDQ_METHOD(nested_decode, 11)
{
    const size_t n = integer(v[1]);
    const uint32_t M = (uint32_t)integer(v[2]), bucket = (uint32_t)integer(v[4]);
    const float alpha = real(v[3]), side_scale = real(v[8]);
    const at::Tensor &codes = tensor(v[0], "codes"), &steps = tensor(v[5], "steps"), &side = tensor(v[7], "side"),
                     &out = tensor(v[9], "out");
    const ndq_dither d = dither(v[6]);
    check_message(codes, steps, n, lib.code_bits(M), bucket);
    check_values(out, n, "out and side must hold n float32");
    check_values(side, n, "out and side must hold n float32");
    const int add = truth(v[10]);
    void* s = current_stream();
    return status(lib.nested_decode, address(codes), n, M, alpha, bucket, (const float*)address(steps), &d,
                  (const float*)address(side), side_scale, (float*)address(out), add, s);
}

// gs, scale, out
NDQ_METHOD(aggregate, 3)
{
    Sequence gs(v[0]);
    const size_t W = gs.size();
    if (W == 0u) fail(PyExc_ValueError, "nothing to sum");
    Few<const float*, 32> list(W);
    size_t n = 0;
    for (size_t w = 0; w < W; ++w) {
        const at::Tensor& g = tensor(gs[w], "gs[w]");
        if (w == 0) n = count(g);
        if (!is_f32(g) || count(g) != n) fail(PyExc_ValueError, "all inputs must be float32 of equal length");
        list[w] = (const float*)address(g);
    }
    const float scale = real(v[1]);
    const at::Tensor& out = tensor(v[2], "out");
    void* s = current_stream();
    return status(lib.aggregate, list.data(), (uint32_t)W, n, scale, (float*)address(out), s);
}

// (codes, steps, kind, levels_or_M, d[, alpha])
ndq_worker worker_message(PyObject* entry, size_t n, uint32_t bucket)
{
    Sequence f(entry);
    if (f.size() < 5u) fail(PyExc_ValueError, "a worker has at least five entries");
    const at::Tensor &codes = tensor(f[0], "codes"), &steps = tensor(f[1], "steps");
    ndq_worker wk;
    wk.kind = (uint32_t)integer(f[2]);
    wk.levels_or_M = (uint32_t)integer(f[3]);
    wk.alpha = f.size() > 5u ? real(f[5]) : 1.0f;
    wk.dither = dither_or_fields(f[4]);
    check_message(codes, steps, n, lib.code_bits(wk.levels_or_M), bucket);
    wk.codes = address(codes);
    wk.steps = (const float*)address(steps);
    return wk;
}

// workers, decoded, n, bucket, scale, out
NDQ_METHOD(decode_mean, 6)
{
    Sequence workers(v[0]), decoded(v[1]);
    const size_t W = workers.size();
    if (decoded.size() != W) fail(PyExc_ValueError, "one decoded vector per worker");
    const size_t n = integer(v[2]);
    const uint32_t bucket = (uint32_t)integer(v[3]);
    const float scale = real(v[4]);
    Few<ndq_worker, 32> list(W);
    Few<float*, 32> values(W);
    for (size_t w = 0; w < W; ++w) {
        list[w] = worker_message(workers[w], n, bucket);
        const at::Tensor& t = tensor(decoded[w], "decoded[w]");
        check_values(t, n, "decoded[w] must hold n float32");
        values[w] = (float*)address(t);
    }
    const at::Tensor& out = tensor(v[5], "out");
    check_values(out, n, "out must hold n float32");
    void* s = current_stream();
    return status(lib.decode_mean, list.data(), values.data(), (uint32_t)W, n, bucket, scale, (float*)address(out),
                  s);
}

// workers, n, bucket, scale, out
NDQ_METHOD(decode_chain, 5)
{
    Sequence workers(v[0]);
    const size_t W = workers.size();
    const size_t n = integer(v[1]);
    const uint32_t bucket = (uint32_t)integer(v[2]);
    const float scale = real(v[3]);
    Few<ndq_worker, 32> list(W);
    for (size_t w = 0; w < W; ++w) list[w] = worker_message(workers[w], n, bucket);
    const at::Tensor& out = tensor(v[4], "out");
    check_values(out, n, "out must hold n float32");
    void* s = current_stream();
    return status(lib.decode_chain, list.data(), (uint32_t)W, n, bucket, scale, (float*)address(out), s);
}

// codes (or None for n == 0), n, bits, hist_out, entropy_out or None
NDQ_METHOD(code_entropy, 5)
{
    const size_t n = integer(v[1]);
    const uint32_t bits = (uint32_t)integer(v[2]);
    const void* codes = nullptr;
    if (n) {
        const at::Tensor& t = tensor(v[0], "codes");
        if (t.nbytes() < lib.packed_bytes(n, bits))
            fail(PyExc_ValueError, "codes hold fewer than ndq_packed_bytes(n, bits) bytes");
        codes = address(t);
    }
    const at::Tensor& hist = tensor(v[3], "hist_out");
    double* entropy = v[4] == Py_None ? nullptr : (double*)address(tensor(v[4], "entropy_out"));
    void* s = current_stream();
    return status(lib.code_entropy, codes, n, bits, (uint64_t*)address(hist), entropy, s);
}

// codes, n, levels, dense_out
NDQ_METHOD(dense_pack, 4)
{
    const at::Tensor &in = tensor(v[0], "codes"), &out = tensor(v[3], "dense_out");
    const size_t n = integer(v[1]);
    const uint32_t levels = (uint32_t)integer(v[2]);
    if (out.nbytes() < lib.dense_bytes(n, levels)) fail(PyExc_ValueError, "dense_out too small");
    void* s = current_stream();
    return status(lib.dense_pack, address(in), n, levels, address(out), s);
}

// dense, n, levels, codes_out
NDQ_METHOD(dense_unpack, 4)
{
    const at::Tensor &in = tensor(v[0], "dense"), &out = tensor(v[3], "codes_out");
    const size_t n = integer(v[1]);
    const uint32_t levels = (uint32_t)integer(v[2]);
    if (out.nbytes() < lib.packed_bytes(n, lib.code_bits(levels))) fail(PyExc_ValueError, "codes_out too small");
    void* s = current_stream();
    return status(lib.dense_unpack, address(in), n, levels, address(out), s);
}

void check_pair(const at::Tensor& a, const at::Tensor& b)
{
    if (!is_f32(a) || !is_f32(b) || count(a) != count(b))
        fail(PyExc_ValueError, "a and b must be float32 of equal length");
}

// a, b, workspace, out
NDQ_METHOD(sqdiff, 4)
{
    const at::Tensor &a = tensor(v[0], "a"), &b = tensor(v[1], "b"), &work = tensor(v[2], "workspace"),
                     &out = tensor(v[3], "out");
    check_pair(a, b);
    const size_t n = count(a);
    void* s = current_stream();
    return status(lib.sqdiff, (const float*)address(a), (const float*)address(b), n, (double*)address(work),
                  (double*)address(out), s);
}

// a, b, out
NDQ_METHOD(sqdiff_static, 3)
{
    const at::Tensor &a = tensor(v[0], "a"), &b = tensor(v[1], "b"), &out = tensor(v[2], "out");
    check_pair(a, b);
    if (!is_f64(out) || count(out) < 1u) fail(PyExc_ValueError, "out must hold one float64");
    const size_t n = count(a);
    void* s = current_stream();
    return status(lib.sqdiff_static, (const float*)address(a), (const float*)address(b), n, (double*)address(out), s);
}

template <class F> bool take(PyObject* addresses, const char* name, F* slot)
{
    PyObject* a = PyDict_GetItemString(addresses, name);      // borrowed
    if (!a) {
        PyErr_Format(PyExc_KeyError, "no address for %s", name);
        return false;
    }
    void* p = PyLong_AsVoidPtr(a);
    if (!p) {
        if (!PyErr_Occurred()) PyErr_Format(PyExc_ValueError, "null address for %s", name);
        return false;
    }
    *slot = (F)p;
    return true;
}

// addresses by name, the ctypes dither class, current-device and raw-stream functions of torch
PyObject* bind(PyObject*, PyObject* const* v, Py_ssize_t n)
{
    if (n != 4 || !PyDict_Check(v[0])) {
        PyErr_SetString(PyExc_TypeError, "bind takes a dict, a class and two functions");
        return nullptr;
    }
    Library l = {};
    if (!take(v[0], "ndq_code_bits", &l.code_bits) || !take(v[0], "ndq_packed_bytes", &l.packed_bytes) ||
        !take(v[0], "ndq_num_buckets", &l.num_buckets) || !take(v[0], "ndq_absmax", &l.absmax) ||
        !take(v[0], "ndq_dq_encode", &l.dq_encode) ||
        !take(v[0], "ndq_dq_encode_with_step", &l.dq_encode_with_step) ||
        !take(v[0], "ndq_nested_encode", &l.nested_encode) ||
        !take(v[0], "ndq_nested_encode_with_step", &l.nested_encode_with_step) ||
        !take(v[0], "ndq_encode_workers", &l.encode_workers) || !take(v[0], "ndq_encode_check", &l.encode_check) ||
        !take(v[0], "ndq_dq_decode", &l.dq_decode) || !take(v[0], "ndq_dq_decode_half", &l.dq_decode_half) ||
        !take(v[0], "ndq_nested_decode", &l.nested_decode) || !take(v[0], "ndq_aggregate", &l.aggregate) ||
        !take(v[0], "ndq_decode_chain", &l.decode_chain) || !take(v[0], "ndq_decode_mean", &l.decode_mean) ||
        !take(v[0], "ndq_code_entropy", &l.code_entropy) || !take(v[0], "ndq_dense_pack", &l.dense_pack) ||
        !take(v[0], "ndq_dense_unpack", &l.dense_unpack) || !take(v[0], "ndq_dense_bytes", &l.dense_bytes) ||
        !take(v[0], "ndq_sqdiff", &l.sqdiff) || !take(v[0], "ndq_sqdiff_static", &l.sqdiff_static))
        return nullptr;
    Py_INCREF(v[1]); Py_XSETREF(dither_type, v[1]);
    Py_INCREF(v[2]); Py_XSETREF(get_device, v[2]);
    Py_INCREF(v[3]); Py_XSETREF(get_raw_stream, v[3]);
    lib = l;
    Py_RETURN_NONE;
}

#define NDQ_ENTRY(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    NDQ_ENTRY(bind), NDQ_ENTRY(absmax), NDQ_ENTRY(dq_encode), NDQ_ENTRY(dq_encode_with_step),
    NDQ_ENTRY(nested_encode), NDQ_ENTRY(nested_encode_with_step), NDQ_ENTRY(encode_workers), NDQ_ENTRY(dq_decode),
    NDQ_ENTRY(dq_decode_half), NDQ_ENTRY(nested_decode), NDQ_ENTRY(aggregate), NDQ_ENTRY(decode_chain), NDQ_ENTRY(decode_mean),
    NDQ_ENTRY(code_entropy), NDQ_ENTRY(dense_pack), NDQ_ENTRY(dense_unpack), NDQ_ENTRY(sqdiff),
    NDQ_ENTRY(sqdiff_static), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
