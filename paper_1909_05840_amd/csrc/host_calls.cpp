// The Python binding's hot half: checks of the tensors, allocation of outputs that were not passed in, the current
// stream, and the call of the C entry point, for every call that takes GPU tensors.
//
// What bounds the small calls is the host: a linear of a few tokens keeps the GPU busy for about 3 us per launch, and the
// same marshalling written in Python over ctypes took 10.5 us per call (torch.empty 1.7 us per output,
// torch.cuda.current_stream() 2.7 us, the conversion of up to 17 arguments the rest), so that a layer forward of eight
// calls took 82 us for 8 and for 4096 tokens alike.  Here a call costs 4.2-4.6 us, of which the runtime's launch is 3.5:
// the layer forward takes 39 us at 8 tokens, and is bound by the GPU from about a thousand tokens on.
// binding.py keeps names, defaults and documentation; the functions below take its arguments by position.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <cstdarg>
#include <vector>
#include "../../include/qbert.h"

namespace {

PyObject *g_error = nullptr;  // binding.QBError

using at::Tensor;
typedef PyObject *const *Args;

[[noreturn]] void throw_python_error()  // a Python error is set
{
    python_error e;
    e.persist();
    throw e;
}

[[noreturn]] void raise(PyObject *type, const char *format, ...)
{
    va_list args;
    va_start(args, format);
    PyErr_FormatV(type, format, args);
    va_end(args);
    throw_python_error();
}

// The interpreter lock is given up while this lives.  The runtime blocks in allocations (until memory is given back) and in
// launches (while the stream's queue is full); other threads go on meanwhile, among them a host callback that the stream may
// be waiting for.  (torch's own calls do the same.)
struct Unlocked {
    PyThreadState *const state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked &) = delete;
    Unlocked &operator=(const Unlocked &) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};

const Tensor &tensor(PyObject *o, const char *name)
{
    if (!THPVariable_Check(o)) raise(PyExc_TypeError, "%s must be a tensor", name);
    return THPVariable_Unpack(o);
}

const char *type_name(at::ScalarType t)
{
    switch (t) {
        case at::kFloat: return "torch.float32";
        case at::kBFloat16: return "torch.bfloat16";
        case at::kChar: return "torch.int8";
        case at::kByte: return "torch.uint8";
        case at::kInt: return "torch.int32";
        default: return "torch.int64";
    }
}

// an input whose type matters: contiguous, on the GPU
const Tensor &typed(PyObject *o, at::ScalarType t, const char *name)
{
    if (!THPVariable_Check(o) || !THPVariable_Unpack(o).is_cuda() || THPVariable_Unpack(o).scalar_type() != t ||
        !THPVariable_Unpack(o).is_contiguous())
        raise(PyExc_TypeError, "%s must be a contiguous %s tensor on the GPU", name, type_name(t));
    return THPVariable_Unpack(o);
}

const Tensor &matrix(PyObject *o, at::ScalarType t, const char *name)
{
    const Tensor &x = typed(o, t, name);
    if (x.dim() != 2) raise(PyExc_ValueError, "%s must have two dimensions", name);
    return x;
}

// a tensor of which the first dimensions are read, any more being the caller's affair
const Tensor &leading(PyObject *o, at::ScalarType t, const char *name, int dims)
{
    const Tensor &x = typed(o, t, name);
    if (x.dim() < dims) raise(PyExc_IndexError, "%s must have %d dimensions or more", name, dims);
    return x;
}

// a tensor or None, as a pointer
template <typename T>
T *ptr(PyObject *o, const char *name)
{
    return o == Py_None ? nullptr : static_cast<T *>(tensor(o, name).data_ptr());
}
template <typename T>
T *ptr(const Tensor &t)
{
    return static_cast<T *>(t.data_ptr());
}
uint16_t *bits16(const Tensor &t) { return t.defined() ? static_cast<uint16_t *>(t.data_ptr()) : nullptr; }

Tensor fresh(at::IntArrayRef size, at::ScalarType t, const at::Device &dev)
{
    const Unlocked unlocked;
    return Tensor(at::detail::empty_cuda(size, t, dev, std::nullopt));
}

// the caller's output, or a new one
Tensor out(PyObject *o, at::IntArrayRef size, at::ScalarType t, const at::Device &dev, const char *name)
{
    return o == Py_None ? fresh(size, t, dev) : tensor(o, name);
}

// Numbers.  The single calls take integers and what stands for one (a numpy integer, a tensor of one), no floats or strings;
// a job's entries may be anything that int() takes.  A value that does not fit is an OverflowError.
int64_t integer(PyObject *o, PyObject *(*convert)(PyObject *) = PyNumber_Index)
{
    PyObject *const n = PyLong_CheckExact(o) ? Py_NewRef(o) : convert(o);
    if (!n) throw_python_error();
    const int64_t v = PyLong_AsLongLong(n);
    Py_DECREF(n);
    if (v == -1 && PyErr_Occurred()) throw_python_error();
    return v;
}

int small(PyObject *o, PyObject *(*convert)(PyObject *) = PyNumber_Index)  // an argument the C side takes as int
{
    const int64_t v = integer(o, convert);
    if (v > INT32_MAX || v < INT32_MIN) raise(PyExc_OverflowError, "integer does not fit a C int");
    return static_cast<int>(v);
}

float real(PyObject *o)  // what float() takes
{
    if (PyFloat_CheckExact(o)) return static_cast<float>(PyFloat_AS_DOUBLE(o));
    PyObject *const f = PyNumber_Float(o);
    if (!f) throw_python_error();
    const double v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return static_cast<float>(v);
}

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Calls a C entry point without the interpreter lock and raises if it fails.  The arguments are converted before, with the
// lock; what they point into belongs to objects that are held until it has returned (the call's arguments, Jobs, Tensor).
template <typename T>
struct Same {
    using type = T;
};
template <typename... P>
void call(qb_status (*entry)(P...), typename Same<P>::type... args)
{
    const qb_status s = [&] {
        const Unlocked unlocked;
        return entry(args...);
    }();
    if (s == QB_OK) return;
    PyObject *e = PyObject_CallFunction(g_error, "is", static_cast<int>(s), qb_status_string(s));
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    throw_python_error();
}

PyObject *tuple(std::initializer_list<Tensor> ts)
{
    PyObject *r = PyTuple_New(static_cast<Py_ssize_t>(ts.size()));
    if (!r) throw_python_error();
    Py_ssize_t i = 0;
    for (const Tensor &t : ts) {  // an undefined tensor becomes None
        PyObject *v = t.defined() ? THPVariable_Wrap(t) : Py_NewRef(Py_None);
        if (!v) {
            Py_DECREF(r);
            throw_python_error();
        }
        PyTuple_SET_ITEM(r, i++, v);
    }
    return r;
}

#define QB_CALL(name, count)                                                                              \
    PyObject *name##_impl(Args a);                                                                        \
    PyObject *name(PyObject *, Args a, Py_ssize_t n)                                                      \
    {                                                                                                     \
        HANDLE_TH_ERRORS                                                                                  \
        if (n != (count)) raise(PyExc_TypeError, #name ": %d arguments expected", (int)(count));         \
        return name##_impl(a);                                                                            \
        END_HANDLE_TH_ERRORS                                                                              \
    }                                                                                                     \
    PyObject *name##_impl(Args a)

// ---- weights

Tensor packed_buffer(PyObject *o, int64_t N, int64_t K, int bits, const at::Device &dev)
{
    const int64_t bytes = static_cast<int64_t>(qb_packed_nbytes(N, K, bits));
    return out(o, {bytes > 0 ? bytes : 1}, at::kByte, dev, "packed");
}

QB_CALL(quantize_groupwise, 7)  // W, bits, groups, packed, h, m, rs_w
{
    const int bits = small(a[1]), groups = small(a[2]);
    const Tensor &W = matrix(a[0], at::kFloat, "W");
    const int64_t N = W.size(0), K = W.size(1);
    const at::Device dev = W.device();
    const Tensor p = packed_buffer(a[3], N, K, bits, dev);
    const Tensor h = out(a[4], {groups > 0 ? groups : 1}, at::kFloat, dev, "h");
    const Tensor m = out(a[5], {groups > 0 ? groups : 1}, at::kFloat, dev, "m");
    const Tensor rs = out(a[6], {N}, at::kInt, dev, "rs_w");
    call(qb_quantize_groupwise, ptr<float>(W), N, K, bits, groups, p.data_ptr(), ptr<float>(h), ptr<float>(m),
                                ptr<int32_t>(rs), stream());
    return tuple({p, h, m, rs});
}

QB_CALL(quantize_groupwise_clip, 6)  // W, bits, m_in, packed, h, rs_w
{
    const int bits = small(a[1]);
    const Tensor &W = matrix(a[0], at::kFloat, "W"), &m = leading(a[2], at::kFloat, "m_in", 1);
    const int64_t N = W.size(0), K = W.size(1), G = m.size(0);
    const at::Device dev = W.device();
    const Tensor p = packed_buffer(a[3], N, K, bits, dev);
    const Tensor h = out(a[4], {G}, at::kFloat, dev, "h"), rs = out(a[5], {N}, at::kInt, dev, "rs_w");
    call(qb_quantize_groupwise_clip, ptr<float>(W), N, K, bits, static_cast<int>(G), ptr<float>(m), p.data_ptr(), ptr<float>(h),
                                     ptr<int32_t>(rs), stream());
    return tuple({p, h, rs});
}

QB_CALL(quantize_groupwise_asym, 7)  // W, bits, groups, packed, delta, q0, rs_w
{
    const int bits = small(a[1]), groups = small(a[2]);
    const Tensor &W = matrix(a[0], at::kFloat, "W");
    const int64_t N = W.size(0), K = W.size(1);
    const at::Device dev = W.device();
    const Tensor p = packed_buffer(a[3], N, K, bits, dev);
    const Tensor d = out(a[4], {groups}, at::kFloat, dev, "delta"), q0 = out(a[5], {groups}, at::kFloat, dev, "q0");
    const Tensor rs = out(a[6], {N}, at::kInt, dev, "rs_w");
    call(qb_quantize_groupwise_asym, ptr<float>(W), N, K, bits, groups, p.data_ptr(), ptr<float>(d), ptr<float>(q0),
                                     ptr<int32_t>(rs), stream());
    return tuple({p, d, q0, rs});
}

QB_CALL(quantize_groupwise_asym_range, 8)  // W, bits, lo, hi, packed, delta, q0, rs_w
{
    const int bits = small(a[1]);
    const Tensor &W = matrix(a[0], at::kFloat, "W"), &lo = typed(a[2], at::kFloat, "lo"), &hi = typed(a[3], at::kFloat, "hi");
    const int64_t N = W.size(0), K = W.size(1), G = lo.numel();
    const at::Device dev = W.device();
    const Tensor p = packed_buffer(a[4], N, K, bits, dev);
    const Tensor d = out(a[5], {G}, at::kFloat, dev, "delta"), q0 = out(a[6], {G}, at::kFloat, dev, "q0");
    const Tensor rs = out(a[7], {N}, at::kInt, dev, "rs_w");
    call(qb_quantize_groupwise_asym_range, ptr<float>(W), N, K, bits, static_cast<int>(G), ptr<float>(lo), ptr<float>(hi),
                                           p.data_ptr(), ptr<float>(d), ptr<float>(q0), ptr<int32_t>(rs), stream());
    return tuple({p, d, q0, rs});
}

// ---- lists of jobs: mappings with the names of the single calls' arguments

PyObject *key(const char *name)  // interned once per name: `name` is a literal at a fixed call site
{
    PyObject *k = PyUnicode_InternFromString(name);
    if (!k) throw_python_error();
    return k;
}

struct Jobs {
    PyObject *seq = nullptr;
    std::vector<PyObject *> held;  // the entries read, until the call has returned: it runs without the interpreter lock
    explicit Jobs(PyObject *o)
    {
        if (PyObject_Size(o) >= 0) seq = PySequence_Tuple(o);  // (what has no length, a generator, is refused)
        if (!seq) throw_python_error();
    }
    ~Jobs()
    {
        for (PyObject *v : held) Py_DECREF(v);
        Py_DECREF(seq);
    }
    Jobs(const Jobs &) = delete;
    Jobs &operator=(const Jobs &) = delete;
    Py_ssize_t size() const { return PyTuple_GET_SIZE(seq); }
    // held by this object; None where an optional entry is absent.  A job is whatever has [] and, for the optional entries,
    // get(); a plain dict is read directly.
    PyObject *get(Py_ssize_t i, PyObject *k, bool required)
    {
        static PyObject *const kGet = key("get");
        PyObject *const d = PyTuple_GET_ITEM(seq, i);
        PyObject *v;
        if (PyDict_CheckExact(d)) {
            v = PyDict_GetItemWithError(d, k);
            if (!v && !PyErr_Occurred()) {
                if (!required) return Py_None;
                PyErr_SetObject(PyExc_KeyError, k);
            }
            Py_XINCREF(v);
        } else {
            v = required ? PyObject_GetItem(d, k) : PyObject_CallMethodOneArg(d, kGet, k);
        }
        if (!v) throw_python_error();
        held.push_back(v);
        return v;
    }
};

PyObject *new_list(Py_ssize_t n)
{
    PyObject *r = PyList_New(n);
    if (!r) throw_python_error();
    return r;
}

QB_CALL(quantize_groupwise_batched, 1)
{
    static PyObject *const kW = key("W"), *const kBits = key("bits"), *const kGroups = key("groups"), *const kPacked = key("packed"),
                    *const kH = key("h"), *const kM = key("m"), *const kRs = key("rs_w");
    Jobs jobs(a[0]);
    const Py_ssize_t n = jobs.size();
    std::vector<qb_quant_job> arr(n);
    THPObjectPtr outs(new_list(n));
    for (Py_ssize_t i = 0; i < n; ++i) {
        const Tensor &W = matrix(jobs.get(i, kW, true), at::kFloat, "W");
        const int64_t N = W.size(0), K = W.size(1);
        const int bits = small(jobs.get(i, kBits, true), PyNumber_Long), groups = small(jobs.get(i, kGroups, true), PyNumber_Long);
        const at::Device dev = W.device();
        const Tensor p = packed_buffer(jobs.get(i, kPacked, false), N, K, bits, dev);
        const Tensor h = out(jobs.get(i, kH, false), {groups > 0 ? groups : 1}, at::kFloat, dev, "h");
        const Tensor m = out(jobs.get(i, kM, false), {groups > 0 ? groups : 1}, at::kFloat, dev, "m");
        const Tensor rs = out(jobs.get(i, kRs, false), {N}, at::kInt, dev, "rs_w");
        arr[i] = qb_quant_job{ptr<float>(W), N, K, bits, groups, p.data_ptr(), ptr<float>(h), ptr<float>(m), ptr<int32_t>(rs)};
        PyList_SET_ITEM(outs.get(), i, tuple({p, h, m, rs}));
    }
    call(qb_quantize_groupwise_batched, arr.data(), static_cast<int>(n), stream());
    return outs.release();
}

QB_CALL(quantize_act_batched, 1)
{
    static PyObject *const kX = key("X"), *const kClip = key("clip"), *const kXq = key("Xq"), *const kRs = key("rs_x");
    Jobs jobs(a[0]);
    const Py_ssize_t n = jobs.size();
    std::vector<qb_act_job> arr(n);
    THPObjectPtr outs(new_list(n));
    for (Py_ssize_t i = 0; i < n; ++i) {
        const Tensor &X = matrix(jobs.get(i, kX, true), at::kFloat, "X");
        const int64_t T = X.size(0), K = X.size(1);
        PyObject *oq = jobs.get(i, kXq, false), *ors = jobs.get(i, kRs, false);
        const Tensor Xq = oq == Py_None ? fresh({T, K}, at::kChar, X.device()) : typed(oq, at::kChar, "Xq");
        const Tensor rs = ors == Py_None ? fresh({T}, at::kInt, X.device()) : typed(ors, at::kInt, "rs_x");
        arr[i] = qb_act_job{ptr<float>(X), T, K, real(jobs.get(i, kClip, true)), ptr<int8_t>(Xq), ptr<int32_t>(rs)};
        PyList_SET_ITEM(outs.get(), i, tuple({Xq, rs}));
    }
    call(qb_quantize_act_batched, arr.data(), static_cast<int>(n), stream());
    return outs.release();
}

QB_CALL(qlinear_fwd_batched, 1)
{
    static PyObject *const kXq = key("Xq"), *const kRs = key("rs_x"), *const kClip = key("clip"), *const kPacked = key("packed"),
                    *const kH = key("h"), *const kRw = key("rs_w"), *const kBits = key("bits"), *const kGroups = key("groups"),
                    *const kN = key("N"), *const kBias = key("bias"), *const kY = key("Y");
    Jobs jobs(a[0]);
    const Py_ssize_t n = jobs.size();
    std::vector<qb_fwd_job> arr(n);
    THPObjectPtr outs(new_list(n));
    for (Py_ssize_t i = 0; i < n; ++i) {
        const Tensor &Xq = matrix(jobs.get(i, kXq, true), at::kChar, "Xq");
        const int64_t T = Xq.size(0), K = Xq.size(1), N = integer(jobs.get(i, kN, true), PyNumber_Long);
        PyObject *oy = jobs.get(i, kY, false), *ob = jobs.get(i, kBias, false);
        const Tensor Y = oy == Py_None ? fresh({T, N}, at::kFloat, Xq.device()) : typed(oy, at::kFloat, "Y");
        arr[i] = qb_fwd_job{ptr<int8_t>(Xq), ptr<int32_t>(typed(jobs.get(i, kRs, true), at::kInt, "rs_x")),
                            real(jobs.get(i, kClip, true)), typed(jobs.get(i, kPacked, true), at::kByte, "packed").data_ptr(),
                            ptr<float>(typed(jobs.get(i, kH, true), at::kFloat, "h")), ptr<int32_t>(typed(jobs.get(i, kRw, true), at::kInt, "rs_w")),
                            small(jobs.get(i, kBits, true), PyNumber_Long), small(jobs.get(i, kGroups, true), PyNumber_Long), T, N, K,
                            ob == Py_None ? nullptr : ptr<float>(typed(ob, at::kFloat, "bias")), ptr<float>(Y)};
        PyObject *v = THPVariable_Wrap(Y);
        if (!v) throw_python_error();
        PyList_SET_ITEM(outs.get(), i, v);
    }
    call(qb_qlinear_fwd_batched, arr.data(), static_cast<int>(n), stream());
    return outs.release();
}

// ---- activations

QB_CALL(quantize_act, 4)  // X, clip, Xq, rs_x
{
    const float clip = real(a[1]);
    const Tensor &X = matrix(a[0], at::kFloat, "X");
    const int64_t T = X.size(0), K = X.size(1);
    const Tensor Xq = out(a[2], {T, K}, at::kChar, X.device(), "Xq"), rs = out(a[3], {T}, at::kInt, X.device(), "rs_x");
    call(qb_quantize_act, ptr<float>(X), T, K, clip, ptr<int8_t>(Xq), ptr<int32_t>(rs), stream());
    return tuple({Xq, rs});
}

QB_CALL(quantize_act_dyn, 4)  // X, Xq, rs_x, hx_rows
{
    const Tensor &X = matrix(a[0], at::kFloat, "X");
    const int64_t T = X.size(0), K = X.size(1);
    const at::Device dev = X.device();
    const Tensor Xq = out(a[1], {T, K}, at::kChar, dev, "Xq"), rs = out(a[2], {T}, at::kInt, dev, "rs_x");
    const Tensor hx = out(a[3], {T}, at::kFloat, dev, "hx_rows");
    call(qb_quantize_act_dyn, ptr<float>(X), T, K, ptr<int8_t>(Xq), ptr<int32_t>(rs), ptr<float>(hx), stream());
    return tuple({Xq, rs, hx});
}

QB_CALL(quantize_act_dyn_tensor, 5)  // X, Xq, rs_x, hx_rows, c
{
    const Tensor &X = matrix(a[0], at::kFloat, "X");
    const int64_t T = X.size(0), K = X.size(1);
    const at::Device dev = X.device();
    const Tensor Xq = out(a[1], {T, K}, at::kChar, dev, "Xq"), rs = out(a[2], {T}, at::kInt, dev, "rs_x");
    const Tensor hx = out(a[3], {T}, at::kFloat, dev, "hx_rows"), c = out(a[4], {1}, at::kFloat, dev, "c");
    call(qb_quantize_act_dyn_tensor, ptr<float>(X), T, K, ptr<int8_t>(Xq), ptr<int32_t>(rs), ptr<float>(hx), ptr<float>(c), stream());
    return tuple({Xq, rs, hx, c});
}

// ---- forward

// Y, and A4 if it was asked for or passed in
PyObject *forward_result(const Tensor &Y, const Tensor &A4)
{
    if (A4.defined()) return tuple({Y, A4});
    PyObject *v = THPVariable_Wrap(Y);
    if (!v) throw_python_error();
    return v;
}

Tensor debug_output(PyObject *given, PyObject *wanted, int64_t T, int64_t N, const at::Device &dev)
{
    if (given != Py_None) return tensor(given, "A4_debug");
    const int w = PyObject_IsTrue(wanted);
    if (w < 0) throw_python_error();
    return w ? fresh({T, N}, at::kInt, dev) : Tensor();
}

int32_t *debug_ptr(const Tensor &t) { return t.defined() ? ptr<int32_t>(t) : nullptr; }

QB_CALL(qlinear_fwd, 13)  // Xq, rs_x, clip, packed, h, rs_w, bits, groups, N, bias, Y, A4_debug, want_a4
{
    const float clip = real(a[2]);
    const int bits = small(a[6]), groups = small(a[7]);
    const int64_t N = integer(a[8]);
    const Tensor &Xq = matrix(a[0], at::kChar, "Xq");
    const int64_t T = Xq.size(0), K = Xq.size(1);
    const Tensor Y = out(a[10], {T, N}, at::kFloat, Xq.device(), "Y");
    const Tensor A4 = debug_output(a[11], a[12], T, N, Xq.device());
    call(qb_qlinear_fwd, ptr<int8_t>(Xq), ptr<int32_t>(a[1], "rs_x"), clip, ptr<void>(a[3], "packed"),
                         ptr<float>(a[4], "h"), ptr<int32_t>(a[5], "rs_w"), bits, groups, T, N, K,
                         ptr<float>(a[9], "bias"), ptr<float>(Y), debug_ptr(A4), stream());
    return forward_result(Y, A4);
}

QB_CALL(qlinear_fwd_dyn, 12)  // Xq, rs_x, hx_rows, packed, h, rs_w, bits, groups, N, bias, Y, want_a4
{
    const int bits = small(a[6]), groups = small(a[7]);
    const int64_t N = integer(a[8]);
    const Tensor &Xq = matrix(a[0], at::kChar, "Xq"), &hx = typed(a[2], at::kFloat, "hx_rows");
    const int64_t T = Xq.size(0), K = Xq.size(1);
    const Tensor Y = out(a[10], {T, N}, at::kFloat, Xq.device(), "Y");
    const Tensor A4 = debug_output(Py_None, a[11], T, N, Xq.device());
    call(qb_qlinear_fwd_dyn, ptr<int8_t>(Xq), ptr<int32_t>(a[1], "rs_x"), ptr<float>(hx), ptr<void>(a[3], "packed"),
                             ptr<float>(a[4], "h"), ptr<int32_t>(a[5], "rs_w"), bits, groups, T, N, K,
                             ptr<float>(a[9], "bias"), ptr<float>(Y), debug_ptr(A4), stream());
    return forward_result(Y, A4);
}

QB_CALL(qlinear_fwd_asym, 13)  // Xq, rs_x, clip, packed, delta, q0, rs_w, bits, groups, N, bias, Y, want_a4
{
    const float clip = real(a[2]);
    const int bits = small(a[7]), groups = small(a[8]);
    const int64_t N = integer(a[9]);
    const Tensor &Xq = matrix(a[0], at::kChar, "Xq"), &d = typed(a[4], at::kFloat, "delta"), &q0 = typed(a[5], at::kFloat, "q0");
    const int64_t T = Xq.size(0), K = Xq.size(1);
    const Tensor Y = out(a[11], {T, N}, at::kFloat, Xq.device(), "Y");
    const Tensor A4 = debug_output(Py_None, a[12], T, N, Xq.device());
    call(qb_qlinear_fwd_asym, ptr<int8_t>(Xq), ptr<int32_t>(a[1], "rs_x"), clip, ptr<void>(a[3], "packed"),
                              ptr<float>(d), ptr<float>(q0), ptr<int32_t>(a[6], "rs_w"), bits, groups, T, N, K,
                              ptr<float>(a[10], "bias"), ptr<float>(Y), debug_ptr(A4), stream());
    return forward_result(Y, A4);
}

QB_CALL(qlinear_fwd_asym_dyn, 13)  // Xq, rs_x, hx_rows, packed, delta, q0, rs_w, bits, groups, N, bias, Y, want_a4
{
    const int bits = small(a[7]), groups = small(a[8]);
    const int64_t N = integer(a[9]);
    const Tensor &Xq = matrix(a[0], at::kChar, "Xq"), &hx = typed(a[2], at::kFloat, "hx_rows");
    const Tensor &d = typed(a[4], at::kFloat, "delta"), &q0 = typed(a[5], at::kFloat, "q0");
    const int64_t T = Xq.size(0), K = Xq.size(1);
    const Tensor Y = out(a[11], {T, N}, at::kFloat, Xq.device(), "Y");
    const Tensor A4 = debug_output(Py_None, a[12], T, N, Xq.device());
    call(qb_qlinear_fwd_asym_dyn, ptr<int8_t>(Xq), ptr<int32_t>(a[1], "rs_x"), ptr<float>(hx), ptr<void>(a[3], "packed"),
                                  ptr<float>(d), ptr<float>(q0), ptr<int32_t>(a[6], "rs_w"), bits, groups, T, N, K,
                                  ptr<float>(a[10], "bias"), ptr<float>(Y), debug_ptr(A4), stream());
    return forward_result(Y, A4);
}

QB_CALL(qlinear_fwd_q8, 14)  // Xq, rs_x, clip, packed, h, rs_w, bits, groups, N, clip_out, bias, act, Yq, rs_y
{
    const float clip = real(a[2]);
    const float clip_out = real(a[9]);
    const int act = small(a[11], PyNumber_Long);
    const int bits = small(a[6]), groups = small(a[7]);
    const int64_t N = integer(a[8]);
    const Tensor &Xq = matrix(a[0], at::kChar, "Xq");
    const int64_t T = Xq.size(0), K = Xq.size(1);
    const Tensor Yq = out(a[12], {T, N}, at::kChar, Xq.device(), "Yq"), rs = out(a[13], {T}, at::kInt, Xq.device(), "rs_y");
    call(qb_qlinear_fwd_q8, ptr<int8_t>(Xq), ptr<int32_t>(a[1], "rs_x"), clip, ptr<void>(a[3], "packed"),
                            ptr<float>(a[4], "h"), ptr<int32_t>(a[5], "rs_w"), bits, groups, T, N, K,
                            ptr<float>(a[10], "bias"), act, clip_out, ptr<int8_t>(Yq), ptr<int32_t>(rs),
                            stream());
    return tuple({Yq, rs});
}

// ---- backward

struct Bwd {
    const Tensor &dY, &Xq;
    int64_t T, N, K;
    Tensor dX, dW, workspace;
    // the outputs wanted and the workspace; each the caller's or new
    Bwd(PyObject *dy, PyObject *xq) : dY(matrix(dy, at::kBFloat16, "dY")), Xq(leading(xq, at::kChar, "Xq", 2))
    {
        T = dY.size(0);
        N = dY.size(1);
        K = Xq.size(1);
    }
    void outputs(PyObject *want_dx, PyObject *want_dw, PyObject *dx, PyObject *dw, PyObject *ws)
    {
        const at::Device dev = dY.device();
        const int wx = PyObject_IsTrue(want_dx), ww = PyObject_IsTrue(want_dw);
        if (wx < 0 || ww < 0) throw_python_error();
        if (dx != Py_None) dX = tensor(dx, "dX");
        else if (wx) dX = fresh({T, K}, at::kBFloat16, dev);
        if (dw != Py_None) dW = tensor(dw, "dW");
        else if (ww) dW = fresh({N, K}, at::kFloat, dev);
        if (ws != Py_None) workspace = tensor(ws, "workspace");
        else {
            const int64_t bytes = static_cast<int64_t>(qb_bwd_workspace_nbytes(T, N, K));
            workspace = fresh({bytes > 256 ? bytes : 256}, at::kByte, dev);
        }
    }
    float *dw_ptr() const { return dW.defined() ? ptr<float>(dW) : nullptr; }
};

QB_CALL(qlinear_bwd_ste, 12)  // dY, Xq, clip, packed, h, bits, groups, want_dx, want_dw, dX, dW, workspace
{
    const float clip = real(a[2]);
    const int bits = small(a[5]), groups = small(a[6]);
    Bwd b(a[0], a[1]);
    b.outputs(a[7], a[8], a[9], a[10], a[11]);
    call(qb_qlinear_bwd_ste, bits16(b.dY), ptr<int8_t>(b.Xq), clip, ptr<void>(a[3], "packed"),
                             ptr<float>(a[4], "h"), bits, groups, b.T, b.N, b.K, bits16(b.dX), b.dw_ptr(),
                             b.workspace.data_ptr(), stream());
    return tuple({b.dX, b.dW});
}

QB_CALL(qlinear_bwd_ste_static, 9)  // dY, Xq, clip, packed, h, bits, groups, dX, dW
{
    const float clip = real(a[2]);
    const int bits = small(a[5]), groups = small(a[6]);
    const Bwd b(a[0], a[1]);
    call(qb_qlinear_bwd_ste_static, bits16(b.dY), ptr<int8_t>(b.Xq), clip, ptr<void>(a[3], "packed"),
                                    ptr<float>(a[4], "h"), bits, groups, b.T, b.N, b.K, ptr<uint16_t>(a[7], "dX"),
                                    ptr<float>(a[8], "dW"), stream());
    return PyTuple_Pack(2, a[7], a[8]);
}

QB_CALL(qlinear_bwd_ste_masked, 15)  // dY, Xq, clip, packed, h, bits, groups, X, W, m, want_dx, want_dw, dX, dW, workspace
{
    const float clip = real(a[2]);
    const int bits = small(a[5]), groups = small(a[6]);
    Bwd b(a[0], a[1]);
    if (a[7] != Py_None) {
        const Tensor &X = typed(a[7], at::kFloat, "X");
        if (X.dim() != 2 || X.size(0) != b.T || X.size(1) != b.K) raise(PyExc_ValueError, "X must be [T, K]");
    }
    if (a[8] != Py_None) {
        const Tensor &W = typed(a[8], at::kFloat, "W");
        if (W.dim() != 2 || W.size(0) != b.N || W.size(1) != b.K) raise(PyExc_ValueError, "W must be [N, K]");
    }
    if (a[9] != Py_None && typed(a[9], at::kFloat, "m").numel() != groups)
        raise(PyExc_ValueError, "m must hold one range per group");
    b.outputs(a[10], a[11], a[12], a[13], a[14]);
    call(qb_qlinear_bwd_ste_masked, bits16(b.dY), ptr<int8_t>(b.Xq), clip, ptr<void>(a[3], "packed"),
                                    ptr<float>(a[4], "h"), bits, groups, b.T, b.N, b.K, ptr<float>(a[7], "X"),
                                    ptr<float>(a[8], "W"), ptr<float>(a[9], "m"), bits16(b.dX), b.dw_ptr(), b.workspace.data_ptr(),
                                    stream());
    return tuple({b.dX, b.dW});
}

QB_CALL(qlinear_bwd_ste_asym, 13)  // dY, Xq, clip, packed, delta, q0, bits, groups, want_dx, want_dw, dX, dW, workspace
{
    const float clip = real(a[2]);
    const int bits = small(a[6]), groups = small(a[7]);
    Bwd b(a[0], a[1]);
    b.outputs(a[8], a[9], a[10], a[11], a[12]);
    call(qb_qlinear_bwd_ste_asym, bits16(b.dY), ptr<int8_t>(b.Xq), clip, ptr<void>(a[3], "packed"),
                                  ptr<float>(a[4], "delta"), ptr<float>(a[5], "q0"), bits, groups, b.T, b.N, b.K,
                                  bits16(b.dX), b.dw_ptr(), b.workspace.data_ptr(), stream());
    return tuple({b.dX, b.dW});
}

// ---- embedding

// the 8-bit table's entry points, or with bits those for either width
template <typename F>
PyObject *embedding_quantize_with(const F &entry, int64_t bits, int groups, PyObject *e, PyObject *given_codes, PyObject *given_h, PyObject *given_m)
{
    const Tensor &E = matrix(e, at::kFloat, "E");
    const int64_t V = E.size(0), d = E.size(1);
    const at::Device dev = E.device();
    const Tensor codes = out(given_codes, {V, d * bits / 8}, at::kByte, dev, "codes");
    const Tensor h = out(given_h, {groups > 0 ? groups : 1}, at::kFloat, dev, "h"), m = out(given_m, {groups > 0 ? groups : 1}, at::kFloat, dev, "m");
    entry(ptr<float>(E), V, d, ptr<uint8_t>(codes), ptr<float>(h), ptr<float>(m));
    return tuple({codes, h, m});
}

template <typename F>
PyObject *embedding_gather_with(const F &entry, int bits, const Tensor &codes, PyObject *given_ids, PyObject *given_out)
{
    const Tensor &ids = leading(given_ids, at::kLong, "ids", 1);
    const int64_t V = codes.size(0), d = bits > 0 ? codes.size(1) * 8 / bits : 0, n = ids.size(0);
    const Tensor o = out(given_out, {n, d}, at::kFloat, codes.device(), "out");
    entry(V, d, ptr<int64_t>(ids), n, ptr<float>(o));
    PyObject *v = THPVariable_Wrap(o);
    if (!v) throw_python_error();
    return v;
}

QB_CALL(embedding_quantize, 5)  // E, groups, codes, h, m
{
    const int groups = small(a[1]);
    return embedding_quantize_with([&](const float *E, int64_t V, int64_t d, uint8_t *codes, float *h, float *m) {
        call(qb_embedding_quantize, E, V, d, groups, codes, h, m, stream());
    }, 8, groups, a[0], a[2], a[3], a[4]);
}

QB_CALL(embedding_quantize_bits, 6)  // E, bits, groups, codes, h, m
{
    const int bits = small(a[1]), groups = small(a[2]);
    return embedding_quantize_with([&](const float *E, int64_t V, int64_t d, uint8_t *codes, float *h, float *m) {
        call(qb_embedding_quantize_bits, E, V, d, bits, groups, codes, h, m, stream());
    }, bits, groups, a[0], a[3], a[4], a[5]);
}

QB_CALL(embedding_gather, 5)  // codes, h, groups, ids, out
{
    const int groups = small(a[2]);
    const Tensor &codes = matrix(a[0], at::kByte, "codes");
    return embedding_gather_with([&](int64_t V, int64_t d, const int64_t *ids, int64_t n, float *o) {
        call(qb_embedding_gather, ptr<uint8_t>(codes), ptr<float>(a[1], "h"), V, d, groups, ids, n, o, stream());
    }, 8, codes, a[3], a[4]);
}

QB_CALL(embedding_gather_bits, 6)  // codes, h, bits, groups, ids, out
{
    const int bits = small(a[2]), groups = small(a[3]);
    const Tensor &codes = leading(a[0], at::kByte, "codes", 2);
    return embedding_gather_with([&](int64_t V, int64_t d, const int64_t *ids, int64_t n, float *o) {
        call(qb_embedding_gather_bits, ptr<uint8_t>(codes), ptr<float>(a[1], "h"), V, d, bits, groups, ids, n, o, stream());
    }, bits, codes, a[4], a[5]);
}

PyObject *set_error(PyObject *, PyObject *cls)
{
    Py_INCREF(cls);
    Py_XSETREF(g_error, cls);
    Py_RETURN_NONE;
}

#define QB_ENTRY(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    QB_ENTRY(quantize_groupwise), QB_ENTRY(quantize_groupwise_clip), QB_ENTRY(quantize_groupwise_asym),
    QB_ENTRY(quantize_groupwise_asym_range), QB_ENTRY(quantize_groupwise_batched), QB_ENTRY(quantize_act_batched),
    QB_ENTRY(qlinear_fwd_batched), QB_ENTRY(quantize_act), QB_ENTRY(quantize_act_dyn), QB_ENTRY(quantize_act_dyn_tensor),
    QB_ENTRY(qlinear_fwd), QB_ENTRY(qlinear_fwd_dyn), QB_ENTRY(qlinear_fwd_asym), QB_ENTRY(qlinear_fwd_asym_dyn),
    QB_ENTRY(qlinear_fwd_q8), QB_ENTRY(qlinear_bwd_ste), QB_ENTRY(qlinear_bwd_ste_static), QB_ENTRY(qlinear_bwd_ste_masked),
    QB_ENTRY(qlinear_bwd_ste_asym), QB_ENTRY(embedding_quantize), QB_ENTRY(embedding_quantize_bits), QB_ENTRY(embedding_gather),
    QB_ENTRY(embedding_gather_bits),
    {"set_error", set_error, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&g_module); }
