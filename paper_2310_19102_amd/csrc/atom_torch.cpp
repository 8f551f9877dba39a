// The run-time entry points for Python: torch tensors in, one call into libatom.so, torch tensors out.
//
// What bounds it: a decode-sized call is host work.  Marshalling through ctypes (a python object per
// pointer, size and stream, a data_ptr() and stride() call per tensor) cost 10 to 12 us per call, twice
// what the kernels of such a call take on the GPU; read here from the tensor structs it is below 1 us,
// and the launch itself is what is left.  The functions are called by the wrappers of the same name in
// binding.py, which hold names, defaults and documentation; arguments arrive by position.
//
// No arithmetic of the method happens here.

#include <Python.h>

#include <ATen/hip/EmptyTensor.h>
#include <ATen/hip/HIPContext.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPGraphsC10Utils.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <initializer_list>

#include "atom.h"

namespace {

using at::Tensor;

PyObject *g_atom_error = nullptr;          // binding.AtomError

struct Raised {};                          // a python exception is set

[[noreturn]] void value_error(const char *text)
{
    PyErr_SetString(PyExc_ValueError, text);
    throw Raised();
}

[[noreturn]] void value_error(const char *name, const char *text)
{
    PyErr_Format(PyExc_ValueError, "%s %s", name, text);
    throw Raised();
}

const Tensor &tensor(PyObject *o, const char *name)
{
    if (!THPVariable_CheckExact(o) && !THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s: expected a torch tensor, got %s", name, Py_TYPE(o)->tp_name);
        throw Raised();
    }
    return THPVariable_Unpack(o);
}

struct Kind { at::ScalarType type; const char *name; };
constexpr Kind kHalf = {at::kHalf, "torch.float16"}, kByte = {at::kByte, "torch.uint8"},
               kChar = {at::kChar, "torch.int8"}, kInt = {at::kInt, "torch.int32"},
               kShort = {at::kShort, "torch.int16"};

// A device tensor of the given type (what binding.py has always asked of its arguments).
const Tensor &device(PyObject *o, Kind k, const char *name)
{
    const Tensor &t = tensor(o, name);
    if (!t.is_cuda()) value_error(name, "must be a device tensor");
    if (t.scalar_type() != k.type) {
        PyObject *got = PyObject_GetAttrString(o, "dtype");
        if (got) PyErr_Format(PyExc_TypeError, "%s: expected %s, got %S", name, k.name, got);
        Py_XDECREF(got);
        throw Raised();
    }
    return t;
}

const Tensor &contiguous(PyObject *o, Kind k, const char *name)
{
    const Tensor &t = device(o, k, name);
    if (!t.is_contiguous()) value_error(name, "must be contiguous");
    return t;
}

void *data(const Tensor &t) { return t.data_ptr(); }

// An optional device tensor's address: None is NULL.
void *maybe(PyObject *o, Kind k, const char *name) { return o == Py_None ? nullptr : data(device(o, k, name)); }

long whole(PyObject *o)
{
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised();
    return v;
}

float real(PyObject *o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Raised();
    return (float)v;
}

// Groups of a row (a group size that is none is left for the library to refuse).
int64_t groups(int64_t K, int64_t gs) { return gs > 0 ? K / gs : 0; }

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

// A new tensor on the device of `like`: what at::empty ends at after its dispatch (0.6 us each, and a front-end call
// makes three).
Tensor make(at::IntArrayRef shape, Kind k, const Tensor &like)
{
    return Tensor(at::detail::empty_cuda(shape, k.type, like.device(), std::nullopt));
}

Tensor make(std::initializer_list<int64_t> shape, Kind k, const Tensor &like) { return make(at::IntArrayRef(shape), k, like); }

// (the default stream cannot be captured, and the question takes 0.15 us)
bool capturing() { return stream() && c10::hip::currentStreamCaptureStatusMayInitCtx() != c10::hip::CaptureStatus::None; }

// Memory for the length of a call only may be part of a captured graph where it comes from a pool that the graph keeps (torch.cuda.graph).  In a
// capture that the allocator does not know of the block would be free again when the call returns, and a replay would write into
// whatever has it by then.
bool safe_to_capture(const Tensor &t)
{
    if (!capturing()) return true;
    const size_t at = (size_t)t.data_ptr();
    try {
        for (const auto &s : c10::hip::HIPCachingAllocator::snapshot().segments)
            if (s.device == t.device().index() && at - s.address < s.total_size) return s.owner_private_pool_id != c10::MempoolId_t{0, 0};
    } catch (const c10::Error &) {                                     // (an allocator of the program's own that does not say)
    }
    return false;
}

// Whether the allocator is likely to have n bytes without giving back what it keeps.  A request that neither its free blocks nor the device
// can serve makes it return every free block to the device, behind a synchronisation, before it raises: too much for memory that a call can do
// without, and that asks again with every call.  (Under capture it returns nothing, and the device is not asked.)
bool has_room(int64_t n, c10::DeviceIndex device)
{
    namespace allocator = c10::hip::HIPCachingAllocator;
    if (capturing()) return true;
    try {
        size_t largest = 1;                                            // (0: the device's free memory counts as well)
        allocator::cacheInfo(device, &largest);
        if (largest >= (size_t)n) return true;
        const double with = (double)n + (double)(20 << 20);           // (what it takes from the device is rounded up, to 20 MB at least)
        const double fraction = allocator::getMemoryFraction(device);
        if (fraction < 1.0) {
            const auto stats = allocator::getDeviceStats(device);
            const auto &reserved = stats.reserved_bytes[static_cast<size_t>(c10::CachingAllocator::StatType::AGGREGATE)];
            if ((double)reserved.current + with > fraction * (double)at::cuda::getDeviceProperties(device)->totalGlobalMem) return false;
        }
        largest = 0;
        allocator::cacheInfo(device, &largest);
        return (double)largest >= with;
    } catch (const c10::Error &) {                                     // (an allocator of the program's own that does not say)
        return true;
    }
}

// Row stride of a matrix with `cols` columns (a single row may report any stride).
int64_t ld(const Tensor &t, int64_t rows, int64_t cols)
{
    return rows > 1 ? t.stride(0) : std::max<int64_t>(cols, t.stride(0));
}

void matrix(const Tensor &t, const char *text)
{
    if (t.dim() != 2 || t.stride(1) != 1) value_error(text);
}

// A code or scale array whose two sizes say what a call computes (weights stacked over layers, with a dimension in front,
// are not one: their first sizes would be taken for rows and outliers).
void rows_and_columns(const Tensor &t, const char *name)
{
    if (t.dim() != 2) value_error(name, "must have two dimensions");
}

size_t bytes(const Tensor &t) { return (size_t)t.numel() * t.element_size(); }

void check(int status, const char *where)
{
    if (status == 0) return;
    PyObject *e = PyObject_CallFunction(g_atom_error, "is", status, where);
    if (e) PyErr_SetObject(g_atom_error, e);
    Py_XDECREF(e);
    throw Raised();
}

// Other python threads run while this lives; it takes the interpreter back also where an exception leaves the scope.
struct Released {
    PyThreadState *state = PyEval_SaveThread();
    Released() = default;
    ~Released() { PyEval_RestoreThread(state); }
    Released(const Released &) = delete;
    Released &operator=(const Released &) = delete;
};

// The call into the library on the current stream.  Every address is an argument here, so all of them were read before other
// threads may run.
template <class F, class... A> int call(F f, A... a)
{
    void *s = stream();
    const Released others;
    return f(a..., s);
}
#define ATOM_CALL(f, ...) check(call(f, __VA_ARGS__), #f)

// A python result object: the caller's own (out= arguments, held until the call is over: an iterator gives its only
// reference) or a new tensor's.
struct Out {
    PyObject *o = nullptr;
    const Tensor *t = nullptr;
    Tensor own;
    Out() = default;
    ~Out() { Py_XDECREF(o); }
    Out(const Out &) = delete;
    Out &operator=(const Out &) = delete;
    void given(PyObject *p, const char *name) { t = &tensor(p, name); o = p; Py_INCREF(o); }
    void fresh(Tensor &&n) { own = std::move(n); t = &own; }
    void take(PyObject *p, const char *name, std::initializer_list<int64_t> shape, Kind k, const Tensor &like)
    {
        if (p == Py_None) fresh(make(shape, k, like));
        else given(p, name);
    }
    void *data() const { return t->data_ptr(); }
    PyObject *give() const               // new reference
    {
        if (o) { Py_INCREF(o); return o; }
        return THPVariable_Wrap(own);
    }
};

PyObject *tuple(std::initializer_list<const Out *> v)
{
    PyObject *r = PyTuple_New((Py_ssize_t)v.size());
    if (!r) throw Raised();
    Py_ssize_t i = 0;
    for (const Out *x : v) PyTuple_SET_ITEM(r, i++, x->give());
    return r;
}

PyObject *first_three(PyObject *o)
{
    PyObject *r = PyTuple_New(3);
    for (Py_ssize_t i = 0; r && i < 3; ++i) {
        PyObject *n = PyLong_FromSsize_t(i), *item = n ? PyObject_GetItem(o, n) : nullptr;
        Py_XDECREF(n);
        if (item) PyTuple_SET_ITEM(r, i, item);
        else Py_CLEAR(r);
    }
    return r;
}

// Three tensors given as any iterable (codes, outliers, scales / codes, scales, zeros), held while this lives: a list may be
// changed by another thread meanwhile, so its items are taken over into a tuple (a tuple is kept as it is).
struct Three {
    PyObject *seq = nullptr;
    PyObject *item[3];
    explicit Three(PyObject *o, bool indexed = false)      // indexed: items 0, 1 and 2 of what may have more
    {
        seq = indexed ? first_three(o) : PySequence_Tuple(o);
        if (!seq) throw Raised();
        if (PyTuple_GET_SIZE(seq) != 3) {
            Py_DECREF(seq);
            value_error("expected three tensors");
        }
        for (int i = 0; i < 3; ++i) item[i] = PyTuple_GET_ITEM(seq, i);
    }
    ~Three() { Py_XDECREF(seq); }
    Three(const Three &) = delete;
    Three &operator=(const Three &) = delete;
};

// Codes, outliers and scales of `rows` rows: the caller's or new ones.
struct Codes {
    Out q4, q8, sc;
    void take(PyObject *out, int64_t rows, int64_t K, int64_t gs, int64_t O, const Tensor &like, bool indexed = false)
    {
        if (out == Py_None) {
            q4.fresh(make({rows, (K - O) / 2}, kByte, like));
            q8.fresh(make({rows, O}, kChar, like));
            sc.fresh(make({rows, groups(K, gs)}, kHalf, like));
        } else {
            Three t(out, indexed);
            q4.given(t.item[0], "q4");
            q8.given(t.item[1], "q8");
            sc.given(t.item[2], "scale");
        }
    }
};

atom_desc desc(int64_t K, int64_t gs, int64_t O, int64_t bits = 4)
{
    return {(int32_t)K, (int32_t)gs, (int32_t)O, (int32_t)bits, 8};
}

typedef PyObject *const *Args;

PyObject *quantize_act(Args a)
{
    const Tensor &x = device(a[0], kHalf, "x");
    void *idx = maybe(a[3], kInt, "reorder_idx"), *gamma = maybe(a[1], kHalf, "gamma");
    matrix(x, "x must be [M, K] with a contiguous last dimension");
    const int64_t M = x.size(0), K = x.size(1), gs = whole(a[4]), O = whole(a[5]);
    const float eps = real(a[2]), clip = real(a[6]);
    Codes q;
    q.take(a[7], M, K, gs, O, x);
    const atom_desc d = desc(K, gs, O, whole(a[8]));
    ATOM_CALL(atom_quantize_act, data(x), M, ld(x, M, K), gamma, eps, (const int32_t *)idx, &d, clip, q.q4.data(),
              q.q8.data(), q.sc.data());
    return tuple({&q.q4, &q.q8, &q.sc});
}

PyObject *add_quantize_act(Args a)
{
    const Tensor &x = device(a[0], kHalf, "x"), &r = device(a[1], kHalf, "residual");
    void *idx = maybe(a[4], kInt, "reorder_idx"), *gamma = maybe(a[2], kHalf, "gamma");
    if (x.dim() != 2 || x.stride(1) != 1 || r.sizes() != x.sizes() || r.stride(1) != 1)
        value_error("x and residual must be [M, K] with a contiguous last dimension");
    const int64_t M = x.size(0), K = x.size(1), gs = whole(a[5]), O = whole(a[6]);
    const float eps = real(a[3]), clip = real(a[7]);
    Out sum;
    sum.take(a[8], "sum_out", {M, K}, kHalf, x);
    if (sum.o) device(sum.o, kHalf, "sum_out");
    if (sum.t->sizes() != x.sizes() || sum.t->stride(1) != 1)
        value_error("sum_out must be [M, K] with a contiguous last dimension");
    Codes q;
    q.take(a[9], M, K, gs, O, x);
    const atom_desc d = desc(K, gs, O, whole(a[10]));
    ATOM_CALL(atom_add_quantize_act, data(x), data(r), M, ld(x, M, K), ld(r, M, K), sum.data(), ld(*sum.t, M, K), gamma,
              eps, (const int32_t *)idx, &d, clip, q.q4.data(), q.q8.data(), q.sc.data());
    return tuple({&sum, &q.q4, &q.q8, &q.sc});
}

PyObject *swiglu_quantize_act(Args a)
{
    const Tensor &g = device(a[0], kHalf, "gate"), &u = device(a[1], kHalf, "up");
    void *idx = maybe(a[2], kInt, "reorder_idx");
    if (g.dim() != 2 || g.stride(1) != 1 || u.sizes() != g.sizes() || u.stride(1) != 1)
        value_error("gate and up must be [M, K] with a contiguous last dimension");
    const int64_t M = g.size(0), K = g.size(1), gs = whole(a[3]), O = whole(a[4]);
    const float clip = real(a[5]);
    Codes q;
    q.take(a[6], M, K, gs, O, g);
    const atom_desc d = desc(K, gs, O, whole(a[7]));
    ATOM_CALL(atom_swiglu_quantize_act, data(g), data(u), M, ld(g, M, K), ld(u, M, K), (const int32_t *)idx, &d, clip,
              q.q4.data(), q.q8.data(), q.sc.data());
    return tuple({&q.q4, &q.q8, &q.sc});
}

// The [M, N, G] int32 array of per-group sums, or NULL.
int32_t *partial_sums(PyObject *o, int64_t M, int64_t N, int64_t G)
{
    if (o == Py_None) return nullptr;
    const Tensor &t = device(o, kInt, "partials");
    if (t.dim() != 3 || t.size(0) != M || t.size(1) != N || t.size(2) != G || !t.is_contiguous())
        value_error("partials must be contiguous int32 [M, N, G]");
    return (int32_t *)data(t);
}

PyObject *w4a4_gemm(Args a)
{
    const Tensor &a4 = contiguous(a[0], kByte, "a_q4"), &a8 = contiguous(a[1], kChar, "a_q8"),
                 &as = contiguous(a[2], kHalf, "a_scale"), &w4 = contiguous(a[3], kByte, "w_q4"),
                 &w8 = contiguous(a[4], kChar, "w_q8"), &ws = contiguous(a[5], kHalf, "w_scale");
    rows_and_columns(a8, "a_q8");
    const int64_t M = a8.size(0), O = a8.size(1), N = w8.size(0), K = 2 * a4.size(1) + O, gs = whole(a[6]);
    if (w4.size(1) != a4.size(1) || w8.size(1) != O) value_error("activation and weight code shapes disagree");
    Out y;
    y.take(a[7], "out", {M, N}, kHalf, a4);
    if (y.o) device(y.o, kHalf, "out");
    int32_t *partials = partial_sums(a[8], M, N, groups(K, gs));
    const atom_desc d = desc(K, gs, O);
    const size_t need = atom_w4a4_gemm_workspace_bytes(M, N, &d);
    Tensor own;
    const Tensor *w = a[9] == Py_None ? nullptr : &tensor(a[9], "workspace");
    if (need && (!w || bytes(*w) < need)) {
        own = make({(int64_t)need}, kByte, a4);
        w = &own;
    }
    // room to pack the operands on the way where that is faster; a call that finds none goes without
    const size_t room = need || w || partials ? 0 : atom_w4a4_gemm_scratch_bytes(M, N, &d);
    if (room && has_room((int64_t)room, a4.device().index())) {
        try {
            own = make({(int64_t)room}, kByte, a4);
            if (safe_to_capture(own)) w = &own;
        } catch (const c10::OutOfMemoryError &) {
        }
    }
    // packed operands go only where all the bytes that the tensor counts are its own and the device's (a workspace is never required, and
    // any tensor is taken for one)
    const bool usable = w && w->device() == a4.device() && w->is_contiguous();
    ATOM_CALL(atom_w4a4_gemm, data(a4), data(a8), data(as), M, data(w4), data(w8), data(ws), N, &d, y.data(),
              ld(*y.t, M, N), partials, usable ? data(*w) : nullptr, usable ? bytes(*w) : 0);
    return y.give();
}

PyObject *w4a4_gemm_decode_tiled(Args a)
{
    const Tensor &a4 = tensor(a[0], "a_q4"), &a8 = tensor(a[1], "a_q8"), &as = tensor(a[2], "a_scale"),
                 &w4 = tensor(a[3], "w_q4_tiled"), &w8 = tensor(a[4], "w_q8_tiled"), &ws = tensor(a[5], "w_scale");
    rows_and_columns(a8, "a_q8");
    rows_and_columns(ws, "w_scale");
    const int64_t M = a8.size(0), O = a8.size(1), N = ws.size(0), gs = whole(a[6]), K = ws.size(1) * gs;
    Out y;
    y.take(a[7], "out", {M, N}, kHalf, a4);
    const atom_desc d = desc(K, gs, O);
    ATOM_CALL(atom_w4a4_gemm_decode_tiled, data(a4), data(a8), data(as), M, data(w4), data(w8), data(ws), N, &d,
              y.data(), ld(*y.t, M, N));
    return y.give();
}

PyObject *decode_linear(Args a)
{
    const Tensor &x = device(a[0], kHalf, "x");
    void *idx = maybe(a[3], kInt, "reorder_idx"), *gamma = maybe(a[1], kHalf, "gamma");
    const Tensor &w4 = device(a[4], kByte, "w_q4"), &w8 = device(a[5], kChar, "w_q8"),
                 &ws = device(a[6], kHalf, "w_scale");
    matrix(x, "x must be [M, K] with a contiguous last dimension");
    rows_and_columns(w8, "w_q8");
    const int64_t M = x.size(0), K = x.size(1), N = w8.size(0), O = w8.size(1), gs = whole(a[7]);
    const float eps = real(a[2]), clip = real(a[8]);
    Out y;
    y.take(a[9], "out", {M, N}, kHalf, x);
    const int debug = PyObject_IsTrue(a[10]);
    if (debug < 0) throw Raised();
    Codes q;
    if (debug) q.take(Py_None, M, K, gs, O, x);
    const atom_desc d = desc(K, gs, O, whole(a[11]));
    void *c4 = nullptr, *c8 = nullptr, *cs = nullptr;
    Tensor own;
    if (debug) {
        c4 = q.q4.data(); c8 = q.q8.data(); cs = q.sc.data();
    } else if (atom_decode_linear_wants_codes(M, N, &d, gamma != nullptr)) {   // one array for the three, each from a 256-byte boundary
        const auto up = [](int64_t n) { return (n + 255) / 256 * 256; };
        const int64_t n4 = up(M * (K - O) / 2), n8 = up(M * O);
        try {
            own = make({n4 + n8 + M * groups(K, gs) * 2}, kByte, x);
            if (safe_to_capture(own)) { c4 = data(own); c8 = (char *)c4 + n4; cs = (char *)c8 + n8; }
        } catch (const c10::OutOfMemoryError &) {       // one launch then, the same bits
        }
    }
    ATOM_CALL(atom_decode_linear, data(x), M, ld(x, M, K), gamma, eps, (const int32_t *)idx, &d, clip, data(w4),
              data(w8), data(ws), N, y.data(), ld(*y.t, M, N), c4, c8, cs);
    if (!debug) return y.give();
    PyObject *codes = tuple({&q.q4, &q.q8, &q.sc});
    return Py_BuildValue("(NN)", y.give(), codes);
}

PyObject *decode_linear_coop(Args a)
{
    const Tensor &x = device(a[0], kHalf, "x");
    void *idx = maybe(a[3], kInt, "reorder_idx"), *gamma = maybe(a[1], kHalf, "gamma");
    const Tensor &w4 = device(a[4], kByte, "w_q4"), &w8 = device(a[5], kChar, "w_q8"),
                 &ws = device(a[6], kHalf, "w_scale"), &sync = device(a[7], kInt, "sync_words");
    if (4 * (size_t)sync.numel() < atom_decode_linear_coop_sync_bytes() || !sync.is_contiguous())
        value_error("sync_words is too small: take atom_decode_linear_coop_sync()");
    matrix(x, "x must be [M, K] with a contiguous last dimension");
    rows_and_columns(w8, "w_q8");
    const int64_t M = x.size(0), K = x.size(1), N = w8.size(0), O = w8.size(1), gs = whole(a[8]);
    const float eps = real(a[2]), clip = real(a[9]);
    Out y;
    y.take(a[10], "out", {M, N}, kHalf, x);
    Codes q;
    q.take(a[11], M, K, gs, O, x, true);
    const atom_desc d = desc(K, gs, O, whole(a[12]));
    ATOM_CALL(atom_decode_linear_coop, data(x), M, ld(x, M, K), gamma, eps, (const int32_t *)idx, &d, clip, data(w4),
              data(w8), data(ws), N, y.data(), ld(*y.t, M, N), q.q4.data(), q.q8.data(), q.sc.data(), data(sync));
    PyObject *codes;
    if (a[11] != Py_None) { codes = a[11]; Py_INCREF(codes); }       // the caller's own sequence
    else codes = tuple({&q.q4, &q.q8, &q.sc});
    return Py_BuildValue("(NN)", y.give(), codes);
}

// The packed image of M rows: the caller's buffer or a new one.
void packed_out(Out &out, PyObject *o, int64_t M, const atom_desc &d, const Tensor &like)
{
    if (o == Py_None) out.fresh(make({(int64_t)std::max<size_t>(atom_pack_weight_bytes(M, &d), 1)}, kByte, like));
    else out.given(o, "out"), device(o, kByte, "out");
}

PyObject *pack_act(Args a)
{
    const Tensor &a4 = contiguous(a[0], kByte, "a_q4"), &a8 = contiguous(a[1], kChar, "a_q8"),
                 &as = contiguous(a[2], kHalf, "a_scale");
    rows_and_columns(a8, "a_q8");
    const int64_t M = a8.size(0), O = a8.size(1), K = 2 * a4.size(1) + O;
    const atom_desc d = desc(K, whole(a[3]), O);
    Out out;
    packed_out(out, a[4], M, d, a4);
    ATOM_CALL(atom_pack_act, data(a4), data(a8), data(as), M, &d, out.data(), (size_t)out.t->numel());
    return out.give();
}

PyObject *quantize_act_packed(Args a)
{
    const Tensor &x = device(a[0], kHalf, "x");
    matrix(x, "x must be [M, K] with a contiguous last dimension");
    void *idx = maybe(a[3], kInt, "reorder_idx"), *gamma = maybe(a[1], kHalf, "gamma");
    const int64_t M = x.size(0), K = x.size(1);
    const float eps = real(a[2]), clip = real(a[6]);
    const atom_desc d = desc(K, whole(a[4]), whole(a[5]), whole(a[8]));
    Out out;
    packed_out(out, a[7], M, d, x);
    ATOM_CALL(atom_quantize_act_packed, data(x), M, ld(x, M, K), gamma, eps, (const int32_t *)idx, &d, clip, out.data(),
              (size_t)out.t->numel());
    return out.give();
}

// The packed forms take as second operand whatever holds the first one's rows at its first stride: a matrix with more rows or
// columns (its first ones are read), one with dimensions of one element in between, for one row anything contiguous.
bool covers(const Tensor &t, const Tensor &x)
{
    const int64_t M = x.size(0), K = x.size(1);
    if (t.dim() == 2 && t.stride(1) == 1 && t.size(0) >= M && t.size(1) >= K) return true;
    if (t.dim() < 1) return false;
    if (M == 1 && t.is_contiguous()) return t.numel() >= K;
    return t.dim() > 2 && t.size(0) >= M && t.select(0, 0).is_contiguous() && t.numel() >= t.size(0) * K;
}

PyObject *add_quantize_act_packed(Args a)
{
    const Tensor &x = device(a[0], kHalf, "x"), &r = device(a[1], kHalf, "residual");
    if (x.dim() != 2 || x.stride(1) != 1 || !covers(r, x))
        value_error("x and residual must be [M, K] with a contiguous last dimension");
    void *idx = maybe(a[4], kInt, "reorder_idx"), *gamma = maybe(a[2], kHalf, "gamma");
    const int64_t M = x.size(0), K = x.size(1);
    const float eps = real(a[3]), clip = real(a[7]);
    Out h, out;
    h.take(a[8], "sum_out", {M, K}, kHalf, x);
    const atom_desc d = desc(K, whole(a[5]), whole(a[6]), whole(a[10]));
    packed_out(out, a[9], M, d, x);
    ATOM_CALL(atom_add_quantize_act_packed, data(x), data(r), M, ld(x, M, K), ld(r, M, K), h.data(), ld(*h.t, M, K),
              gamma, eps, (const int32_t *)idx, &d, clip, out.data(), (size_t)out.t->numel());
    return tuple({&h, &out});
}

PyObject *swiglu_quantize_act_packed(Args a)
{
    const Tensor &g = device(a[0], kHalf, "gate"), &u = device(a[1], kHalf, "up");
    if (g.dim() != 2 || g.stride(1) != 1 || !covers(u, g))
        value_error("gate and up must be [M, K] with a contiguous last dimension");
    void *idx = maybe(a[2], kInt, "reorder_idx");
    const int64_t M = g.size(0), K = g.size(1);
    const float clip = real(a[5]);
    const atom_desc d = desc(K, whole(a[3]), whole(a[4]), whole(a[7]));
    Out out;
    packed_out(out, a[6], M, d, g);
    ATOM_CALL(atom_swiglu_quantize_act_packed, data(g), data(u), M, ld(g, M, K), ld(u, M, K), (const int32_t *)idx, &d,
              clip, out.data(), (size_t)out.t->numel());
    return out.give();
}

PyObject *w4a4_gemm_prepacked(Args a)
{
    const Tensor &ap = device(a[0], kByte, "a_packed"), &wp = device(a[2], kByte, "w_packed");
    const int64_t M = whole(a[1]), N = whole(a[3]), K = whole(a[4]), gs = whole(a[5]), O = whole(a[6]);
    const atom_desc d = desc(K, gs, O);
    if ((size_t)ap.numel() < atom_pack_weight_bytes(M, &d) || (size_t)wp.numel() < atom_pack_weight_bytes(N, &d))
        value_error("a packed operand is smaller than atom_pack_weight_bytes of its rows");
    Out y;
    y.take(a[7], "out", {M, N}, kHalf, ap);
    if (y.o) device(y.o, kHalf, "out");
    int32_t *partials = partial_sums(a[8], M, N, groups(K, gs));
    ATOM_CALL(atom_w4a4_gemm_prepacked, data(ap), M, data(wp), N, &d, y.data(), ld(*y.t, M, N), partials);
    return y.give();
}

PyObject *w4a4_gemm_packed(Args a)
{
    const Tensor &a4 = contiguous(a[0], kByte, "a_q4"), &a8 = contiguous(a[1], kChar, "a_q8"),
                 &as = contiguous(a[2], kHalf, "a_scale"), &wp = contiguous(a[3], kByte, "w_packed");
    rows_and_columns(a8, "a_q8");
    const int64_t M = a8.size(0), O = a8.size(1), K = 2 * a4.size(1) + O, N = whole(a[4]), gs = whole(a[5]);
    const atom_desc d = desc(K, gs, O);
    if ((size_t)wp.numel() < atom_pack_weight_bytes(N, &d)) value_error("w_packed is smaller than atom_pack_weight_bytes(N)");
    Out y;
    y.take(a[6], "out", {M, N}, kHalf, a4);
    if (y.o) device(y.o, kHalf, "out");
    int32_t *partials = partial_sums(a[7], M, N, groups(K, gs));
    const size_t need = atom_w4a4_gemm_packed_workspace_bytes(M, N, &d);
    Tensor own;
    const Tensor *w = a[8] == Py_None ? nullptr : &tensor(a[8], "workspace");
    if (!w || bytes(*w) < need) {
        own = make({(int64_t)std::max<size_t>(need, 1)}, kByte, a4);
        w = &own;
    }
    ATOM_CALL(atom_w4a4_gemm_packed, data(a4), data(a8), data(as), M, data(wp), N, &d, y.data(), ld(*y.t, M, N),
              partials, data(*w), bytes(*w));
    return y.give();
}

// A KV cache of one tensor: codes [B, Hkv, Tmax, D/2], scales and zero points [B, Hkv, Tmax].
struct Cache {
    Three t;
    const Tensor &codes, &scale, &zero;
    Cache(PyObject *o, const char *n0, const char *n1, const char *n2)
        : t(o), codes(device(t.item[0], kByte, n0)), scale(device(t.item[1], kHalf, n1)), zero(device(t.item[2], kShort, n2)) {}
    bool contiguous() const { return codes.is_contiguous() && scale.is_contiguous() && zero.is_contiguous(); }
    bool shaped(int64_t B, int64_t H, int64_t T, int64_t half) const
    {
        const int64_t s4[] = {B, H, T, half}, s3[] = {B, H, T};
        return codes.sizes() == at::IntArrayRef(s4) && scale.sizes() == at::IntArrayRef(s3) &&
               zero.sizes() == at::IntArrayRef(s3);
    }
};

PyObject *kv_quantize(Args a)
{
    const Tensor &x = device(a[0], kHalf, "x");
    const float clip = real(a[1]);
    if (x.dim() < 1 || !x.is_contiguous()) value_error("x must be contiguous [..., D]");
    const int64_t D = x.size(-1), R = D ? x.numel() / D : 0;
    if (a[2] == Py_None) {
        if (a[3] != Py_None) value_error("pos needs a cache to append to");
        auto lead = x.sizes().slice(0, (size_t)x.dim() - 1);
        c10::SmallVector<int64_t, 8> cshape(lead.begin(), lead.end());
        cshape.push_back(D / 2);
        Out c, sc, z;
        c.fresh(make(at::IntArrayRef(cshape), kByte, x));
        sc.fresh(make(lead, kHalf, x));
        z.fresh(make(lead, kShort, x));
        ATOM_CALL(atom_kv_quantize, data(x), R, D, (int32_t)D, clip, nullptr, 0, 0, c.data(), sc.data(), z.data());
        return tuple({&c, &sc, &z});
    }
    const Cache k(a[2], "cache codes", "cache scale", "cache zero");
    if (a[3] == Py_None) value_error("appending to a cache needs pos");
    const Tensor &pos = device(a[3], kInt, "pos");
    if (x.dim() != 3 || k.codes.dim() != 4 || !k.contiguous())
        value_error("x must be [B, Hkv, D] and the cache contiguous [B, Hkv, Tmax, ...]");
    const int64_t B = k.codes.size(0), H = k.codes.size(1), T = k.codes.size(2);
    if (x.size(0) != B || x.size(1) != H || k.codes.size(3) * 2 != D || !k.shaped(B, H, T, k.codes.size(3)) ||
        pos.dim() != 1 || pos.size(0) != B || !pos.is_contiguous())
        value_error("cache, x and pos shapes disagree");
    ATOM_CALL(atom_kv_quantize, data(x), R, D, (int32_t)D, clip, (const int32_t *)data(pos), (int32_t)H, T,
              data(k.codes), data(k.scale), data(k.zero));
    return PyTuple_Pack(3, k.t.item[0], k.t.item[1], k.t.item[2]);
}

PyObject *kv_quantize_pair(Args a)
{
    const Tensor &pos = device(a[4], kInt, "pos");
    const float clip = real(a[5]);
    const Tensor &k = device(a[0], kHalf, "k");
    const Cache kc(a[2], "k cache codes", "k cache scale", "k cache zero");
    if (k.dim() != 3 || kc.codes.dim() != 4 || !k.is_contiguous() || !kc.contiguous())
        value_error("k must be contiguous [B, Hkv, D] and its cache contiguous [B, Hkv, Tmax, ...]");
    const Tensor &v = device(a[1], kHalf, "v");
    const Cache vc(a[3], "v cache codes", "v cache scale", "v cache zero");
    if (v.dim() != 3 || vc.codes.dim() != 4 || !v.is_contiguous() || !vc.contiguous())
        value_error("v must be contiguous [B, Hkv, D] and its cache contiguous [B, Hkv, Tmax, ...]");
    const int64_t B = kc.codes.size(0), H = kc.codes.size(1), T = kc.codes.size(2), D = k.size(2);
    if (k.size(0) != B || k.size(1) != H || v.sizes() != k.sizes() || !kc.shaped(B, H, T, D / 2) ||
        !vc.shaped(B, H, T, D / 2))
        value_error("cache and row shapes disagree");
    if (pos.dim() != 1 || pos.size(0) != B || !pos.is_contiguous()) value_error("pos must be contiguous int32 [B]");
    ATOM_CALL(atom_kv_quantize_pair, data(k), data(v), B * H, D, (int32_t)D, clip, (const int32_t *)data(pos),
              (int32_t)H, T, data(kc.codes), data(kc.scale), data(kc.zero), data(vc.codes), data(vc.scale),
              data(vc.zero));
    return PyTuple_Pack(2, a[2], a[3]);
}

// a: q, k_cache, v_cache, seq_len, sm_scale, out, and (not the static form) workspace
PyObject *attention(Args a, bool fixed)
{
    const Tensor &q = device(a[0], kHalf, "q"), &len = device(a[3], kInt, "seq_len");
    if (q.dim() != 3 || !q.is_contiguous()) value_error("q must be contiguous [B, H, D]");
    const int64_t B = q.size(0), H = q.size(1), D = q.size(2);
    const Cache k(a[1], "k codes", "k scale", "k zero"), v(a[2], "v codes", "v scale", "v zero");
    const Tensor *all[] = {&k.codes, &v.codes, &k.scale, &v.scale, &k.zero, &v.zero};
    const char *names[] = {"k codes", "v codes", "k scale", "v scale", "k zero", "v zero"};
    for (int i = 0; i < 6; ++i)
        if (!all[i]->is_contiguous()) value_error(names[i], "must be contiguous");
    if (k.codes.dim() != 4 || k.codes.size(0) != B || k.codes.size(3) * 2 != D) value_error("k codes must be [B, Hkv, Tmax, D/2]");
    const int64_t Hkv = k.codes.size(1), T = k.codes.size(2);
    if (!k.shaped(B, Hkv, T, D / 2) || !v.shaped(B, Hkv, T, D / 2) || len.dim() != 1 || len.size(0) != B ||
        !len.is_contiguous())
        value_error("cache and seq_len shapes disagree");
    Out out;
    out.take(a[5], "out", {B, H, D}, kHalf, q);
    if (out.o) {
        device(out.o, kHalf, "out");
        if (out.t->sizes() != q.sizes() || !out.t->is_contiguous()) value_error("out must be contiguous [B, H, D]");
    }
    const float sm = real(a[4]);
    const int32_t *n = (const int32_t *)data(len);
    if (fixed) {
        ATOM_CALL(atom_decode_attention_kv4_static, data(q), (int32_t)B, (int32_t)H, (int32_t)Hkv, (int32_t)D, T, n,
                  data(k.codes), data(k.scale), data(k.zero), data(v.codes), data(v.scale), data(v.zero), sm,
                  out.data());
        return out.give();
    }
    const size_t need = atom_decode_attention_kv4_workspace_bytes((int32_t)B, (int32_t)H, (int32_t)Hkv, (int32_t)D, T);
    Tensor own;
    const Tensor *w = a[6] == Py_None ? nullptr : &tensor(a[6], "workspace");
    if (need && (!w || bytes(*w) < need)) {
        own = make({(int64_t)need}, kByte, q);
        w = &own;
    }
    ATOM_CALL(atom_decode_attention_kv4, data(q), (int32_t)B, (int32_t)H, (int32_t)Hkv, (int32_t)D, T, n, data(k.codes),
              data(k.scale), data(k.zero), data(v.codes), data(v.scale), data(v.zero), sm, out.data(),
              w ? data(*w) : nullptr, w ? bytes(*w) : 0);
    return out.give();
}

PyObject *decode_attention_kv4(Args a) { return attention(a, false); }
PyObject *decode_attention_kv4_static(Args a) { return attention(a, true); }

PyObject *mx_quantize_act(Args a)
{
    const Tensor &x = device(a[0], kHalf, "x"), &idx = device(a[3], kInt, "reorder_idx");
    void *gamma = maybe(a[1], kHalf, "gamma");
    matrix(x, "x must be [M, K] with a contiguous last dimension");
    const int64_t M = x.size(0), K = x.size(1), O = whole(a[4]);
    const float eps = real(a[2]), clip = real(a[5]);
    Out q4, q8, e8;
    if (a[6] == Py_None) {                     // step-major: [K step][row][64 bytes], scales [128-channel slab][row][4 bytes]
        q4.fresh(make({(K - O) / 128, M, 64}, kByte, x));
        q8.fresh(make({O / 64, M, 64}, kByte, x));
        e8.fresh(make({K / 128, M, 4}, kByte, x));
    } else {
        Three t(a[6]);
        q4.given(t.item[0], "q4");
        q8.given(t.item[1], "q8");
        e8.given(t.item[2], "e8");
    }
    const atom_desc d = desc(K, 32, O);
    ATOM_CALL(atom_mx_quantize_act, data(x), M, ld(x, M, K), gamma, eps, (const int32_t *)data(idx), &d, clip,
              q4.data(), q8.data(), e8.data());
    return tuple({&q4, &q8, &e8});
}

PyObject *mx_gemm(Args a)
{
    const Tensor &a4 = contiguous(a[0], kByte, "a_q4"), &a8 = contiguous(a[1], kByte, "a_q8"),
                 &ae = contiguous(a[2], kByte, "a_e8"), &w4 = contiguous(a[3], kByte, "w_q4"),
                 &w8 = contiguous(a[4], kByte, "w_q8"), &we = contiguous(a[5], kByte, "w_e8");
    if (a4.dim() != 3 || a8.dim() != 3 || w4.dim() != 3 || w8.dim() != 3)
        value_error("operands must be the step-major arrays atom_mx_quantize_* produce");
    const int64_t M = a8.size(1), N = w8.size(1), O = a8.size(0) * 64, K = a4.size(0) * 128 + O;
    const int64_t sa[] = {K / 128, M, 4}, sw[] = {K / 128, N, 4};
    if (w4.size(0) != a4.size(0) || w8.size(0) != a8.size(0) || a4.size(1) != M || w4.size(1) != N ||
        ae.sizes() != at::IntArrayRef(sa) || we.sizes() != at::IntArrayRef(sw))
        value_error("activation and weight code shapes disagree");
    Out y;
    y.take(a[6], "out", {M, N}, kHalf, a4);
    if (y.o) device(y.o, kHalf, "out");
    const atom_desc d = desc(K, 32, O);
    ATOM_CALL(atom_mx_gemm, data(a4), data(a8), data(ae), M, data(w4), data(w8), data(we), N, &d, y.data(),
              ld(*y.t, M, N));
    return y.give();
}

// One python-callable function of n positional arguments.
template <PyObject *(*F)(Args), int n>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    if (nargs != n) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", n, nargs);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Raised &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

PyObject *set_error(PyObject *, PyObject *cls)
{
    Py_INCREF(cls);
    Py_XDECREF(g_atom_error);
    g_atom_error = cls;
    Py_RETURN_NONE;
}

#define ENTRY(f, n) {#f, (PyCFunction)(void (*)(void))&entry<f, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    ENTRY(quantize_act, 9), ENTRY(add_quantize_act, 11), ENTRY(swiglu_quantize_act, 8), ENTRY(w4a4_gemm, 10),
    ENTRY(w4a4_gemm_decode_tiled, 8), ENTRY(decode_linear, 12), ENTRY(decode_linear_coop, 13), ENTRY(pack_act, 5),
    ENTRY(quantize_act_packed, 9), ENTRY(add_quantize_act_packed, 11), ENTRY(swiglu_quantize_act_packed, 8),
    ENTRY(w4a4_gemm_prepacked, 9), ENTRY(w4a4_gemm_packed, 9), ENTRY(kv_quantize, 4), ENTRY(kv_quantize_pair, 6),
    ENTRY(decode_attention_kv4, 7), ENTRY(decode_attention_kv4_static, 6), ENTRY(mx_quantize_act, 7), ENTRY(mx_gemm, 7),
    {"set_error", set_error, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
