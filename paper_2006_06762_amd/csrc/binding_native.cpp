// The operators of binding.py for the calls that programs make over and over: plain float32 GPU tensors, a descriptor within
// its fields' ranges.  Anything else (and every error) goes to the Python function of the same
// name, so what is accepted, refused and raised is decided there.
//
// Marshalling in Python took 1.6 to 2.2 us of a call, more than the launch: back to back on the GPU 128 x 128 x 128 ran every 4.6
// us where the launches alone allow 2.8, a depthwise 97 x 8 x 8 every 4.8 of 2.5.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <string>
#include <unordered_map>

#include "anr.h"

namespace {

// ---- what binding.py hands over (setup): its functions, the library's entry points
enum Op { GEMM, CONV2D, CONV_BN_RELU, CONV2D_PACKED, CONV_BN_RELU_PACKED, DWCONV, TBG, TBS, NRM, OPS };
PyObject* g_python[OPS];
using Call3 = anr_status (*)(const void*, const void*, const void*, void*, void*, size_t, void*);
using CallBn = anr_status (*)(const void*, const void*, const void*, const void*, const void*, const void*, const void*, float, void*, void*, size_t, void*);
using CallNrm = anr_status (*)(const void*, const void*, void*, void*, size_t, void*);
using CallFastSize = anr_status (*)(const void*, size_t*);
using CallSize = anr_status (*)(int, const void*, size_t*);
void* g_entry[OPS];
CallFastSize g_fast_size;
CallSize g_size;

// A tensor that is memory on a GPU and nothing else: no subclass, no wrapper of a transform, float32.
const at::Tensor* plain(PyObject* o, at::ScalarType type = at::kFloat)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined()) return nullptr;
    const c10::TensorImpl* impl = t.unsafeGetTensorImpl();
    constexpr c10::DispatchKeySet usual({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::AutocastCUDA, c10::DispatchKey::ADInplaceOrView});
    if ((impl->key_set().raw_repr() & ~usual.raw_repr()) != 0 || impl->has_symbolic_sizes_strides() || !impl->has_storage()) return nullptr;
    return t.is_cuda() && t.scalar_type() == type ? &t : nullptr;
}

void* data(const at::Tensor* t) { return t->mutable_data_ptr(); }

// Arguments by position and name, as a Python function with these parameters takes them; absent ones stay null.  False
// where that function would complain.
template <int N>
bool arguments(const char* const (&names)[N], int required, PyObject* const* args, Py_ssize_t n, PyObject* kwnames, PyObject* (&out)[N])
{
    if (n > N) return false;
    for (int i = 0; i < N; ++i) out[i] = i < n ? args[i] : nullptr;
    const Py_ssize_t named = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < named; ++k) {
        PyObject* const name = PyTuple_GET_ITEM(kwnames, k);
        int i = 0;
        while (i < N && PyUnicode_CompareWithASCIIString(name, names[i]) != 0) ++i;
        if (i == N || out[i]) return false;
        out[i] = args[n + k];
    }
    for (int i = 0; i < required; ++i)
        if (!out[i]) return false;
    return true;
}

bool int32(PyObject* o, int32_t* out)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    *out = (int32_t)v;
    return !overflow && v == *out;
}

bool pair(PyObject* o, int32_t absent, int32_t* a, int32_t* b)
{
    if (!o) {
        *a = *b = absent;
        return true;
    }
    return PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == 2 && int32(PyTuple_GET_ITEM(o, 0), a) && int32(PyTuple_GET_ITEM(o, 1), b);
}

bool fits(int64_t v, int32_t* out)
{
    *out = (int32_t)v;
    return v == *out;
}

// Element strides of a four-dimensional tensor, zeros for a packed one.
void strides4(const at::Tensor* t, int64_t* out)
{
    const bool packed = t->is_contiguous();
    for (int i = 0; i < 4; ++i) out[i] = packed ? 0 : t->stride(i);
}

struct Stream {
    c10::DeviceIndex device = c10::hip::current_device();
    hipStream_t stream = c10::hip::getCurrentHIPStream(device).stream();

    bool capturing() const
    {
        hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
        return hipStreamIsCapturing(stream, &status) != hipSuccess || status != hipStreamCaptureStatusNone;
    }
};

// Smaller workspaces of a thread, one for each of the eight streams it used last: asking the allocator takes 0.9 us of a call, which
// shows where the GPU is done before the host (norms 5.9 against 6.9 us; 1 x 32 x 28 x 28 -> 32, 1.7 MB, 7.9 against 8.3; from
// 8 MB on calls take 15 us and more).  Not of all threads together: another one's launches may come between those of a call.
// Given back when the thread ends.
class Kept {
public:
    static constexpr size_t kMost = (size_t)8 << 20;

    void* get(size_t need, const Stream& s)
    {
        Entry* e = entries_;
        while (e != entries_ + kStreams && !(e->ptr && e->device == s.device && e->stream == s.stream)) ++e;
        if (e == entries_ + kStreams) e = &entries_[next_++ % kStreams];
        else if (e->bytes >= need) return e->ptr;
        size_t bytes = (size_t)1 << 16;
        while (bytes < need) bytes *= 2;
        void* const ptr = c10::hip::HIPCachingAllocator::raw_alloc_with_stream(bytes, s.stream);
        if (e->ptr) c10::hip::HIPCachingAllocator::raw_delete(e->ptr);
        *e = {s.device, s.stream, ptr, bytes};
        return ptr;
    }
    ~Kept()
    {
        for (const Entry& e : entries_) try {
                if (e.ptr) c10::hip::HIPCachingAllocator::raw_delete(e.ptr);
            } catch (...) {                       // (at the end of the process)
            }
    }

private:
    static constexpr int kStreams = 8;
    struct Entry {
        c10::DeviceIndex device;
        hipStream_t stream;
        void* ptr;
        size_t bytes;
    };
    Entry entries_[kStreams] = {};
    unsigned next_ = 0;
};
thread_local Kept t_kept;

// Memory for the launches of one call (see _with_workspace in binding.py); none of zero bytes, and not in a capture, where
// Python looks after it.
struct Workspace {
    const bool here;
    const size_t bytes;
    void* const ptr;

    Workspace(size_t need, const Stream& s) : here(need == 0 || !s.capturing()), bytes(need), ptr(need && here ? take(need, s) : nullptr) {}
    ~Workspace()
    {
        if (ptr && bytes > Kept::kMost) c10::hip::HIPCachingAllocator::raw_delete(ptr);
    }
    Workspace(const Workspace&) = delete;
    Workspace& operator=(const Workspace&) = delete;

private:
    static void* take(size_t need, const Stream& s)
    {
        return need > Kept::kMost ? c10::hip::HIPCachingAllocator::raw_alloc_with_stream(need, s.stream) : t_kept.get(need, s);
    }
};

// Other threads run while the library is called, as they do around a ctypes call: a launch may wait for room in its queue.
struct WithoutGil {
    PyThreadState* const state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

template <typename Call, typename... Args>
bool accepted(Op op, Args... args)
{
    WithoutGil released;
    return reinterpret_cast<Call>(g_entry[op])(args...) == ANR_OK;
}

// anr_conv2d_fast_workspace_size of a descriptor, asked once for each of up to 4096.
size_t fast_size(const anr_conv_desc& d)
{
    static std::unordered_map<std::string, size_t> known;
    std::string key(reinterpret_cast<const char*>(&d), sizeof d);
    const auto at = known.find(key);
    if (at != known.end()) return at->second;
    size_t bytes = 0;
    if (g_fast_size(&d, &bytes) != ANR_OK) bytes = 0;       // (what is refused here is refused by the call itself)
    if (known.size() >= 4096) known.clear();
    known.emplace(std::move(key), bytes);
    return bytes;
}

bool conv_desc(const at::Tensor* x, const at::Tensor* w, const at::Tensor* y, PyObject* stride, PyObject* pad, PyObject* dil, PyObject* groups, PyObject* route,
               anr_conv_desc* d)
{
    if (x->dim() != 4 || w->dim() != 4 || y->dim() != 4 || !w->is_contiguous()) return false;
    std::memset(d, 0, sizeof *d);
    d->groups = 1;
    d->route = ANR_CONV_ROUTE_AUTO;
    d->layout = ANR_LAYOUT_NCHW;
    strides4(x, d->x_stride);
    strides4(y, d->y_stride);
    return fits(x->size(0), &d->N) && fits(x->size(1), &d->C) && fits(x->size(2), &d->H) && fits(x->size(3), &d->W) && fits(w->size(0), &d->K) &&
           fits(w->size(2), &d->R) && fits(w->size(3), &d->S) && pair(stride, 1, &d->stride_h, &d->stride_w) && pair(pad, 0, &d->pad_h, &d->pad_w) &&
           pair(dil, 1, &d->dil_h, &d->dil_w) && (!groups || int32(groups, &d->groups)) && (!route || int32(route, &d->route));
}

// The operators: true with the call made and accepted; false leaves it to Python, with nothing done.
bool run_gemm(PyObject* const* a)
{
    const at::Tensor *A = plain(a[0]), *B = plain(a[1]), *C = plain(a[2]);
    if (!A || !B || !C) return false;
    const int64_t n = A->dim();
    if ((n != 2 && n != 3) || B->dim() != n || C->dim() != n || A->stride(n - 1) != 1 || B->stride(n - 1) != 1 || C->stride(n - 1) != 1) return false;
    anr_gemm_desc d{};
    d.M = A->size(n - 2);
    d.K = A->size(n - 1);
    d.N = B->size(n - 1);
    d.lda = A->stride(n - 2);
    d.ldb = B->stride(n - 2);
    d.ldc = C->stride(n - 2);
    d.batch = n == 3 ? A->size(0) : 1;
    if (n == 3) {
        d.strideA = A->stride(0);
        d.strideB = B->stride(0);
        d.strideC = C->stride(0);
    }
    return accepted<Call3>(GEMM, &d, data(A), data(B), data(C), nullptr, 0, Stream().stream);
}

bool run_conv2d(PyObject* const* a)
{
    const at::Tensor *x = plain(a[0]), *w = plain(a[1]), *y = plain(a[2]);
    anr_conv_desc d;
    if (!x || !w || !y || (a[5] && a[5] != Py_None) || !conv_desc(x, w, y, a[3], a[4], a[6], a[7], a[8], &d)) return false;
    const Stream s;
    const Workspace ws(fast_size(d), s);
    return ws.here && accepted<Call3>(CONV2D, &d, data(x), data(w), data(y), ws.ptr, ws.bytes, s.stream);
}

bool run_conv_bn_relu(PyObject* const* a)
{
    const at::Tensor *x = plain(a[0]), *w = plain(a[1]), *y = plain(a[7]);
    anr_conv_desc d;
    if (!x || !w || !y || !PyFloat_CheckExact(a[6]) || (a[10] && a[10] != Py_None) || !conv_desc(x, w, y, a[8], a[9], a[11], a[12], a[13], &d)) return false;
    void* bn[4];
    for (int i = 0; i < 4; ++i) {
        const at::Tensor* const v = plain(a[2 + i]);
        if (!v || v->dim() != 1 || v->size(0) != d.K || !v->is_contiguous()) return false;
        bn[i] = data(v);
    }
    const Stream s;
    const Workspace ws(fast_size(d), s);
    return ws.here && accepted<CallBn>(CONV_BN_RELU, &d, data(x), data(w), bn[0], bn[1], bn[2], bn[3], (float)PyFloat_AS_DOUBLE(a[6]), data(y), ws.ptr,
                                       ws.bytes, s.stream);
}

bool run_packed(Op op, PyObject* const* a)
{
    const at::Tensor *x = plain(a[1]), *pack = plain(a[2], at::kByte), *y = plain(a[3]);
    if (!x || !pack || !y || (a[4] && a[4] != Py_None) || x->dim() != 4 || y->dim() != 4 || !x->is_contiguous() || !PyObject_CheckBuffer(a[0])) return false;
    Py_buffer view;
    if (PyObject_GetBuffer(a[0], &view, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return false;
    }
    anr_conv_desc d;
    const bool whole = view.len == (Py_ssize_t)sizeof d;
    if (whole) std::memcpy(&d, view.buf, sizeof d);
    PyBuffer_Release(&view);
    if (!whole) return false;
    for (int i = 0; i < 4; ++i) d.x_stride[i] = 0;
    strides4(y, d.y_stride);
    const Stream s;
    const Workspace ws(fast_size(d), s);
    return ws.here && accepted<Call3>(op, &d, data(x), data(pack), data(y), ws.ptr, ws.bytes, s.stream);
}

bool run_dwconv(PyObject* const* a)
{
    const at::Tensor *x = plain(a[0]), *w = plain(a[1]), *y = plain(a[2]);
    anr_conv_desc d;
    if (!x || !w || !y || !conv_desc(x, w, y, a[3], a[4], a[5], nullptr, nullptr, &d)) return false;
    return accepted<Call3>(DWCONV, &d, data(x), data(w), data(y), nullptr, 0, Stream().stream);
}

bool run_scores(Op op, PyObject* const* a)
{
    const at::Tensor *q = plain(a[0]), *k = plain(a[1]), *out = plain(a[2]);
    if (!q || !k || !out || q->dim() != 4 || k->dim() != 4 || out->dim() != 4) return false;
    anr_tbg_desc d{};
    if (!fits(q->size(0), &d.B) || !fits(q->size(1), &d.S) || !fits(q->size(2), &d.H) || !fits(q->size(3), &d.D)) return false;
    strides4(q, d.q_stride);
    strides4(k, d.k_stride);
    strides4(out, d.o_stride);
    return accepted<Call3>(op, &d, data(q), data(k), data(out), nullptr, 0, Stream().stream);
}

bool run_nrm(PyObject* const* a)
{
    const at::Tensor *x = plain(a[0]), *out = plain(a[1]);
    if (!x || !out || (a[2] && a[2] != Py_None)) return false;
    const int64_t n = x->dim();
    if ((n != 2 && n != 3) || x->stride(n - 1) != 1 || !out->is_contiguous()) return false;
    anr_nrm_desc d{};
    d.N = x->size(n - 2);
    d.M = x->size(n - 1);
    d.ld = x->stride(n - 2);
    d.batch = n == 3 ? x->size(0) : 1;
    d.stride = d.batch > 1 ? x->stride(0) : 0;
    if (out->numel() != d.batch) return false;
    size_t need = 0;
    if (g_size(ANR_OP_NRM, &d, &need) != ANR_OK) return false;
    const Stream s;
    const Workspace ws(need, s);
    return ws.here && accepted<CallNrm>(NRM, &d, data(x), data(out), ws.ptr, ws.bytes, s.stream);
}

// Parameters of each operator, the required ones first, and which of them it returns.
const char* const kGemm[] = {"A", "B", "C"};
const char* const kConv[] = {"x", "w", "y", "stride", "pad", "ws", "dil", "groups", "route"};
const char* const kConvBn[] = {"x", "w", "gamma", "beta", "mean", "var", "eps", "y", "stride", "pad", "ws", "dil", "groups", "route"};
const char* const kPacked[] = {"desc", "x", "pack", "y", "ws"};
const char* const kDw[] = {"x", "w", "y", "stride", "pad", "dil"};
const char* const kScores[] = {"q", "k", "out"};
const char* const kNrm[] = {"x", "out", "ws"};

template <int OP, int N, typename Run>
PyObject* call(const char* const (&names)[N], int required, int result, Run run, PyObject* const* args, Py_ssize_t n, PyObject* kwnames)
{
    PyObject* a[N];
    if (!g_python[OP]) {
        PyErr_SetString(PyExc_RuntimeError, "the operators are those of paper_2006_06762_amd.binding, which is not imported");
        return nullptr;
    }
    try {
        if (!at::impl::torch_function_mode_enabled() && arguments(names, required, args, n, kwnames, a) && run(a)) {
            Py_INCREF(a[result]);
            return a[result];
        }
    } catch (...) {
        // (memory that cannot be had: Python raises it)
    }
    if (PyErr_Occurred()) PyErr_Clear();
    return PyObject_Vectorcall(g_python[OP], args, (size_t)n, kwnames);
}

#define ANR_OPERATOR(fn, op, names, required, result, ...)                                        \
    PyObject* fn(PyObject*, PyObject* const* args, Py_ssize_t n, PyObject* kwnames)               \
    {                                                                                             \
        return call<op>(names, required, result, [](PyObject* const* a) { return __VA_ARGS__; }, args, n, kwnames); \
    }
ANR_OPERATOR(py_gemm, GEMM, kGemm, 3, 2, run_gemm(a))
ANR_OPERATOR(py_conv2d, CONV2D, kConv, 3, 2, run_conv2d(a))
ANR_OPERATOR(py_conv_bn_relu, CONV_BN_RELU, kConvBn, 8, 7, run_conv_bn_relu(a))
ANR_OPERATOR(py_conv2d_packed, CONV2D_PACKED, kPacked, 4, 3, run_packed(CONV2D_PACKED, a))
ANR_OPERATOR(py_conv_bn_relu_packed, CONV_BN_RELU_PACKED, kPacked, 4, 3, run_packed(CONV_BN_RELU_PACKED, a))
ANR_OPERATOR(py_dwconv, DWCONV, kDw, 3, 2, run_dwconv(a))
ANR_OPERATOR(py_tbg, TBG, kScores, 3, 2, run_scores(TBG, a))
ANR_OPERATOR(py_tbs, TBS, kScores, 3, 2, run_scores(TBS, a))
ANR_OPERATOR(py_nrm, NRM, kNrm, 2, 1, run_nrm(a))
#undef ANR_OPERATOR

// setup(functions, entries, fast_size, size): tuples in the order of the operators, entry points as integers.
PyObject* py_setup(PyObject*, PyObject* args)
{
    PyObject *functions, *entries, *fast_size, *size;
    if (!PyArg_ParseTuple(args, "O!O!OO", &PyTuple_Type, &functions, &PyTuple_Type, &entries, &fast_size, &size)) return nullptr;
    if (PyTuple_GET_SIZE(functions) != OPS || PyTuple_GET_SIZE(entries) != OPS) {
        PyErr_SetString(PyExc_ValueError, "one function and one entry point per operator");
        return nullptr;
    }
    for (int i = 0; i < OPS; ++i) {
        g_entry[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(entries, i));
        if (!g_entry[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
            return nullptr;
        }
        Py_XSETREF(g_python[i], Py_NewRef(PyTuple_GET_ITEM(functions, i)));
    }
    g_fast_size = reinterpret_cast<CallFastSize>(PyLong_AsVoidPtr(fast_size));
    g_size = reinterpret_cast<CallSize>(PyLong_AsVoidPtr(size));
    if (!g_fast_size || !g_size) return nullptr;
    Py_RETURN_NONE;
}

PyCFunction as_cfunction(PyObject* (*f)(PyObject*, PyObject* const*, Py_ssize_t, PyObject*)) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }

PyMethodDef g_methods[] = {
    {"gemm", as_cfunction(py_gemm), METH_FASTCALL | METH_KEYWORDS,
     "gemm(A, B, C)\n--\n\nC = A.B.  A [M,K] / [b,M,K], B [K,N] / [b,K,N], C [M,N] / [b,M,N]; last dim contiguous."},
    {"conv2d", as_cfunction(py_conv2d), METH_FASTCALL | METH_KEYWORDS,
     "conv2d(x, w, y, stride=(1, 1), pad=(0, 0), ws=None, dil=(1, 1), groups=1, route=0)\n--\n\n"
     "y = conv2d(x, w); x [N,C,H,W], w [K,C/groups,R,S] packed, y [N,K,OH,OW] (may be strided views).\n"
     "ws: optional workspace tensor of at least workspace_size(ANR_OP_CONV2D, desc) bytes; with fewer than\n"
     "conv2d_fast_workspace_size(desc) the kernel that conv2d_route reports runs."},
    {"conv_bn_relu", as_cfunction(py_conv_bn_relu), METH_FASTCALL | METH_KEYWORDS,
     "conv_bn_relu(x, w, gamma, beta, mean, var, eps, y, stride=(1, 1), pad=(0, 0), ws=None, dil=(1, 1), groups=1, route=0)\n--\n\n"
     "y = relu(batch norm(conv2d(x, w))) with the batch norm's vectors of K floats."},
    {"conv2d_packed", as_cfunction(py_conv2d_packed), METH_FASTCALL | METH_KEYWORDS,
     "conv2d_packed(desc, x, pack, y, ws=None)\n--\n\n"
     "conv2d with weights from conv2d_pack_weights (desc: the descriptor it returned).  x may be a strided view; one\n"
     "whose rows are no whole 16-byte units is copied first where the pack is in the patch kernel's order."},
    {"conv_bn_relu_packed", as_cfunction(py_conv_bn_relu_packed), METH_FASTCALL | METH_KEYWORDS,
     "conv_bn_relu_packed(desc, x, pack, y, ws=None)\n--\n\nconv + batch norm + ReLU with a pack made with bn=(gamma, beta, mean, var)."},
    {"dwconv", as_cfunction(py_dwconv), METH_FASTCALL | METH_KEYWORDS,
     "dwconv(x, w, y, stride=(1, 1), pad=(0, 0), dil=(1, 1))\n--\n\nDepthwise convolution: x [N,C,H,W], w [C,1,R,S] packed, y [N,C,OH,OW]."},
    {"tbg", as_cfunction(py_tbg), METH_FASTCALL | METH_KEYWORDS,
     "tbg(q, k, out)\n--\n\nout[b,h,i,j] = sum_d q[b,i,h,d] k[b,j,h,d]; q,k [B,S,H,D], out [B,H,S,S]."},
    {"tbs", as_cfunction(py_tbs), METH_FASTCALL | METH_KEYWORDS, "tbs(q, k, out)\n--\n\ntbg followed by a softmax over the last axis."},
    {"nrm", as_cfunction(py_nrm), METH_FASTCALL | METH_KEYWORDS,
     "nrm(x, out, ws=None)\n--\n\nout[b] = sqrt(sum of squares of x[b]).  x [N,M] or [b,N,M] with unit column stride, out [1] / [b]."},
    {"setup", py_setup, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&g_module); }
