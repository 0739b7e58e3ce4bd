"""Binding of libanr.so: argument marshalling only, in Python over ctypes and, for the operators' usual calls, in the
extension module ``_native`` (csrc/binding_native.cpp).

Function names and arguments mirror ``include/anr.h``.  Every tensor argument
is a torch CUDA tensor (float32); torch is used for device memory and for the
current HIP stream, nothing else.  There is no CPU path: if the library has not
been built, importing this module raises.
"""
import ctypes
import os
import struct

# torch ships its own HIP runtime (libamdhip64.so.7).  It must be in the process before
# libanr.so is opened, so that the library binds to that same runtime instance: streams
# and device pointers are only meaningful inside the runtime that created them.
import torch  # noqa: F401

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libanr.so")

if not all(os.path.exists(p) for p in (LIB_PATH, os.path.join(_HERE, "_native.so"))):
    raise ImportError(
        "%s or _native.so is missing: build it with `python -m paper_2006_06762_amd.build` "
        "(there is no fallback path)" % LIB_PATH)

_lib = ctypes.CDLL(LIB_PATH)

from paper_2006_06762_amd import _native  # noqa: E402

ANR_OK, ANR_ERR_NULL, ANR_ERR_INVALID_ARG, ANR_ERR_UNSUPPORTED, ANR_ERR_WORKSPACE, ANR_ERR_LAUNCH = range(6)
ANR_LAYOUT_NCHW = 0
ANR_OP_GEMM, ANR_OP_CONV2D, ANR_OP_CONV_BN_RELU, ANR_OP_DWCONV, ANR_OP_TBG, ANR_OP_TBS, ANR_OP_NRM = range(7)

EXPORTS = ("anr_gemm", "anr_conv2d", "anr_conv2d_noalloc", "anr_conv2d_packed_size", "anr_conv2d_pack_weights",
           "anr_conv2d_packed", "anr_conv_bn_relu_packed", "anr_conv_bn_relu", "anr_dwconv", "anr_tbg", "anr_tbs", "anr_nrm",
           "anr_workspace_size", "anr_conv2d_fast_workspace_size", "anr_conv2d_route", "anr_status_string", "anr_version", "anr_last_hip_error",
           "anr_last_hip_error_string")


class GemmDesc(ctypes.Structure):
    _fields_ = [("M", ctypes.c_int64), ("N", ctypes.c_int64), ("K", ctypes.c_int64),
                ("lda", ctypes.c_int64), ("ldb", ctypes.c_int64), ("ldc", ctypes.c_int64),
                ("batch", ctypes.c_int64),
                ("strideA", ctypes.c_int64), ("strideB", ctypes.c_int64), ("strideC", ctypes.c_int64)]


class ConvDesc(ctypes.Structure):
    _fields_ = [("N", ctypes.c_int32), ("C", ctypes.c_int32), ("H", ctypes.c_int32), ("W", ctypes.c_int32),
                ("K", ctypes.c_int32), ("R", ctypes.c_int32), ("S", ctypes.c_int32),
                ("stride_h", ctypes.c_int32), ("stride_w", ctypes.c_int32),
                ("pad_h", ctypes.c_int32), ("pad_w", ctypes.c_int32),
                ("dil_h", ctypes.c_int32), ("dil_w", ctypes.c_int32),
                ("layout", ctypes.c_int32),
                ("x_stride", ctypes.c_int64 * 4), ("y_stride", ctypes.c_int64 * 4),
                ("groups", ctypes.c_int32), ("route", ctypes.c_int32)]


class ConvRoute(ctypes.Structure):
    _fields_ = [("kernel", ctypes.c_int32), ("tile_m", ctypes.c_int32), ("tile_n", ctypes.c_int32),
                ("ksplit", ctypes.c_int32), ("wave_groups", ctypes.c_int32), ("work_groups", ctypes.c_int32),
                ("workspace_bytes", ctypes.c_uint64)]


ANR_CONV_ROUTE_AUTO, ANR_CONV_ROUTE_PATCH, ANR_CONV_ROUTE_GENERAL = 0, 1, 2
ANR_CONV_KERNEL_PATCH, ANR_CONV_KERNEL_TAPS, ANR_CONV_KERNEL_BIGTAPS, ANR_CONV_KERNEL_GATHER, \
    ANR_CONV_KERNEL_DIRECT, ANR_CONV_KERNEL_POINTWISE = 1, 2, 3, 4, 5, 6


class NrmDesc(ctypes.Structure):
    _fields_ = [("N", ctypes.c_int64), ("M", ctypes.c_int64), ("ld", ctypes.c_int64),
                ("batch", ctypes.c_int64), ("stride", ctypes.c_int64)]


class TbgDesc(ctypes.Structure):
    _fields_ = [("B", ctypes.c_int32), ("S", ctypes.c_int32), ("H", ctypes.c_int32), ("D", ctypes.c_int32),
                ("q_stride", ctypes.c_int64 * 4), ("k_stride", ctypes.c_int64 * 4),
                ("o_stride", ctypes.c_int64 * 4)]


_vp = ctypes.c_void_p
_lib.anr_gemm.argtypes = [ctypes.POINTER(GemmDesc), _vp, _vp, _vp, _vp, ctypes.c_size_t, _vp]
_lib.anr_conv2d.argtypes = [ctypes.POINTER(ConvDesc), _vp, _vp, _vp, _vp, ctypes.c_size_t, _vp]
_lib.anr_conv2d_noalloc.argtypes = [ctypes.POINTER(ConvDesc), _vp, _vp, _vp, _vp]
_lib.anr_conv2d_packed_size.argtypes = [ctypes.POINTER(ConvDesc), ctypes.POINTER(ctypes.c_size_t)]
_lib.anr_conv2d_pack_weights.argtypes = [ctypes.POINTER(ConvDesc), _vp, _vp, _vp, _vp, _vp, ctypes.c_float, _vp,
                                         ctypes.c_size_t, _vp]
_lib.anr_conv2d_packed.argtypes = [ctypes.POINTER(ConvDesc), _vp, _vp, _vp, _vp, ctypes.c_size_t, _vp]
_lib.anr_conv_bn_relu_packed.argtypes = [ctypes.POINTER(ConvDesc), _vp, _vp, _vp, _vp, ctypes.c_size_t, _vp]
_lib.anr_conv_bn_relu.argtypes = [ctypes.POINTER(ConvDesc), _vp, _vp, _vp, _vp, _vp, _vp, ctypes.c_float,
                                  _vp, _vp, ctypes.c_size_t, _vp]
_lib.anr_dwconv.argtypes = [ctypes.POINTER(ConvDesc), _vp, _vp, _vp, _vp, ctypes.c_size_t, _vp]
_lib.anr_tbg.argtypes = [ctypes.POINTER(TbgDesc), _vp, _vp, _vp, _vp, ctypes.c_size_t, _vp]
_lib.anr_tbs.argtypes = [ctypes.POINTER(TbgDesc), _vp, _vp, _vp, _vp, ctypes.c_size_t, _vp]
_lib.anr_nrm.argtypes = [ctypes.POINTER(NrmDesc), _vp, _vp, _vp, ctypes.c_size_t, _vp]
_lib.anr_workspace_size.argtypes = [ctypes.c_int, _vp, ctypes.POINTER(ctypes.c_size_t)]
_lib.anr_conv2d_fast_workspace_size.argtypes = [ctypes.POINTER(ConvDesc), ctypes.POINTER(ctypes.c_size_t)]
_lib.anr_conv2d_route.argtypes = [ctypes.POINTER(ConvDesc), ctypes.POINTER(ConvRoute)]
for _name in ("anr_gemm", "anr_conv2d", "anr_conv2d_noalloc", "anr_conv2d_packed_size", "anr_conv2d_pack_weights",
              "anr_conv2d_packed", "anr_conv_bn_relu_packed", "anr_conv_bn_relu", "anr_dwconv", "anr_tbg", "anr_tbs",
              "anr_workspace_size", "anr_conv2d_fast_workspace_size"):
    getattr(_lib, _name).restype = ctypes.c_int
_lib.anr_status_string.argtypes = [ctypes.c_int]
_lib.anr_status_string.restype = ctypes.c_char_p
_lib.anr_version.argtypes = []
_lib.anr_version.restype = ctypes.c_int
_lib.anr_last_hip_error.argtypes = []
_lib.anr_last_hip_error.restype = ctypes.c_int
_lib.anr_last_hip_error_string.argtypes = []
_lib.anr_last_hip_error_string.restype = ctypes.c_char_p


class AnrError(RuntimeError):
    def __init__(self, status, where):
        self.status = status
        msg = "%s: %s (status %d)" % (where, status_string(status), status)
        if status == ANR_ERR_LAUNCH:
            msg += " [hip error %d: %s]" % (_lib.anr_last_hip_error(),
                                            _lib.anr_last_hip_error_string().decode())
        super().__init__(msg)


def raw():
    """The ctypes library handle, for tests that call the C ABI with hand-made arguments."""
    return _lib


def status_string(status: int) -> str:
    return _lib.anr_status_string(int(status)).decode()


def version() -> int:
    return int(_lib.anr_version())


def _check(status, where):
    if status != ANR_OK:
        raise AnrError(status, where)


# The operators' own handle on the library: the same functions with plain pointer arguments, so that a call
# passes integers and a packed descriptor as they are.  With ctypes structures, pointer objects and torch's
# Stream object around every call, the host took 8 us per launch, more than most of the small kernels run.
_fast = ctypes.CDLL(LIB_PATH)
_sz, _fl, _vp4 = ctypes.c_size_t, ctypes.c_float, [_vp] * 4
_fast.anr_gemm.argtypes = _vp4 + [_vp, _sz, _vp]
_fast.anr_conv2d.argtypes = _vp4 + [_vp, _sz, _vp]
_fast.anr_conv2d_noalloc.argtypes = _vp4 + [_vp]
_fast.anr_conv2d_packed.argtypes = _vp4 + [_vp, _sz, _vp]
_fast.anr_conv_bn_relu_packed.argtypes = _vp4 + [_vp, _sz, _vp]
_fast.anr_conv_bn_relu.argtypes = [_vp] * 7 + [_fl, _vp, _vp, _sz, _vp]
_fast.anr_dwconv.argtypes = _vp4 + [_vp, _sz, _vp]
_fast.anr_tbg.argtypes = _vp4 + [_vp, _sz, _vp]
_fast.anr_tbs.argtypes = _vp4 + [_vp, _sz, _vp]
_fast.anr_nrm.argtypes = [_vp] * 3 + [_vp, _sz, _vp]

_pack_gemm = struct.Struct("@10q").pack
_pack_conv = struct.Struct("@14i8q2i").pack
_pack_tbg = struct.Struct("@4i12q").pack
_pack_nrm = struct.Struct("@5q").pack
assert [struct.calcsize(f) for f in ("@10q", "@14i8q2i", "@4i12q", "@5q")] == \
    [ctypes.sizeof(t) for t in (GemmDesc, ConvDesc, TbgDesc, NrmDesc)]
_NO_STRIDES = (0, 0, 0, 0)
_f32 = torch.float32


def _ptr(t):
    if not isinstance(t, torch.Tensor) or t.dtype is not _f32 or not t.is_cuda:
        raise TypeError("expected a float32 CUDA tensor")
    return t.data_ptr()


def _stream():
    """torch's current stream on the current device, as the integer the library takes."""
    return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())


def conv_desc(x_shape, K, R, S, stride=(1, 1), pad=(0, 0), x_stride=None, y_stride=None, dil=(1, 1),
              layout=ANR_LAYOUT_NCHW, groups=1, route=ANR_CONV_ROUTE_AUTO) -> ConvDesc:
    N, C, H, W = x_shape
    d = ConvDesc(N, C, H, W, K, R, S, stride[0], stride[1], pad[0], pad[1], dil[0], dil[1], layout)
    d.groups = groups
    d.route = route
    if x_stride is not None:
        d.x_stride = (ctypes.c_int64 * 4)(*x_stride)
    if y_stride is not None:
        d.y_stride = (ctypes.c_int64 * 4)(*y_stride)
    return d


def _packed(t, shape):
    """True when tensor t is the packed row-major layout of `shape`."""
    return tuple(t.shape) == tuple(shape) and t.is_contiguous()


def workspace_size(op: int, desc) -> int:
    n = ctypes.c_size_t(0)
    _check(_lib.anr_workspace_size(op, ctypes.cast(ctypes.byref(desc), _vp), ctypes.byref(n)),
           "anr_workspace_size")
    return int(n.value)


def conv2d_route(desc: ConvDesc) -> ConvRoute:
    """Which kernel anr_conv2d would run for the descriptor (aligned pointers assumed) with workspace_size bytes,
    its tile, split and workspace need; host-side planning only.  The operators here give a layer
    conv2d_fast_workspace_size bytes: where that is more, it runs on pieces instead."""
    r = ConvRoute()
    _check(_lib.anr_conv2d_route(ctypes.byref(desc), ctypes.byref(r)), "anr_conv2d_route")
    return r


def conv2d_fast_workspace_size(desc: ConvDesc) -> int:
    """Bytes of workspace with which the convolutions run `desc` fastest."""
    n = ctypes.c_size_t(0)
    _check(_lib.anr_conv2d_fast_workspace_size(ctypes.byref(desc), ctypes.byref(n)), "anr_conv2d_fast_workspace_size")
    return int(n.value)


_fast_sizes = {}        # descriptor of a convolution, packed -> conv2d_fast_workspace_size


def _fast_size(desc):
    size = _fast_sizes.get(desc)
    if size is None:
        if len(_fast_sizes) >= 4096:
            _fast_sizes.clear()
        n = ctypes.c_size_t(0)
        # (a descriptor that is refused here is refused by the call itself)
        size = n.value if _lib.anr_conv2d_fast_workspace_size(ctypes.byref(ConvDesc.from_buffer_copy(desc)), ctypes.byref(n)) == ANR_OK else 0
        _fast_sizes[desc] = size
    return size


def _least_size(op, desc):
    """anr_workspace_size of a packed descriptor, zero for one that is refused (by the call itself then, too)."""
    n = ctypes.c_size_t(0)
    return n.value if _lib.anr_workspace_size(op, desc, ctypes.byref(n)) == ANR_OK else 0


def _allocate(need, op, desc, stream):
    """(address, bytes) of a workspace of `need` bytes, or where those cannot be had of anr_workspace_size."""
    if not need:
        return None, 0
    try:
        return torch.cuda.caching_allocator_alloc(need, stream=stream), need
    except torch.OutOfMemoryError:
        least = _least_size(op, desc)
        if least >= need:
            raise
    return _allocate(least, op, desc, stream)


def _only_replays_hold(buffer):
    """True in a capture that is not torch's own, whose graph has no pool: nothing but its replays knows of the buffer."""
    return torch.cuda.is_current_stream_capturing() and not any(
        s["address"] <= buffer < s["address"] + s["total_size"] for s in torch.cuda.memory_snapshot() if tuple(s["segment_pool_id"]) != (0, 0))


def _with_workspace(fn, name, op, desc, args, ws, desc_type=ConvDesc):
    """Calls fn(desc, *args, workspace, bytes, stream).  The workspace is the caller's tensor, else memory of torch's
    allocator for this call alone, with which a convolution runs fastest (at most 256 MB), or if there is no such room
    what it cannot do without.  It goes back as soon as the launches are enqueued: the allocator gives it to nothing but
    later work on the same stream, and a call that torch captures (torch.cuda.graph) has it from the graph's own pool,
    where nothing but the graph's later work gets it.  A call that is captured in another way keeps its memory for good;
    it had better bring a workspace.  (Not a buffer kept for the stream: a call is several launches, and another thread's
    may come between them; and a captured call would go on using it when it is replaced by a larger one, or when two
    graphs run at once.  The extension module keeps those of up to 8 MB for a thread and stream, outside captures.)"""
    stream = _stream()
    if ws is None:
        need = _fast_size(desc) if desc_type is ConvDesc else _least_size(op, desc)
        buffer, need = _allocate(need, op, desc, stream)
        try:
            status = fn(desc, *args, buffer, need, stream)
        finally:
            if buffer and not _only_replays_hold(buffer):
                torch.cuda.caching_allocator_delete(buffer)
    else:
        need = workspace_size(op, desc_type.from_buffer_copy(desc))
        size = ws.numel() * ws.element_size()
        fast = _fast_size(desc) if desc_type is ConvDesc else 0
        if ws.is_cuda and ws.is_contiguous() and (size >= need > 0 or size >= fast > 0):
            status = fn(desc, *args, ws.data_ptr(), size, stream)
        elif need == 0:
            status = fn(desc, *args, None, 0, stream)
        else:
            raise ValueError("workspace must be a contiguous CUDA tensor of at least %d bytes" % need)
    if status != ANR_OK:
        raise AnrError(status, name)


def _gemm(A, B, C):
    """C = A.B.  A [M,K] / [b,M,K], B [K,N] / [b,K,N], C [M,N] / [b,M,N]; last dim contiguous."""
    sa, sb, sc = A.stride(), B.stride(), C.stride()
    if len(sa) == 2:
        M, K = A.shape
        N = B.shape[1]
        d = _pack_gemm(M, N, K, sa[0], sb[0], sc[0], 1, 0, 0, 0)
    else:
        b, M, K = A.shape
        N = B.shape[2]
        d = _pack_gemm(M, N, K, sa[1], sb[1], sc[1], b, sa[0], sb[0], sc[0])
    if sa[-1] != 1 or sb[-1] != 1 or sc[-1] != 1:
        raise ValueError("innermost dimension must be contiguous")
    status = _fast.anr_gemm(d, _ptr(A), _ptr(B), _ptr(C), None, 0, _stream())
    if status != ANR_OK:
        raise AnrError(status, "anr_gemm")
    return C


def _conv_strides(t):
    return _NO_STRIDES if t.is_contiguous() else tuple(t.stride())


def _conv_packed_desc(x, w, y, stride, pad, dil, groups, route):
    """The descriptor of a call on x, w and y, as the bytes of an anr_conv_desc."""
    K, _, R, S = w.shape
    if not w.is_contiguous():
        raise ValueError("weights must be packed")
    N, C, H, W = x.shape
    xs, ys = _conv_strides(x), _conv_strides(y)
    try:
        return _pack_conv(N, C, H, W, K, R, S, stride[0], stride[1], pad[0], pad[1], dil[0], dil[1], ANR_LAYOUT_NCHW,
                          *xs, *ys, groups, route)
    except struct.error:        # numbers beyond the fields' range: as the structure takes them
        return bytes(conv_desc((N, C, H, W), K, R, S, stride, pad, xs, ys, dil=dil, groups=groups, route=route))


def _conv2d(x, w, y, stride=(1, 1), pad=(0, 0), ws=None, dil=(1, 1), groups=1, route=ANR_CONV_ROUTE_AUTO):
    """y = conv2d(x, w); x [N,C,H,W], w [K,C/groups,R,S] packed, y [N,K,OH,OW] (may be strided views).
    ws: optional workspace tensor of at least workspace_size(ANR_OP_CONV2D, desc) bytes; with fewer than
    conv2d_fast_workspace_size(desc) the kernel that conv2d_route reports runs."""
    d = _conv_packed_desc(x, w, y, stride, pad, dil, groups, route)
    _with_workspace(_fast.anr_conv2d, "anr_conv2d", ANR_OP_CONV2D, d, (_ptr(x), _ptr(w), _ptr(y)), ws)
    return y


STATIC_SCRATCH_BYTES = 16 << 20


def conv2d_noalloc(x, w, y, stride=(1, 1), pad=(0, 0), dil=(1, 1), groups=1, route=ANR_CONV_ROUTE_AUTO):
    """conv2d without a workspace argument: split reductions use the library's static scratch array."""
    d = _conv_packed_desc(x, w, y, stride, pad, dil, groups, route)
    _check(_fast.anr_conv2d_noalloc(d, _ptr(x), _ptr(w), _ptr(y), _stream()), "anr_conv2d_noalloc")
    return y


def conv2d_packed_size(desc: ConvDesc) -> int:
    n = ctypes.c_size_t(0)
    _check(_lib.anr_conv2d_packed_size(ctypes.byref(desc), ctypes.byref(n)), "anr_conv2d_packed_size")
    return int(n.value)


def conv2d_pack_weights(x_shape, w, stride=(1, 1), pad=(0, 0), bn=None, eps=0.0, dil=(1, 1), groups=1,
                        route=ANR_CONV_ROUTE_AUTO):
    """Packs w (and, with bn = (gamma, beta, mean, var), the folded batch norm) for the layer that
    x_shape, w and the geometry describe.  Returns (descriptor, pack): the pack is a new uint8 CUDA
    tensor (torch's allocations are 256-byte aligned) to hand to conv2d_packed / conv_bn_relu_packed."""
    K, _, R, S = w.shape
    if not w.is_contiguous():
        raise ValueError("weights must be packed OIHW")
    d = conv_desc(tuple(x_shape), K, R, S, stride, pad, dil=dil, groups=groups, route=route)
    pack = torch.empty(conv2d_packed_size(d), dtype=torch.uint8, device=w.device)
    vecs = [None] * 4 if bn is None else [_ptr(v) for v in bn]
    _check(_lib.anr_conv2d_pack_weights(ctypes.byref(d), _ptr(w), vecs[0], vecs[1], vecs[2], vecs[3],
                                        ctypes.c_float(eps), ctypes.c_void_p(pack.data_ptr()), pack.numel(), _stream()),
           "anr_conv2d_pack_weights")
    return d, pack


def _run_packed(fn, name, op, desc, x, pack, y, ws):
    d = ConvDesc.from_buffer_copy(desc)
    xs = d.x_stride = _conv_strides(x)
    if xs is not _NO_STRIDES and (xs[0] % 4 or xs[1] % 4 or xs[2] % 4 or xs[0] * x.shape[0] >= 1 << 29):
        # The order of a pack goes by its descriptor's strides: a view that would have made another one is copied
        # (the two orders always differ in size).
        if conv2d_packed_size(d) != conv2d_packed_size(desc):
            x = x.contiguous()
            d.x_stride = _NO_STRIDES
    d.y_stride = _conv_strides(y)
    _with_workspace(fn, name, op, bytes(d), (_ptr(x), pack.data_ptr(), _ptr(y)), ws)
    return y


def _conv2d_packed(desc, x, pack, y, ws=None):
    """conv2d with weights from conv2d_pack_weights (desc: the descriptor it returned).  x may be a strided view; one
    whose rows are no whole 16-byte units is copied first where the pack is in the patch kernel's order."""
    return _run_packed(_fast.anr_conv2d_packed, "anr_conv2d_packed", ANR_OP_CONV2D, desc, x, pack, y, ws)


def _conv_bn_relu_packed(desc, x, pack, y, ws=None):
    """conv + batch norm + ReLU with a pack made with bn=(gamma, beta, mean, var)."""
    return _run_packed(_fast.anr_conv_bn_relu_packed, "anr_conv_bn_relu_packed", ANR_OP_CONV_BN_RELU, desc, x, pack, y, ws)


def _conv_bn_relu(x, w, gamma, beta, mean, var, eps, y, stride=(1, 1), pad=(0, 0), ws=None, dil=(1, 1), groups=1,
                 route=ANR_CONV_ROUTE_AUTO):
    if not w.is_contiguous():
        raise ValueError("weights must be packed")
    K = w.shape[0]
    for v in (gamma, beta, mean, var):
        if v.shape != (K,) or not v.is_contiguous():
            raise ValueError("batch-norm vectors must be packed [K]")
    d = _conv_packed_desc(x, w, y, stride, pad, dil, groups, route)
    args = (_ptr(x), _ptr(w), _ptr(gamma), _ptr(beta), _ptr(mean), _ptr(var), eps, _ptr(y))
    _with_workspace(_fast.anr_conv_bn_relu, "anr_conv_bn_relu", ANR_OP_CONV_BN_RELU, d, args, ws)
    return y


def _dwconv(x, w, y, stride=(1, 1), pad=(0, 0), dil=(1, 1)):
    d = _conv_packed_desc(x, w, y, stride, pad, dil, 1, ANR_CONV_ROUTE_AUTO)
    _check(_fast.anr_dwconv(d, _ptr(x), _ptr(w), _ptr(y), None, 0, _stream()), "anr_dwconv")
    return y


def _tbg_desc(q, k, out):
    B, S, H, D = q.shape
    strides = _conv_strides(q), _conv_strides(k), _conv_strides(out)
    try:
        return _pack_tbg(B, S, H, D, *strides[0], *strides[1], *strides[2])
    except struct.error:        # numbers beyond the fields' range: as the structure takes them
        return bytes(TbgDesc(B, S, H, D, *strides))


def _tbg(q, k, out):
    """out[b,h,i,j] = sum_d q[b,i,h,d] k[b,j,h,d]; q,k [B,S,H,D], out [B,H,S,S]."""
    _check(_fast.anr_tbg(_tbg_desc(q, k, out), _ptr(q), _ptr(k), _ptr(out), None, 0, _stream()), "anr_tbg")
    return out


def _tbs(q, k, out):
    """tbg followed by a softmax over the last axis."""
    _check(_fast.anr_tbs(_tbg_desc(q, k, out), _ptr(q), _ptr(k), _ptr(out), None, 0, _stream()), "anr_tbs")
    return out


def _nrm(x, out, ws=None):
    """out[b] = sqrt(sum of squares of x[b]).  x [N,M] or [b,N,M] with unit column stride, out [1] / [b]."""
    if x.dim() == 2:
        N, M = x.shape
        b, st = 1, (0,) + tuple(x.stride())
    else:
        b, N, M = x.shape
        st = x.stride()
    if st[2] != 1 or not out.is_contiguous() or out.numel() != b:
        raise ValueError("x needs unit column stride and out one packed float per matrix")
    d = _pack_nrm(N, M, st[1], b, st[0] if b > 1 else 0)
    _with_workspace(_fast.anr_nrm, "anr_nrm", ANR_OP_NRM, d, (_ptr(x), _ptr(out)), ws, NrmDesc)
    return out


# The operators as programs call them: the functions above without Python's part in the usual case.
_OPERATORS = ("gemm", "conv2d", "conv_bn_relu", "conv2d_packed", "conv_bn_relu_packed", "dwconv", "tbg", "tbs", "nrm")
for _name in _OPERATORS:
    globals()["_" + _name].__name__ = globals()["_" + _name].__qualname__ = _name      # (what their errors say)
_native.setup(tuple(globals()["_" + n] for n in _OPERATORS),
              tuple(ctypes.cast(getattr(_fast, "anr_" + n), _vp).value for n in _OPERATORS),
              ctypes.cast(_fast.anr_conv2d_fast_workspace_size, _vp).value, ctypes.cast(_fast.anr_workspace_size, _vp).value)
from paper_2006_06762_amd._native import (gemm, conv2d, conv_bn_relu, conv2d_packed, conv_bn_relu_packed, dwconv, tbg, tbs,  # noqa: E402
                                          nrm)
for _name in _OPERATORS:
    globals()[_name].__module__ = __name__          # (where a pickle of one finds it again, in a process that has not imported torch)
