"""What a convolution runs with which workspace, without a GPU: the library's launches go to a recorder in place of the HIP
runtime's entry points."""
import ctypes
import subprocess
import sys
import threading

import pytest

from paper_2006_06762_amd import binding as B

RECORDER = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdio.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim;
static char log_[4096];
int hipLaunchKernel(const void* f, dim grid, dim block, void** args, size_t lds, void* stream)
{
    Dl_info at;
    if (!dladdr(f, &at) || !at.dli_sname || strlen(log_) + strlen(at.dli_sname) + 2 > sizeof log_) return 1;
    strcat(strcat(log_, at.dli_sname), " ");
    return 0;
}
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { return 0; }
int hipGetSymbolAddress(void** p, const void* s) { *p = (void*)0x100000; return 0; }
const char* launches(void) { static char out[4096]; strcpy(out, log_); log_[0] = 0; return out; }
"""

# reads "entry size N C H W K R S stride_h stride_w pad_h pad_w dil_h dil_w groups route", writes the status and the kernels
DRIVER = r"""
import ctypes, struct, sys
recorder = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
recorder.launches.restype = ctypes.c_char_p
lib = ctypes.CDLL(sys.argv[2])
at = ctypes.c_void_p(0x10000)
for line in sys.stdin:
    entry, size, *f = line.split()
    *geometry, groups, route = map(int, f)
    desc = struct.pack("@14i8q2i", *geometry, 0, *[0] * 8, groups, route)
    if entry == "anr_conv2d_noalloc":
        status = lib.anr_conv2d_noalloc(desc, at, at, at, None)
    else:
        status = lib.anr_conv2d(desc, at, at, at, at if int(size) else None, ctypes.c_size_t(int(size)), None)
    print(status, recorder.launches().decode(), flush=True)
"""

# (N, C, H, W, K, R, S, stride, pad, dil, groups), on pieces: less and more room for them than the plan without them needs
LAYERS = [(16, 256, 14, 14, 256, 3, 3, (1, 1), (1, 1), (1, 1), 1), (16, 64, 50, 50, 96, 5, 5, (2, 2), (2, 2), (1, 1), 1),
          (16, 32, 81, 81, 32, 5, 5, (1, 1), (2, 2), (1, 1), 1), (8, 128, 96, 96, 100, 3, 3, (1, 1), (1, 1), (1, 1), 1),
          (8, 512, 27, 12, 80, 7, 7, (2, 2), (6, 6), (2, 2), 4)]


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """launches(calls): (status, names of the kernels launched) of each call (entry, workspace, layer, route)."""
    at = tmp_path_factory.mktemp("recorder")
    (at / "recorder.c").write_text(RECORDER)
    subprocess.run(["gcc", "-shared", "-fPIC", "-Wall", str(at / "recorder.c"), "-o", str(at / "recorder.so"), "-ldl"], check=True)
    (at / "driver.py").write_text(DRIVER)

    def run(calls):
        text = "".join("%s %d %s\n" % (entry, size, " ".join(str(v) for v in (*l[:7], *l[7], *l[8], *l[9], l[10], route)))
                       for entry, size, l, route in calls)
        out = subprocess.run([sys.executable, str(at / "driver.py"), str(at / "recorder.so"), B.LIB_PATH], input=text, text=True, check=True,
                             capture_output=True).stdout
        return [(int(line.split()[0]), line.split()[1:]) for line in out.splitlines()]
    return run


def desc(l, route=B.ANR_CONV_ROUTE_AUTO):
    return B.conv_desc(l[:4], l[4], l[5], l[6], l[7], l[8], dil=l[9], groups=l[10], route=route)


def on_pieces(kernels):
    return any("split_operands" in k for k in kernels)


@pytest.mark.parametrize("layer", LAYERS)
def test_the_workspace_size_selects_the_kernel(launches, layer):
    """With anr_workspace_size() bytes the kernel that the route reports, as anr_conv2d_noalloc runs it; on pieces from the
    faster size on, and in between still the former."""
    d = desc(layer)
    least, fast, route = B.workspace_size(B.ANR_OP_CONV2D, d), B.conv2d_fast_workspace_size(d), B.conv2d_route(d)
    assert fast > least == route.workspace_bytes
    sizes = [least, fast - 16, fast, fast + 16, 1 << 29]
    got = launches([("anr_conv2d", s, layer, 0) for s in sizes] + [("anr_conv2d_noalloc", 0, layer, 0), ("anr_conv2d", max(least - 16, 0), layer, 0)])
    assert [s for s, _ in got[:5]] == [B.ANR_OK] * 5
    plain = got[0][1]
    family = {B.ANR_CONV_KERNEL_PATCH: "conv_patch", B.ANR_CONV_KERNEL_TAPS: "conv_taps", B.ANR_CONV_KERNEL_BIGTAPS: "conv_bigtaps",
              B.ANR_CONV_KERNEL_GATHER: "conv_gather"}[route.kernel]
    assert family in plain[0] and len(plain) == (2 if route.ksplit > 1 else 1)
    assert got[1][1] == plain
    assert all(on_pieces(k) for _, k in got[2:5])
    if least <= B.STATIC_SCRATCH_BYTES:
        assert got[5] == (B.ANR_OK, plain)
    else:
        assert got[5] == (B.ANR_ERR_WORKSPACE, [])
    assert got[6] == ((B.ANR_ERR_WORKSPACE, []) if least else (B.ANR_OK, plain))


def test_noalloc_refuses_what_is_more_than_its_array():
    """Before anything is launched or looked up, also where the pieces would fit."""
    l = LAYERS[1]
    assert B.workspace_size(B.ANR_OP_CONV2D, desc(l)) > B.STATIC_SCRATCH_BYTES
    at = ctypes.c_void_p(0x10000)
    assert B.raw().anr_conv2d_noalloc(ctypes.byref(desc(l)), at, at, at, None) == B.ANR_ERR_WORKSPACE


# ------------------------------------------------------------------ the binding's workspaces
class Allocator:
    """Stands for torch's: addresses in use are never handed out twice."""

    def __init__(self, monkeypatch):
        self.used, self.next = {}, 1 << 20
        self.most = 1 << 40              # that can be had at once
        self.capture = None              # or the pool that the capture in progress allocates from
        monkeypatch.setattr(B, "_stream", lambda: 7)
        monkeypatch.setattr(B.torch.cuda, "is_current_stream_capturing", lambda: self.capture is not None)
        monkeypatch.setattr(B.torch.cuda, "memory_snapshot", lambda: [{"address": p, "total_size": n, "segment_pool_id": self.capture or (0, 0)}
                                                                      for p, n in self.used.items()])
        monkeypatch.setattr(B.torch.cuda, "caching_allocator_alloc", self.alloc)
        monkeypatch.setattr(B.torch.cuda, "caching_allocator_delete", self.delete)

    def alloc(self, size, device=None, stream=None):
        assert stream == 7 and size > 0
        if size > self.most:
            raise B.torch.OutOfMemoryError("no room")
        free = self.next if not self.used else max(p + n for p, n in self.used.items())
        self.used[free] = size
        return free

    def delete(self, ptr):
        del self.used[ptr]


def packed(l):
    return bytes(desc(l))


NORM = bytes(B.NrmDesc(4096, 4096, 4096, 1, 0))


def test_calls_of_two_threads_have_workspaces_of_their_own(monkeypatch):
    """A call is several launches: another thread's on the same stream may come between them."""
    allocator, met, seen = Allocator(monkeypatch), threading.Barrier(2, timeout=20), []

    def fn(d, *args):
        met.wait()                       # both calls are under way
        seen.append((args[-3], args[-3] + args[-2], args[-1]))
        met.wait()
        return B.ANR_OK

    for calls in ([(B.ANR_OP_CONV2D, packed(LAYERS[0]), B.ConvDesc)] * 2, [(B.ANR_OP_NRM, NORM, B.NrmDesc)] * 2,
                  [(B.ANR_OP_CONV2D, packed(LAYERS[2]), B.ConvDesc), (B.ANR_OP_NRM, NORM, B.NrmDesc)]):
        seen.clear()
        threads = [threading.Thread(target=B._with_workspace, args=(fn, "fn", op, d, (1, 2, 3), None, t)) for op, d, t in calls]
        [t.start() for t in threads]
        [t.join() for t in threads]
        (a, a_end, s), (b, b_end, t) = seen
        assert s == t == 7 and (a_end <= b or b_end <= a)
        assert not allocator.used


@pytest.mark.parametrize("op, d, t, need", [(B.ANR_OP_CONV2D, packed(LAYERS[0]), B.ConvDesc, B.conv2d_fast_workspace_size(desc(LAYERS[0]))),
                                            (B.ANR_OP_CONV2D, packed((1, 512, 7, 7, 512, 3, 3, (1, 1), (1, 1), (1, 1), 1)), B.ConvDesc, None),
                                            (B.ANR_OP_CONV2D, packed((2, 16, 8, 8, 16, 3, 3, (1, 1), (1, 1), (1, 1), 1)), B.ConvDesc, 0),
                                            (B.ANR_OP_NRM, NORM, B.NrmDesc, 4096), (B.ANR_OP_NRM, bytes(B.NrmDesc(8, 8, 8, 1, 0)), B.NrmDesc, 0),
                                            (B.ANR_OP_NRM, bytes(B.NrmDesc(0, 8, 8, 1, 0)), B.NrmDesc, 0)])
def test_a_call_is_given_what_it_needs_and_gives_it_back(monkeypatch, op, d, t, need):
    allocator = Allocator(monkeypatch)
    if need is None:
        need = B.workspace_size(op, B.ConvDesc.from_buffer_copy(d))
        assert need > 0

    def fn(_, x, ws, size, stream):
        assert (x, size, stream) == (1, need, 7) and (ws is None) == (need == 0)
        assert list(allocator.used.items()) == ([(ws, need)] if need else [])
        return status
    for status in (B.ANR_OK, B.ANR_ERR_LAUNCH):
        if status == B.ANR_OK:
            B._with_workspace(fn, "fn", op, d, (1,), None, t)
        else:
            with pytest.raises(B.AnrError, match="fn"):
                B._with_workspace(fn, "fn", op, d, (1,), None, t)
        assert not allocator.used


def test_a_captured_call_keeps_its_workspace_from_others(monkeypatch):
    """From the graph's pool it goes back there; without one it is never handed out again, as the graph's replays use it."""
    allocator, seen = Allocator(monkeypatch), []

    def fn(_, x, ws, size, stream):
        seen.append((ws, ws + size))
        return B.ANR_OK

    def call(l):
        B._with_workspace(fn, "fn", B.ANR_OP_CONV2D, packed(l), (1,), None)
        return seen[-1]

    call(LAYERS[0])
    allocator.capture = (0, 3)
    call(LAYERS[0])
    assert not allocator.used
    allocator.capture = (0, 0)
    captured = [call(LAYERS[0]), call(LAYERS[1])]
    allocator.capture = None
    later = [call(LAYERS[0]), call(LAYERS[3])]
    spans = sorted(captured) + [max(later)]
    assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:])) and min(later)[0] >= spans[1][1]
    assert sorted(allocator.used.items()) == [(a, b - a) for a, b in sorted(captured)]


@pytest.mark.parametrize("layer", LAYERS)
def test_without_room_for_the_pieces_a_layer_runs_without_them(monkeypatch, layer):
    allocator, sizes = Allocator(monkeypatch), []

    def fn(_, x, ws, size, stream):
        assert (ws is None) == (size == 0)
        sizes.append(size)
        return B.ANR_OK

    least, fast = B.workspace_size(B.ANR_OP_CONV2D, desc(layer)), B.conv2d_fast_workspace_size(desc(layer))
    for allocator.most in (fast, fast - 1, least):
        B._with_workspace(fn, "fn", B.ANR_OP_CONV2D, packed(layer), (1,), None)
    assert sizes == [fast, least, least] and not allocator.used
    if least:
        allocator.most = least - 1
        with pytest.raises(B.torch.OutOfMemoryError):
            B._with_workspace(fn, "fn", B.ANR_OP_CONV2D, packed(layer), (1,), None)
