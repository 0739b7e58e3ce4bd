"""Calls without a workspace of the caller's: several threads on one stream, each with operands of its own; more streams than
a thread keeps buffers for, and threads that end; graphs, whose
replays go on while the stream that they were captured on does other work and while each other's run."""
import ctypes
import threading

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def conv(anr, seed, N, C, H, K, R, packed=False):
    """(call, output) of a layer with operands of the seed's."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.empty((N, C, H, H), device="cuda").uniform_(-1, 1, generator=gen)
    w = torch.empty((K, C, R, R), device="cuda").uniform_(-1, 1, generator=gen)
    y, pad = torch.empty((N, K, H, H), device="cuda"), (R // 2, R // 2)
    if packed:
        desc, pack = anr.conv2d_pack_weights(x.shape, w, (1, 1), pad)
        return lambda: anr.conv2d_packed(desc, x, pack, y), y
    return lambda ws=None: anr.conv2d(x, w, y, (1, 1), pad, ws=ws), y


def norm(anr, seed):
    x = torch.full((700, 900), float(1 + seed), device="cuda")
    out = torch.empty(1, device="cuda")
    return lambda: anr.nrm(x, out), out


# pieces in one slice and in several, a split reduction on the fp32 instruction, partial sums of a norm; two larger than the last
CALLS = {"pieces": lambda anr, s: conv(anr, s, 16, 256, 14, 256, 3), "pieces packed": lambda anr, s: conv(anr, s, 16, 256, 14, 256, 3, True),
         "pieces split": lambda anr, s: conv(anr, s, 4, 128, 26, 64, 7), "split": lambda anr, s: conv(anr, s, 1, 512, 7, 512, 3), "norm": norm}


@pytest.mark.parametrize("own", [False, True])
def test_threads_on_one_stream(own):
    """The default stream, which all threads share, or one made for them."""
    from paper_2006_06762_amd import binding as anr
    stream = torch.cuda.Stream() if own else torch.cuda.default_stream()
    jobs = [[(c, y, (c(), y.clone())[1]) for c, y in (make(anr, 10 * i + j) for j, make in enumerate(CALLS.values()))] for i in range(4)]
    torch.cuda.synchronize()
    start, wrong = threading.Barrier(len(jobs), timeout=30), []

    def work(mine):
        with torch.cuda.stream(stream):
            start.wait()
            for _ in range(30):
                for call, y, _ in mine:
                    y.fill_(float("nan"))
                for call, y, _ in mine:
                    call()
                wrong.extend(1 for _, y, want in mine if not torch.equal(y, want))

    threads = [threading.Thread(target=work, args=(j,)) for j in jobs]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not wrong


class Captured:
    """A call captured by torch, its output and what that is to be."""

    def __init__(self, call, y, stream):
        torch.cuda.synchronize()         # (the operands are the default stream's work)
        with torch.cuda.stream(stream):
            call()                       # (what a kernel's first launch sets up)
        stream.synchronize()
        self.call, self.y, self.want, self.graph = call, y, y.clone(), torch.cuda.CUDAGraph()      # (the call holds its operands)
        with torch.cuda.graph(self.graph, stream=stream):
            call()
        torch.cuda.synchronize()

    def right(self):
        return torch.equal(self.y, self.want)


@pytest.mark.parametrize("name", list(CALLS))
def test_a_graph_has_memory_of_its_own(name):
    """A larger layer and tensors of every size afterwards on the stream of the capture: the replays write to none of them."""
    from paper_2006_06762_amd import binding as anr
    stream = torch.cuda.Stream()
    g = Captured(*CALLS[name](anr, 60), stream)
    larger, z = conv(anr, 61, 16, 128, 40, 96, 5)
    torch.cuda.synchronize()
    for i in range(3):
        with torch.cuda.stream(stream):
            larger()
            want = z.clone()
            others = [torch.full((n,), 7.0, device="cuda") for n in (1 << 10, 1 << 18, 1 << 20, 1 << 21, 1 << 22, 1 << 23, 1 << 24)]
            g.y.fill_(float("nan"))
            g.graph.replay()
            assert g.right() and all(bool((t == 7.0).all()) for t in others)
            larger()
            assert torch.equal(z, want)
            del others


@pytest.mark.parametrize("name", list(CALLS))
def test_graphs_captured_on_one_stream_run_at_once(name):
    from paper_2006_06762_amd import binding as anr
    stream = torch.cuda.Stream()
    graphs = [Captured(*CALLS[name](anr, 70 + i), stream) for i in range(3)]
    streams = [torch.cuda.Stream() for _ in graphs]
    for _ in range(5):
        for g in graphs:
            g.y.fill_(float("nan"))
        torch.cuda.synchronize()
        for _ in range(20):
            for g, s in zip(graphs, streams):
                with torch.cuda.stream(s):
                    g.graph.replay()
        torch.cuda.synchronize()
        assert all(g.right() for g in graphs)


def test_a_capture_that_is_not_torchs():
    """Replays write to memory that nothing else is given."""
    from paper_2006_06762_amd import binding as anr
    hip = ctypes.CDLL("libamdhip64.so.7")         # (the one that torch has loaded)
    stream = torch.cuda.Stream()
    call, y = CALLS["pieces split"](anr, 80)
    at, graph, program = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_void_p()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        call()
        want = y.clone()
        torch.cuda.synchronize()
        relaxed = 2
        assert hip.hipStreamBeginCapture(at, relaxed) == 0
        call()
        assert hip.hipStreamEndCapture(at, ctypes.byref(graph)) == 0
        assert hip.hipGraphInstantiate(ctypes.byref(program), graph, None, None, 0) == 0
        others = [torch.full((n,), 7.0, device="cuda") for n in (1 << 18, 1 << 20, 1 << 21, 1 << 22, 1 << 23)]
        for _ in range(3):
            y.fill_(float("nan"))
            assert hip.hipGraphLaunch(program, at) == 0
            assert torch.equal(y, want) and all(bool((t == 7.0).all()) for t in others)
        torch.cuda.synchronize()
        assert hip.hipGraphExecDestroy(program) == 0 and hip.hipGraphDestroy(graph) == 0


@pytest.mark.parametrize("N,C,H,K,R", [(16, 256, 56, 64, 5), (16, 64, 150, 96, 5)])
def test_a_layer_runs_where_there_is_no_room_for_its_pieces(N, C, H, K, R):
    """The process is allowed little more than it has: the kernel that needs no workspace, as with an empty one."""
    from paper_2006_06762_amd import binding as anr
    call, y = conv(anr, 90, N, C, H, K, R)
    d = anr.conv_desc((N, C, H, H), K, R, R, (1, 1), (R // 2, R // 2))
    assert anr.workspace_size(anr.ANR_OP_CONV2D, d) == 0 and anr.conv2d_fast_workspace_size(d) > 64 << 20
    call(torch.empty(0, dtype=torch.uint8, device="cuda"))
    want = y.clone()
    call()
    pieces = y.clone()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    try:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (8 << 20)) / total)
        y.fill_(float("nan"))
        call()
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(y, want) and not torch.equal(want, pieces)
    call()
    assert torch.equal(y, pieces)


def test_more_streams_than_a_thread_keeps_buffers_for():
    """Needs that grow and shrink on eleven streams in turn, every call's operands other than the last one's; then again in threads
    that end before their work is done."""
    from paper_2006_06762_amd import binding as anr
    streams = [torch.cuda.Stream() for _ in range(11)]
    gen = torch.Generator(device="cuda").manual_seed(100)
    jobs = []
    for batch, n in ((1, 150), (70, 300), (3, 2000), (1, 300), (300, 260), (16, 700)):
        for i in range(2):
            x = torch.empty((batch, n, n), device="cuda").uniform_(-1, 1, generator=gen)
            jobs.append((x, torch.empty(batch, device="cuda")))
    need = [anr.workspace_size(anr.ANR_OP_NRM, anr.NrmDesc(x.shape[1], x.shape[2], x.shape[2], x.shape[0], x.stride(0))) for x, _ in jobs]
    assert min(need) > 0
    layers = [CALLS["split"](anr, 101), conv(anr, 102, 1, 64, 14, 64, 3), CALLS["split"](anr, 103)]       # 4, 1, 4 MB
    want = [anr.nrm(*j).clone() for j in jobs] + [(c(), y.clone())[1] for c, y in layers]
    calls = [(lambda x=x, o=o: anr.nrm(x, o), o) for x, o in jobs] + layers
    torch.cuda.synchronize()

    def work(offset):
        for turn in range(4):
            for i, (call, out) in enumerate(calls):
                with torch.cuda.stream(streams[(i * 5 + turn * 3 + offset) % len(streams)]):
                    call()

    for offset in range(3):
        for _, out in calls:
            out.fill_(float("nan"))
        torch.cuda.synchronize()
        thread = threading.Thread(target=work, args=(offset,))
        work(offset) if offset == 0 else (thread.start(), thread.join())
        others = [torch.full((1 << s,), 7.0, device="cuda") for s in range(12, 22)]
        torch.cuda.synchronize()
        assert all(torch.equal(out, w) for (_, out), w in zip(calls, want))
        assert all(bool((t == 7.0).all()) for t in others)


def test_another_thread_goes_on_while_one_captures():
    from paper_2006_06762_amd import binding as anr
    stream = torch.cuda.Stream()
    inside = [CALLS[n](anr, 110 + i) for i, n in enumerate(("pieces split", "norm"))]
    beside = [CALLS[n](anr, 120 + i) for i, n in enumerate(CALLS)]
    want = []
    for call, y in inside + beside:
        call()
        want.append(y.clone())
        y.fill_(float("nan"))
    with torch.cuda.stream(stream):
        [call() for call, _ in inside]
    torch.cuda.synchronize()
    graph, failed = torch.cuda.CUDAGraph(), []

    def eager():
        try:
            [call() for _ in range(5) for call, _ in beside]
        except Exception as e:
            failed.append(e)

    with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
        inside[0][0]()
        thread = threading.Thread(target=eager)
        thread.start()
        thread.join()
        inside[1][0]()
    assert not failed
    for _ in range(3):
        for _, y in inside:
            y.fill_(float("nan"))
        graph.replay()
        beside[0][0]()
        torch.cuda.synchronize()
        assert all(torch.equal(y, w) for (_, y), w in zip(inside + beside, want))
