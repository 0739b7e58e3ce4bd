"""The operators' extension module against the Python functions it stands before: the same results for every way to pass the
arguments, views, streams and threads, and the same errors."""
import threading

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rand(*shape):
    return torch.rand(shape, device="cuda") - 0.5


def wide(*shape):
    """A view whose rows lie further apart than they are long."""
    return (torch.rand(shape[:-1] + (shape[-1] + 3,), device="cuda") - 0.5)[..., :shape[-1]]


def calls(anr):
    x, w, bn = rand(2, 16, 12, 12), rand(24, 16, 3, 3), [rand(24).abs() + 0.5 for _ in range(4)]
    desc, pack = anr.conv2d_pack_weights(x.shape, w, (1, 1), (1, 1), bn=bn, eps=1e-5)
    y = lambda: rand(2, 24, 12, 12)
    q, k = rand(2, 40, 3, 16), rand(2, 40, 3, 16)
    big = rand(4, 128, 20, 20), rand(64, 128, 3, 3)
    return {
        "gemm": [((rand(33, 40), rand(40, 50), rand(33, 50)), {}), ((wide(3, 33, 40), wide(3, 40, 50), wide(3, 33, 50)), {}),
                 ((rand(32, 128),), {"C": rand(32, 32), "B": rand(128, 32)})],
        "conv2d": [((x, w, y(), (1, 1), (1, 1)), {}), ((x, w, rand(2, 24, 5, 5)), {"stride": (2, 2)}), ((x, w, y()), {"pad": [1, 1]}),
                   ((x, w, rand(2, 24, 12, 12)), {"pad": (2, 2), "dil": (2, 2), "ws": None, "route": anr.ANR_CONV_ROUTE_GENERAL}),
                   ((wide(2, 16, 12, 12), w[:, :4].contiguous(), wide(2, 24, 12, 12), (1, 1), (1, 1)), {"groups": 4}),
                   ((*big, rand(4, 64, 20, 20), (1, 1), (1, 1)), {})],
        "conv_bn_relu": [((x, w, *bn, 1e-5, y(), (1, 1), (1, 1)), {}), ((x, w, *bn), {"eps": 1, "y": y(), "pad": (1, 1)})],
        "conv2d_packed": [((desc, x, pack, y()), {}), ((desc, wide(2, 16, 12, 12), pack, wide(2, 24, 12, 12)), {})],
        "conv_bn_relu_packed": [((desc, x, pack, y()), {"ws": None})],
        "dwconv": [((x, rand(16, 1, 3, 3), rand(2, 16, 12, 12), (1, 1), (1, 1)), {}), ((wide(2, 16, 12, 12), rand(16, 1, 5, 5), rand(2, 16, 6, 6)),
                                                                                         {"stride": (2, 2), "pad": (2, 2), "dil": (1, 1)})],
        "tbg": [((q, k, rand(2, 3, 40, 40)), {}), ((wide(2, 40, 3, 16), k, wide(2, 3, 40, 40)), {})],
        "tbs": [((q, k, rand(2, 3, 40, 40)), {}), ((q, k), {"out": rand(2, 3, 40, 40)})],
        "nrm": [((rand(70, 300), rand(1)), {}), ((wide(4, 200, 300), rand(4)), {"ws": None}), ((rand(4, 200, 300),), {"out": rand(4)})],
    }


def output(name, args, kwargs):
    names = {"gemm": ("C", 2), "conv2d": ("y", 2), "conv_bn_relu": ("y", 7), "conv2d_packed": ("y", 3), "conv_bn_relu_packed": ("y", 3), "dwconv": ("y", 2),
             "tbg": ("out", 2), "tbs": ("out", 2), "nrm": ("out", 1)}
    key, at = names[name]
    return kwargs[key] if key in kwargs else args[at]


@pytest.mark.parametrize("name", ["gemm", "conv2d", "conv_bn_relu", "conv2d_packed", "conv_bn_relu_packed", "dwconv", "tbg", "tbs", "nrm"])
def test_same_results(name):
    from paper_2006_06762_amd import binding as anr
    for args, kwargs in calls(anr)[name]:
        out = output(name, args, kwargs)
        assert getattr(anr, "_" + name)(*args, **kwargs) is out
        want = out.clone()
        for on in (torch.cuda.current_stream(), torch.cuda.Stream()):
            out.fill_(float("nan"))
            on.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(on):
                assert getattr(anr, name)(*args, **kwargs) is out
            torch.cuda.synchronize()
            assert torch.equal(out, want)
        with torch.no_grad():
            args = tuple(torch.nn.Parameter(a) if isinstance(a, torch.Tensor) and a.dtype is torch.float32 and a is not out else a for a in args)
        getattr(anr, name)(*args, **kwargs)
        assert torch.equal(out, want)


def test_same_errors():
    from paper_2006_06762_amd import binding as anr
    a, x, w, y = rand(32, 32), rand(1, 8, 8, 8), rand(8, 8, 3, 3), rand(1, 8, 8, 8)
    for name, args, kwargs in [("gemm", (a, a), {}), ("gemm", (a, a, a, a), {}), ("gemm", (a, a, a.cpu()), {}), ("gemm", (a, a, a.double()), {}),
                               ("gemm", (a.t(), a, a), {}), ("gemm", (a, a, a), {"D": a}), ("gemm", (a, a, a), {"A": a}), ("gemm", (a[:0], a, a), {}),
                               ("gemm", (1, 2, 3), {}), ("gemm", (a[0], a, a), {}),
                               ("conv2d", (x, w, y, (0, 1)), {}), ("conv2d", (x, w, y, 1), {}),
                               ("conv2d", (x, w.permute(0, 1, 3, 2), y), {}), ("conv2d", (x, w, y), {"route": 3}), ("conv2d", (x, w, y), {"groups": 3}),
                               ("conv2d", (x, w[0], y), {}), ("conv2d", (x, w, y), {"pad": (1, 1), "ws": a.cpu(), "stride": (-1, 1)}),
                               ("conv_bn_relu", (x, w, a[0], a[0], a[0], a[0], 1e-5, y), {}), ("conv_bn_relu", (x, w, y), {}),
                               ("conv2d_packed", (a, x, y, y), {}), ("conv2d_packed", (None, x, y, y), {}),
                               ("dwconv", (x, rand(8, 1, 3, 3), y.half()), {}),
                               ("tbg", (x, 3, y), {}), ("tbs", (x, x), {}), ("nrm", (a.t(), rand(1)), {}), ("nrm", (a, rand(2)), {}), ("nrm", (a, 3), {})]:
        raised = []
        for prefix in ("", "_"):
            with pytest.raises(Exception) as e:
                getattr(anr, prefix + name)(*args, **kwargs)
            raised.append((type(e.value), str(e.value)))
        assert raised[0] == raised[1], (name, raised)


def test_wrapped_tensors_go_to_python():
    """Tensors of transforms and modes, and subclasses, are no plain memory."""
    from paper_2006_06762_amd import binding as anr

    class Sub(torch.Tensor):
        pass

    a, c = rand(32, 32), rand(32, 32)
    want = anr._gemm(a, a, c).clone()
    assert torch.equal(anr.gemm(a.as_subclass(Sub), a, c.zero_()), want)
    with pytest.raises(Exception):
        torch.vmap(lambda t: anr.gemm(t, a, c))(rand(2, 32, 32))
    seen = []

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    with Mode():
        anr.gemm(a, a, c)
    assert torch.Tensor.data_ptr in seen


def test_threads_with_streams_of_their_own():
    from paper_2006_06762_amd import binding as anr
    x, w = rand(1, 256, 14, 14), rand(256, 256, 3, 3)
    want = anr.conv2d(x, w, rand(1, 256, 14, 14), (1, 1), (1, 1)).clone()
    wrong = []

    def work():
        stream, y = torch.cuda.Stream(), rand(1, 256, 14, 14)
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            for _ in range(20):
                anr.conv2d(x, w, y, (1, 1), (1, 1))
                anr.gemm(x[0, 0], x[0, 1], rand(14, 14))
        stream.synchronize()
        if not torch.equal(y, want):
            wrong.append(1)

    threads = [threading.Thread(target=work) for _ in range(6)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not wrong
