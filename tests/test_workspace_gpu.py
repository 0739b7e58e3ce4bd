"""Calls without a workspace of the caller's: several threads on one stream, each with operands of its own."""
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
    return lambda: anr.conv2d(x, w, y, (1, 1), pad), y


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
