"""NRM on both sides of the size from which the matrices are read non-temporally, with slices that leave remainders."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,N,M", [(1, 2896, 2896), (1, 2900, 2900), (3, 1931, 1604), (5, 2051, 1028), (1, 8388612, 1)])
def test_nrm_around_the_non_temporal_size(batch, N, M):
    from paper_2006_06762_amd import binding as anr
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N)
    x = torch.empty(batch, N, M, device="cuda").uniform_(-1.0, 1.0, generator=gen)
    out = torch.empty(batch, device="cuda")
    anr.nrm(x, out)
    want = x.double().square().sum((1, 2)).sqrt()
    # per thread at most N*M / (parts * 1024) + 12 terms are added one after another, then trees: 2^-24 each, halved by the root
    steps = N * M / 1024 / min(2048 // batch, N * M / 16384) + 40
    assert bool(((out.double() - want).abs() <= steps * 2.0 ** -24 * want).all())
    # whole numbers whose squares add up exactly
    x = torch.randint(-1, 2, (batch, N, M), device="cuda", generator=gen).float()
    x[:, N // 2:] = 0
    anr.nrm(x, out)
    assert torch.equal(out, x.double().square().sum((1, 2)).float().sqrt())


@pytest.mark.parametrize("start", [0, 1, 2, 3])
@pytest.mark.parametrize("batch,N,M,ld", [(3, 1, 1, 1), (4, 1, 3, 3), (2, 1, 5, 5), (5, 3, 3, 3), (3, 127, 129, 129), (2, 131, 251, 251),
                                          (3, 601, 83, 83), (2, 300, 1, 7), (2, 40, 255, 256), (2, 70, 256, 300), (2, 130, 257, 261),
                                          (1, 20, 1500, 1501)])
def test_nrm_any_alignment(batch, N, M, ld, start):
    """Matrices that begin 0 to 3 floats past an aligned address, rows back to back and apart: whole numbers, exactly, with
    values around the matrices that would show."""
    from paper_2006_06762_amd import binding as anr
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + M + start)
    stride = N * ld + 1
    buf = torch.full((batch * stride + 16,), float("nan"), device="cuda")
    x = buf[start:].as_strided((batch, N, M), (stride, ld, 1))
    x.copy_(torch.randint(-2, 3, (batch, N, M), device="cuda", generator=gen).float())
    out = torch.empty(batch, device="cuda")
    anr.nrm(x, out)
    assert torch.equal(out, x.double().square().sum((1, 2)).float().sqrt())
