"""Calls that need more and less workspace than the one before on their stream, and a caller's that is too small."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_kept_workspace_grows_with_the_calls_of_a_stream():
    from paper_2006_06762_amd import binding as anr
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    stream = torch.cuda.Stream()
    for C, H in ((64, 7), (256, 14), (512, 7), (64, 7)):
        x = torch.randn(1, C, H, H, device="cuda", generator=gen)
        w = torch.randn(C, C, 3, 3, device="cuda", generator=gen)
        need = anr.workspace_size(anr.ANR_OP_CONV2D, anr.conv_desc(x.shape, C, 3, 3, (1, 1), (1, 1)))
        assert need > 0
        own = torch.empty(need, dtype=torch.uint8, device="cuda")
        y, ref = torch.empty(2, 1, C, H, H, device="cuda")
        anr.conv2d(x, w, ref, (1, 1), (1, 1), ws=own)
        with pytest.raises(ValueError):
            anr.conv2d(x, w, ref, (1, 1), (1, 1), ws=own[:-4])
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            anr.conv2d(x, w, y, (1, 1), (1, 1))
        torch.cuda.synchronize()
        assert torch.equal(y, ref)


def test_arguments_that_are_no_float32_cuda_tensors_are_refused():
    from paper_2006_06762_amd import binding as anr
    a = torch.zeros(32, 32, device="cuda")
    for bad in (a.cpu(), a.double()):
        with pytest.raises(TypeError):
            anr.gemm(bad, a, a.clone())
        with pytest.raises(TypeError):
            anr.nrm(bad, torch.zeros(1, device="cuda"))
    with pytest.raises(ValueError):
        anr.gemm(a.t(), a, a.clone())
    with pytest.raises(anr.AnrError):
        anr.conv2d(a.view(1, 1, 32, 32), a.view(32, 32, 1, 1)[:1, :1], a.view(1, 1, 32, 32), groups=-1)
