"""1 x 1 layers that run as a batched GEMM of weights and images: odd planes and even ones, channel counts past a tile and
a chunk, views, batch norm, packed weights, values the pieces cannot carry."""
import numpy as np
import pytest

import oracle
from paper_2006_06762_amd import inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GUARD = 12345.0
# (N, C, H, W, K)
SHAPES = [(7, 48, 31, 27, 100), (16, 64, 29, 29, 64), (3, 100, 57, 41, 130), (16, 256, 25, 25, 384), (1, 33, 101, 109, 70), (5, 96, 96, 70, 200),
          (16, 200, 37, 27, 500)]


def tensors(shape, seed, ints, start, gap):
    """gap: floats between the channels of x and of y."""
    N, C, H, W, K = shape
    s = I.ConvShape(N, C, H, W, K, 1, 1, (1, 1), (0, 0))
    x, w = I.conv_inputs(s, seed, ints=ints)
    def view(c, fill):
        buf = torch.full((start + N * c * (H * W + gap) + 64,), fill, device="cuda")
        return buf, buf[start:].as_strided((N, c, H, W), (c * (H * W + gap), H * W + gap, W, 1))
    xbuf, xv = view(C, float("nan"))
    xv.copy_(torch.from_numpy(x))
    ybuf, y = view(K, GUARD)
    return s, x, w, xv, torch.from_numpy(w).cuda(), ybuf, y


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("start,gap", [(0, 0), (1, 0), (2, 5)])
def test_whole_numbers(shape, start, gap):
    from paper_2006_06762_amd import binding as anr
    s, x, w, xv, wd, ybuf, y = tensors(shape, 6000 + shape[1], True, start, gap)
    r = anr.conv2d_route(anr.conv_desc(x.shape, s.K, 1, 1))
    assert r.kernel == anr.ANR_CONV_KERNEL_POINTWISE and r.workspace_bytes == 0 and r.ksplit == 1
    anr.conv2d(xv, wd, y)
    ref = torch.einsum("kc,nchw->nkhw", wd[:, :, 0, 0].double(), torch.from_numpy(x).cuda().double())
    assert torch.equal(y.double(), ref)
    assert np.array_equal(y[:1].cpu().numpy().astype(np.float64), oracle.conv2d(x[:1], w, (1, 1), (0, 0)))
    left = int((ybuf == GUARD).sum())
    assert left == ybuf.numel() - y.numel()


@pytest.mark.parametrize("shape", SHAPES)
def test_fused_and_packed(shape):
    from paper_2006_06762_amd import binding as anr
    s, x, w, xv, wd, ybuf, y = tensors(shape, 6100, False, 0, 0)
    bn = [torch.from_numpy(v).cuda() for v in I.bn_inputs(s.K, 6101)]
    anr.conv_bn_relu(xv, wd, *bn, I.BN_EPS, y)
    sums = torch.einsum("kc,nchw->nkhw", wd[:, :, 0, 0].double(), xv.double())
    g, b, m, v = (t.double().view(1, -1, 1, 1) for t in bn)
    want = torch.relu((sums - m) * g / (v + I.BN_EPS).sqrt() + b)
    assert float(((y.double() - want).abs() / want.abs().clamp(min=1.0)).max()) <= 1e-5
    desc, pack = anr.conv2d_pack_weights(x.shape, wd, bn=bn, eps=I.BN_EPS)
    y2 = torch.empty_like(y)
    anr.conv_bn_relu_packed(desc, xv, pack, y2)
    assert torch.equal(y, y2)
    anr.conv2d_packed(desc, xv, pack, y2)
    anr.conv2d(xv, wd, y)
    assert torch.equal(y, y2)
    size = torch.einsum("kc,nchw->nkhw", wd[:, :, 0, 0].double().abs(), xv.double().abs())
    assert bool(((y.double() - sums).abs() <= (s.C + 2) * 2.0 ** -24 * size).all())


@pytest.mark.parametrize("value", [float("inf"), float("nan"), 2.0 ** -120, 3.4e38])
def test_values_the_pieces_cannot_carry(value):
    from paper_2006_06762_amd import binding as anr
    s, x, w, xv, wd, ybuf, y = tensors(SHAPES[2], 6200, True, 0, 0)
    bn = [torch.from_numpy(v).cuda() for v in I.bn_inputs(s.K, 6201)]
    xv[1, 3, 40, 35] = value
    xv[2, 99, 56, 40] = value
    anr.conv2d(xv, wd, y)
    want = torch.nn.functional.conv2d(xv.cpu(), wd.cpu())
    got = y.cpu()
    assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf())
    exact = torch.nn.functional.conv2d(xv.cpu().double(), wd.cpu().double())
    ok = want.isfinite()
    assert bool(((got.double() - exact).abs()[ok] <= 1e-6 * exact.abs().clamp(min=1.0)[ok]).all())
    y2 = torch.empty_like(y)
    anr.conv_bn_relu(xv, wd, *bn, I.BN_EPS, y2)          # the fused epilogue behind the second try
    scale = bn[0] / (bn[3] + I.BN_EPS).sqrt()
    fused = torch.relu(y * scale.view(1, -1, 1, 1) + (bn[1] - bn[2] * scale).view(1, -1, 1, 1))
    ok = ok.cuda() & fused.isfinite()                    # (a scale above one takes 3.4e38 past the largest float)
    assert torch.equal(y2.isinf(), fused.isinf())
    assert bool(((y2 - fused).abs()[ok] <= 1e-4 * fused.abs().clamp(min=1.0)[ok]).all())


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[1] % 32])
@pytest.mark.parametrize("value", [float("inf"), -float("inf")])
def test_an_infinite_pixel_in_channels_that_two_chunks_load(shape, value):
    """C is no multiple of 32, so the last chunk starts at C - 32: an infinite pixel there is multiplied by its own
    weights alone, and the fused form keeps what survives the ReLU."""
    from paper_2006_06762_amd import binding as anr
    s, x, w, xv, wd, ybuf, y = tensors(shape, 6300, False, 0, 0)
    xv[s.N - 1, s.C // 32 * 32 - 1, 7, 5] = value
    anr.conv2d(xv, wd, y)
    at = y[s.N - 1, :, 7, 5]
    want = torch.sign(wd[:, s.C // 32 * 32 - 1, 0, 0]) * value
    assert torch.equal(at, want) and int((~y.isfinite()).sum()) == s.K
    bn = [torch.from_numpy(v).cuda() for v in I.bn_inputs(s.K, 6301)]
    anr.conv_bn_relu(xv, wd, *bn, I.BN_EPS, y)
    assert torch.equal(y[s.N - 1, :, 7, 5], torch.relu(want * bn[0])) and int((~y.isfinite()).sum()) == int((want * bn[0] > 0).sum())
