"""Depthwise layers that run in bands of rows: odd widths and heights around the eight outputs of a thread's walk,
both strides, both kernel sizes, any padding, several planes per work-group, views; small integers, so bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2006_06762_amd import inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GUARD = 12345.0


def run(s, seed, start=0, gap=0, values=()):
    """start: floats x and y begin past an aligned address; gap: floats between the rows of x and of y; values: (value, tap)
    for every third channel's weights."""
    from paper_2006_06762_amd import binding as anr
    x, w = I.dwconv_inputs(s, seed, ints=True)
    for value, tap in values:
        w[tap % 3::3].reshape(-1, s.R * s.R)[:, tap] = value
    xbuf = torch.full((s.N * s.C * s.H * (s.W + gap) + 8,), float("nan"), device="cuda")
    xv = xbuf[start:start + s.N * s.C * s.H * (s.W + gap)].view(s.N, s.C, s.H, s.W + gap)[..., :s.W]
    xv.copy_(torch.from_numpy(x))
    n = s.N * s.C * s.OH * (s.OW + gap)
    ybuf = torch.full((n + 128,), GUARD, device="cuda")
    wide = ybuf[64 + start:64 + start + n].view(s.N, s.C, s.OH, s.OW + gap)
    anr.dwconv(xv, torch.from_numpy(w).cuda(), wide[..., :s.OW], s.stride, s.pad)
    assert np.array_equal(wide[..., :s.OW].cpu().numpy().astype(np.float64), oracle.dwconv(x, w, s.stride, s.pad), equal_nan=True), s
    assert bool((wide[..., s.OW:] == GUARD).all()) and bool((ybuf[:64 + start] == GUARD).all())
    assert bool((ybuf[64 + start + n:] == GUARD).all())


@pytest.mark.parametrize("R", [3, 5])
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("H, W, planes", [(47, 61, 400), (64, 67, 400), (65, 50, 350), (150, 21, 330), (9, 259, 900), (57, 57, 1100)])
def test_bands(R, stride, H, W, planes):
    planes *= stride * stride
    run(I.ConvShape(2, planes // 2, H, W, planes // 2, R, R, (stride, stride), (R // 2, R // 2)), 3000 + H + R)


@pytest.mark.parametrize("R, stride, W, planes", [(3, 1, 1399, 20), (3, 1, 1431, 20), (3, 2, 830, 90), (5, 1, 1190, 10), (5, 2, 747, 40)])
def test_wide_rows(R, stride, W, planes):
    """Eight rows of outputs whose input rows take more than 48 KB of LDS, up to the 56 KB where the direct kernel takes over."""
    s = I.ConvShape(1, planes, 37, W, planes, R, R, (stride, stride), (R // 2, R // 2))
    lds = 4 * ((s.OW - 1) * stride + R) * (7 * stride + R)
    assert 48 * 1024 < lds <= 56 * 1024 and planes * s.OH * s.OW * R * R >= 4000000
    run(s, 3050 + W)


@pytest.mark.parametrize("H, W, R, stride, pad, start, gap", [(13, 13, 3, 1, 1, 1, 0), (14, 14, 5, 1, 2, 3, 0), (7, 9, 3, 1, 1, 2, 0),
                                                              (20, 20, 3, 1, 0, 0, 3), (30, 31, 3, 2, 3, 0, 1), (16, 12, 5, 2, 4, 1, 0)])
def test_planes_in_groups_views_and_padding(H, W, R, stride, pad, start, gap):
    """Planes that are unaligned or whose rows lie apart: several to a work-group, or one."""
    s = I.ConvShape(5, 3001 if H * W < 300 else 901, H, W, 3001 if H * W < 300 else 901, R, R, (stride, stride), (pad, pad))
    run(s, 3100 + H, start, gap)


@pytest.mark.parametrize("R", [3, 5])
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("H, W, planes, pad, start, gap", [(47, 61, 400, 1, 0, 0), (64, 67, 400, 2, 1, 3), (9, 259, 900, 0, 0, 0), (57, 57, 1100, 4, 0, 0),
                                                           (14, 14, 8000, 1, 1, 0)])
def test_weights_that_are_not_finite(R, stride, H, W, planes, pad, start, gap):
    """A tap outside the image is no product: an infinite weight leaves the outputs whose tap it is there as they are."""
    planes *= stride * stride
    s = I.ConvShape(2, planes // 2, H, W, planes // 2, R, R, (stride, stride), (pad, pad))
    run(s, 3200 + H, start, gap, [(float("inf"), 0), (float("nan"), R * R - 1), (-float("inf"), R // 2)])


@pytest.mark.parametrize("N, C, H, W, R, stride", [(2, 100, 7, 7, 3, 1), (3, 33, 14, 14, 5, 1), (2, 40, 13, 9, 3, 2), (1, 30, 7, 9, 7, 1)])
def test_small_planes_pass_over_taps_outside_too(N, C, H, W, R, stride):
    s = I.ConvShape(N, C, H, W, C, R, R, (stride, stride), (R // 2, R // 2))
    run(s, 3300 + H, 0, 0, [(float("inf"), 0), (float("nan"), R * R - 1), (-float("inf"), R // 2)])
