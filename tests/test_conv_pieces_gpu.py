"""Convolutions on pieces made once per call: every tile and group count, split reductions, channels and output channels that
are no whole units, an odd number of units, groups, strides, dilations, rows and columns that differ in all of these, odd planes,
views, operands and workspaces that start anywhere, packs of both orders, values the
pieces cannot carry, and what a call does with less workspace."""
import numpy as np
import pytest

import oracle
from paper_2006_06762_amd import inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (N, C, H, W, K, R, stride, dil, groups)
SHAPES = [
    (8, 512, 27, 12, 80, 7, 2, 2, 4),       # 32 channels, one group of waves, split
    (16, 32, 81, 81, 32, 5, 1, 1, 1),       # 32 channels, one group
    (3, 32, 40, 40, 128, 7, 1, 1, 4),       # 32 channels, four groups
    (4, 100, 31, 31, 80, 7, 1, 1, 4),       # the same, split; 25 channels a group, 20 output channels
    (8, 50, 24, 48, 160, 3, 1, 1, 2),       # 64 channels, one group
    (4, 128, 26, 26, 64, 7, 1, 1, 1),       # the same, split
    (8, 16, 35, 35, 33, 7, 1, 1, 1),        # 64 channels, two groups, one output channel past the tile's half
    (4, 32, 34, 34, 33, 7, 1, 1, 1),        # the same, split
    (16, 256, 14, 14, 256, 3, 1, 1, 1),     # the third stage of a residual network
    (3, 40, 61, 61, 96, 5, 1, 1, 1),        # an odd number of units
    (32, 512, 7, 7, 160, 3, 1, 1, 1),       # tiles across images of 49 pixels
    (7, 192, 73, 73, 32, 3, 1, 1, 1),       # a layer of the 224-pixel tile for any width
    (4, 16, 108, 108, 512, 3, 1, 1, 1),     # packed in the order of a patch kernel, 64 output channels at a time
    (2, 64, 160, 160, 320, 3, 1, 1, 1),     # the same, 32 at a time
]


def layer(shape, seed, ints=False):
    N, C, H, W, K, R, stride, dil, groups = shape
    s = I.ConvShape(N, C, H, W, K, R, R, (stride, stride), (R // 2 * dil, R // 2 * dil), (dil, dil), groups)
    x, w = I.conv_inputs(s, seed, ints=ints)
    return s, x, w, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()


def exact(s, x, w):
    """The layer in 64 bits, and the sums of the products' magnitudes, on the GPU (tap by tap: plain batched products)."""
    def taps(x, w):
        G, Cg, Kg = s.groups, s.C // s.groups, s.K // s.groups
        xp = torch.nn.functional.pad(x, (s.pad[1], s.pad[1], s.pad[0], s.pad[0]))
        y = torch.zeros(s.N, G, Kg, s.OH * s.OW, device="cuda", dtype=torch.float64)
        for r in range(s.R):
            for t in range(s.S):
                part = xp[:, :, r * s.dil[0]:r * s.dil[0] + s.stride[0] * (s.OH - 1) + 1:s.stride[0],
                          t * s.dil[1]:t * s.dil[1] + s.stride[1] * (s.OW - 1) + 1:s.stride[1]]
                y += w[:, :, r, t].reshape(G, Kg, Cg) @ part.reshape(s.N, G, Cg, -1).contiguous()
        return y.reshape(s.N, s.K, s.OH, s.OW)
    x, w = x.double(), w.double()
    return taps(x, w), taps(x.abs(), w.abs())


def sizes(anr, s):
    d = anr.conv_desc((s.N, s.C, s.H, s.W), s.K, s.R, s.S, s.stride, s.pad, dil=s.dil, groups=s.groups)
    return anr.workspace_size(anr.ANR_OP_CONV2D, d), anr.conv2d_fast_workspace_size(d)


@pytest.mark.parametrize("shape", SHAPES)
def test_whole_numbers_and_workspace_limits(shape):
    from paper_2006_06762_amd import binding as anr
    s, x, w, xd, wd = layer(shape, 7000, ints=True)
    least, fast = sizes(anr, s)
    assert fast != least and 0 < fast <= 256e6
    ref = exact(s, xd, wd)[0]
    assert np.array_equal(ref[:1].cpu().numpy(), oracle.conv2d_general(x[:1], w, s.stride, s.pad, s.dil, s.groups))
    ws = torch.full((max(fast, least) + 256,), 0xff, dtype=torch.uint8, device="cuda")
    for size in (fast, fast - 16, least):               # less than fast: another kernel, if it is enough for that
        if size < min(least, fast):
            continue
        y = torch.full(ref.shape, float("nan"), device="cuda")
        anr.conv2d(xd, wd, y, s.stride, s.pad, ws=ws[:size], dil=s.dil, groups=s.groups)
        assert torch.equal(y.double(), ref), size
        assert bool((ws[size:] == 0xff).all())
        ws.fill_(0xff)


@pytest.mark.parametrize("shape", SHAPES)
def test_close_to_the_exact_sums(shape):
    """Sums of n products: one rounding per sixteen, and of the small pieces' sums, at the sum of the magnitudes; the fused
    form; packs of either order; an x that is no whole 16-byte units and a strided y."""
    from paper_2006_06762_amd import binding as anr
    s, x, w, xd, wd = layer(shape, 7100)
    ref, magnitudes = exact(s, xd, wd)
    y = torch.full(ref.shape, float("nan"), device="cuda")
    run = dict(dil=s.dil, groups=s.groups)
    anr.conv2d(xd, wd, y, s.stride, s.pad, **run)
    steps = s.C // s.groups * s.R * s.S / 16
    worst = float(((y - ref).abs() / magnitudes).max())
    assert worst <= (2 + steps ** .5) * 2.0 ** -24
    desc, pack = anr.conv2d_pack_weights(x.shape, wd, s.stride, s.pad, **run)
    z = torch.empty_like(y)
    anr.conv2d_packed(desc, xd, pack, z)
    assert torch.equal(z, y)
    bn = [torch.from_numpy(v).cuda() for v in I.bn_inputs(s.K, 7101)]
    desc, pack = anr.conv2d_pack_weights(x.shape, wd, s.stride, s.pad, bn=bn, eps=I.BN_EPS, **run)
    anr.conv_bn_relu(xd, wd, *bn, I.BN_EPS, y, s.stride, s.pad, **run)
    anr.conv_bn_relu_packed(desc, xd, pack, z)
    assert torch.equal(z, y)
    gamma, beta, mean, var = (v.double().view(1, -1, 1, 1) for v in bn)
    want = torch.relu(gamma * (ref - mean) / torch.sqrt(var + I.BN_EPS) + beta)
    worst = float((y - want).abs().max())
    assert worst <= 1e-4 * max(1.0, float(want.abs().max()))
    # views: rows of x one float longer, y inside a larger tensor
    wide = torch.full((s.N, s.C, s.H, s.W + 1), float("nan"), device="cuda")
    wide[..., 1:] = xd
    out = torch.full((s.N, s.K, s.OH + 1, s.OW + 3), 12345.0, device="cuda")
    view = out[:, :, :s.OH, 1:1 + s.OW]
    anr.conv2d(wide[..., 1:], wd, view, s.stride, s.pad, **run)
    # (where such rows leave the layer to a kernel on the fp32 instruction: one rounding per two products)
    d = anr.conv_desc(x.shape, s.K, s.R, s.S, s.stride, s.pad, wide[..., 1:].stride(), view.stride(), **run)
    pieces = anr.conv2d_fast_workspace_size(d) != anr.workspace_size(anr.ANR_OP_CONV2D, d)
    worst = float(((view - ref).abs() / magnitudes).max())
    assert worst <= (2 + (steps if pieces else 8 * steps) ** .5) * 2.0 ** -24
    view.fill_(12345.0)
    assert bool((out == 12345.0).all())


@pytest.mark.parametrize("shape", [SHAPES[i] for i in (0, 2, 3, 4, 7, 8, 9, 12)])
def test_values_the_pieces_cannot_carry(shape):
    """Infinities, NaN and floats below 2^-110 in x and w: the tiles they reach are those of the fp32 instruction, the others
    as without them."""
    from paper_2006_06762_amd import binding as anr
    s, x, w, xd, wd = layer(shape, 7200)
    run = dict(dil=s.dil, groups=s.groups)
    xd[0, 1, 3, 4], xd[1, 0, 5, 5], xd[0, 2, 6, 1] = float("inf"), float("nan"), 2.0 ** -120 * (1 + 2.0 ** -20)
    y, z = torch.empty((2, s.N, s.K, s.OH, s.OW), device="cuda")
    anr.conv2d(xd, wd, y, s.stride, s.pad, **run)
    anr.conv2d(xd, wd, z, s.stride, s.pad, ws=torch.empty(sizes(anr, s)[0], dtype=torch.uint8, device="cuda"), **run)
    assert torch.equal(y.isnan(), z.isnan()) and torch.equal(y.isinf(), z.isinf())
    keep = z.isfinite()
    worst = float((y - z)[keep].abs().max())
    assert worst <= 1e-4 * float(z[keep].abs().max())
    assert torch.equal(y[~keep].nan_to_num(1.5), z[~keep].nan_to_num(1.5))
    desc, pack = anr.conv2d_pack_weights(x.shape, wd, s.stride, s.pad, **run)
    anr.conv2d_packed(desc, xd, pack, z)
    assert torch.equal(z.nan_to_num(1.5), y.nan_to_num(1.5))
    # one product left in every sum, of a size whose last piece is lost: one rounding of the exact product
    xd.zero_()
    wd.zero_()
    per = s.C // s.groups
    xd[:, ::per] = torch.rand_like(xd[:, ::per]) * 2.0 ** -100
    wd[:, 0, s.R // 2, s.S // 2] = torch.rand(s.K, device="cuda") * 2.0 ** -14
    anr.conv2d(xd, wd, y, s.stride, s.pad, **run)
    ref = exact(s, xd, wd)[0]
    worst = float((y - ref).abs().max())
    assert worst <= 1.01 * 2.0 ** -24 * float(ref.abs().max())
    wd.mul_(2.0 ** -104)                                # weights whose pieces are lost, sums of ordinary size
    xd.mul_(2.0 ** 104)
    desc, pack = anr.conv2d_pack_weights(x.shape, wd, s.stride, s.pad, **run)
    anr.conv2d(xd, wd, y, s.stride, s.pad, **run)
    anr.conv2d_packed(desc, xd, pack, z)
    assert torch.equal(z, y)
    ref = exact(s, xd, wd)[0]
    worst = float((y - ref).abs().max())
    assert worst <= 1.01 * 2.0 ** -24 * float(ref.abs().max())


def test_replays_of_a_captured_call():
    from paper_2006_06762_amd import binding as anr
    s, x, w, xd, wd = layer(SHAPES[7], 7300)                # (one group, no dilation)
    y, ref = torch.empty((2, s.N, s.K, s.OH, s.OW), device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        anr.conv2d(xd, wd, y, s.stride, s.pad)          # the stream's workspace
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        anr.conv2d(xd, wd, y, s.stride, s.pad)
    for i in range(4):
        xd.copy_(torch.from_numpy(x).cuda() * (i + 1))
        y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        anr.conv2d(xd, wd, ref, s.stride, s.pad)
        assert torch.equal(y, ref)


# (N, C, H, W, K, R, S, stride, pad, dil, groups): rows and columns of the kernel, the steps, the padding and the dilation that differ
OBLONG = [
    (8, 64, 40, 50, 96, 3, 5, (1, 2), (1, 2), (1, 1), 1),
    (8, 64, 37, 45, 96, 5, 3, (2, 1), (0, 1), (1, 2), 1),
    (8, 96, 30, 61, 64, 1, 9, (1, 1), (0, 4), (1, 1), 1),
    (8, 96, 61, 30, 64, 9, 1, (1, 1), (4, 0), (1, 1), 1),
    (8, 100, 33, 70, 80, 7, 4, (1, 3), (6, 1), (2, 1), 4),
    (6, 40, 29, 83, 72, 2, 7, (1, 1), (2, 0), (1, 3), 2),
    (4, 48, 57, 31, 40, 4, 12, (1, 1), (3, 11), (1, 1), 1),
]


def oblong(shape, seed, ints):
    N, C, H, W, K, R, S, stride, pad, dil, groups = shape
    s = I.ConvShape(N, C, H, W, K, R, S, stride, pad, dil, groups)
    x, w = I.conv_inputs(s, seed, ints=ints)
    return s, x, w


def exact_oblong(s, x, w):
    """As exact(), for any geometry."""
    G, Cg, Kg = s.groups, s.C // s.groups, s.K // s.groups
    xp = torch.nn.functional.pad(x.double(), (s.pad[1], s.pad[1], s.pad[0], s.pad[0]))
    y = torch.zeros(2, s.N, G, Kg, s.OH * s.OW, device="cuda", dtype=torch.float64)
    for r in range(s.R):
        for t in range(s.S):
            part = xp[:, :, r * s.dil[0]:r * s.dil[0] + s.stride[0] * (s.OH - 1) + 1:s.stride[0],
                      t * s.dil[1]:t * s.dil[1] + s.stride[1] * (s.OW - 1) + 1:s.stride[1]].reshape(s.N, G, Cg, -1).contiguous()
            wt = w.double()[:, :, r, t].reshape(G, Kg, Cg)
            y[0] += wt @ part
            y[1] += wt.abs() @ part.abs()
    return y.reshape(2, s.N, s.K, s.OH, s.OW)


@pytest.mark.parametrize("shape", OBLONG)
def test_rows_and_columns_that_differ(shape):
    """Whole numbers exactly, others to one rounding per sixteen products; weights and an x that are no whole 16-byte units,
    images further apart than they are long, and the fused form of a pack."""
    from paper_2006_06762_amd import binding as anr
    for ints in (True, False):
        s, x, w = oblong(shape, 7400, ints)
        assert sizes(anr, s)[0] < sizes(anr, s)[1]
        run = dict(dil=s.dil, groups=s.groups)
        xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
        ref, magnitudes = exact_oblong(s, xd, wd)
        y = torch.full(ref.shape, float("nan"), device="cuda")
        anr.conv2d(xd, wd, y, s.stride, s.pad, **run)
        if ints:
            assert torch.equal(y.double(), ref)
            assert np.array_equal(ref[:1].cpu().numpy(), oracle.conv2d_general(x[:1], w, s.stride, s.pad, s.dil, s.groups))
            continue
        worst = float(((y - ref).abs() / magnitudes.clamp(min=1e-30)).max())
        assert worst <= (2 + (s.C // s.groups * s.R * s.S / 16) ** .5) * 2.0 ** -24
        # the same bits from operands that start anywhere
        wu = torch.empty(w.size + 1, device="cuda")[1:].view(w.shape).copy_(wd)
        xu = torch.full((x.size + s.N * 5 + 3,), float("nan"), device="cuda")[3:].view(s.N, -1)[:, :x[0].size].view(x.shape).copy_(xd)
        assert xu.stride(0) == x[0].size + 5 and xu.data_ptr() % 16 and wu.data_ptr() % 16
        out = torch.full((s.N, s.K + 1, s.OH, s.OW), 12345.0, device="cuda")
        anr.conv2d(xu, wu, out[:, :s.K], s.stride, s.pad, **run)
        assert torch.equal(out[:, :s.K], y) and bool((out[:, s.K] == 12345.0).all())
        bn = [torch.from_numpy(v).cuda() for v in I.bn_inputs(s.K, 7401)]
        desc, pack = anr.conv2d_pack_weights(x.shape, wd, s.stride, s.pad, bn=bn, eps=I.BN_EPS, **run)
        z = torch.empty_like(y)
        anr.conv_bn_relu(xd, wd, *bn, I.BN_EPS, y, s.stride, s.pad, **run)
        anr.conv_bn_relu_packed(desc, xd, pack, z)
        assert torch.equal(z, y)
        gamma, beta, mean, var = (v.double().view(1, -1, 1, 1) for v in bn)
        want = torch.relu(gamma * (ref - mean) / torch.sqrt(var + I.BN_EPS) + beta)
        assert float((y - want).abs().max()) <= 1e-4 * max(1.0, float(want.abs().max()))


@pytest.mark.parametrize("shape", [OBLONG[0], OBLONG[5]])
def test_a_workspace_that_is_not_aligned(shape):
    """The pieces are left out where nothing else needs a workspace; a split reduction refuses it as ever."""
    from paper_2006_06762_amd import binding as anr
    s, x, w = oblong(shape, 7500, True)
    run = dict(dil=s.dil, groups=s.groups)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    least, fast = sizes(anr, s)
    ws = torch.full((fast + 64,), 0xff, dtype=torch.uint8, device="cuda")
    y = torch.full((s.N, s.K, s.OH, s.OW), float("nan"), device="cuda")
    for start in (4, 8):
        if least:
            with pytest.raises(anr.AnrError):
                anr.conv2d(xd, wd, y, s.stride, s.pad, ws=ws[start:], **run)
            assert bool(y.isnan().all())
        else:
            anr.conv2d(xd, wd, y, s.stride, s.pad, ws=ws[start:], **run)
            assert torch.equal(y.double(), exact_oblong(s, xd, wd)[0])
        assert bool((ws == 0xff).all())
