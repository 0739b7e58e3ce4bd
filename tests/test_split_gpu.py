"""The GEMM and convolution kernels that multiply fp32 operands as three bf16 pieces each.

Values the pieces cannot carry (infinities, NaN, magnitudes that round to infinity in bf16 or lie below
2^-110) must come out as the fp32 instruction gives them; everything else within the bound of an fp32
sum.  The bound: K + 2 roundings of 2^-24 relative to the sum of the absolute products (an fp32 sum in any
order makes K - 1, a product one; the split's small products and what it leaves out add less than one), plus half the
smallest denormal per term.  Tighter bounds for few terms and for sums of one sign stand beside their tests.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def anr():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2006_06762_amd import binding
    return binding


def uniform(seed, *shape):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return torch.empty(shape, device="cuda").uniform_(-1.0, 1.0, generator=gen)


def assert_product(C, A, B):
    ref, size, K = A.double() @ B.double(), A.double().abs() @ B.double().abs(), A.shape[-1]
    finite = ref.abs() <= torch.finfo(torch.float32).max
    got = C.double()
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    inf = ~finite & ~torch.isnan(ref)
    assert torch.equal(got[inf], torch.sign(ref[inf]) * float("inf"))
    off = (got - ref).abs()[finite]
    bound = ((K + 2) * 2.0 ** -24 * size + K * 2.0 ** -149)[finite]
    assert bool((off <= bound).all()), float((off / bound).max())


# K below, at and past the 16- and 32-wide steps, single columns and rows past a tile, odd leading dimensions (what
# each variant of tile and wave groups does at its edges: VARIANTS below)
SHAPES = [(1, 4097, 4095, 129), (1, 2305, 1791, 161), (16, 513, 511, 333), (3, 1009, 1531, 71), (1, 300, 301, 303),
          (1, 33, 47, 1000), (1, 65, 1, 513), (1, 1, 130, 95), (2, 64, 66, 511), (5, 129, 127, 145), (1, 700, 700, 480)]


@pytest.mark.parametrize("batch,M,N,K", SHAPES)
def test_split_gemm_edges(anr, batch, M, N, K):
    A, B = uniform(M, batch, M, K), uniform(N, batch, K, N)
    buf = torch.full((batch * M * N + 128,), 7.0, device="cuda")
    C = buf[64:-64].view(batch, M, N)
    anr.gemm(A, B, C)
    assert_product(C, A, B)
    assert bool((buf[:64] == 7.0).all()) and bool((buf[-64:] == 7.0).all())


# the first two are products of few 32 x 32 tiles (gemm_rows32_kernel), the others the split GEMM's
UNALIGNED = [(300, 260, 333), (700, 700, 545), (2100, 1900, 200), (1100, 1000, 333), (547, 1037, 1025)]


@pytest.mark.parametrize("M,N,K", UNALIGNED)
def test_split_gemm_strided_unaligned_views(anr, M, N, K):
    A = uniform(1, M, K + 5)[:, 3:K + 3]
    B = uniform(2, K, N + 7)[:, 1:N + 1]
    C = torch.full((M, N + 3), 7.0, device="cuda")
    anr.gemm(A, B, C[:, 1:N + 1])
    assert_product(C[:, 1:N + 1], A, B)
    assert bool((C[:, 0] == 7.0).all()) and bool((C[:, N + 1:] == 7.0).all())


# a packed column is a row of the A.B^T form, a strided one is not; K below a chunk, around the plain kernel's range
@pytest.mark.parametrize("M,K", [(65, 1), (130, 31), (65, 100), (700, 160), (40000, 24), (300, 161), (70, 513)])
@pytest.mark.parametrize("batch", [1, 3])
@pytest.mark.parametrize("ldb,ldc", [(1, 1), (3, 1), (1, 4)])
def test_gemm_of_a_single_column(anr, batch, M, K, ldb, ldc):
    A, B = uniform(50, batch, M, K), uniform(51, batch, K, ldb)[:, :, :1]
    C = torch.full((batch, M, ldc), 7.0, device="cuda")
    anr.gemm(A, B, C[:, :, :1])
    assert_product(C[:, :, :1], A, B.contiguous())
    assert bool((C[:, :, 1:] == 7.0).all())


@pytest.mark.parametrize("M,N,K", UNALIGNED)
@pytest.mark.parametrize("what", ["inf", "nan", "huge", "overflow", "denormal", "tiny", "past_k"])
def test_split_gemm_values_the_pieces_cannot_carry(anr, M, N, K, what):
    A, B = uniform(3, M, K), uniform(4, K, N)
    if what == "inf":
        A[M // 2, K - 1] = float("inf")
        B[0, N // 3] = -float("inf")
        B[K - 1, N - 1] = 0.0                       # inf * 0
    elif what == "nan":
        A[M - 1, 0] = float("nan")
    elif what == "huge":                            # finite, but its first piece rounds to infinity
        A[M // 3, K // 2] = 3.4e38
        B[K // 2] = 0.25
    elif what == "overflow":
        A[1] = 1e20
        B[:, 2] = 1e20
    elif what == "denormal":
        A *= 2.0 ** -130
    elif what == "tiny":
        A *= 2.0 ** -118
        B *= 2.0 ** 100
    elif what == "past_k":                          # what lies behind a row's end must not be multiplied
        whole = torch.full((M, K + 8), float("inf"), device="cuda")
        whole[:, :K] = A
        A = whole[:, :K]
    C = torch.empty(M, N, device="cuda")
    anr.gemm(A, B, C)
    assert_product(C, A, B)


@pytest.mark.parametrize("B,S,H,D", [(2, 130, 3, 64), (1, 257, 2, 80), (4, 512, 12, 33), (1, 300, 1, 128), (16, 256, 8, 128),
                                     (8, 200, 16, 80), (8, 192, 16, 32)])
def test_split_scores(anr, B, S, H, D):
    q, k = uniform(5, B, S, H, D), uniform(6, B, S, H, D)
    out = torch.empty(B, H, S, S, device="cuda")
    anr.tbg(q, k, out)
    qt, kt = q.permute(0, 2, 1, 3).contiguous(), k.permute(0, 2, 3, 1).contiguous()
    assert_product(out, qt, kt)
    q[0, S - 1, 0, D - 1] = float("inf")
    anr.tbg(q, k, out)
    assert_product(out, q.permute(0, 2, 1, 3).contiguous(), kt)


# one shape per variant of the split GEMM (tile, wave groups), each with remainders in M, N and K
VARIANTS = {(128, 1): (1, 3971, 4033, 545), (128, 2): (8, 505, 900, 515), (64, 1): (8, 257, 900, 161), (64, 2): (12, 505, 511, 1509),
            (64, 4): (1, 545, 943, 963)}

# Units of 2^-24 of a product: what the products add beside the roundings of the large sum.  The seven small ones
# make at most 2^-7 of a product, rounded seven times; ll, which is left out, at most 2^-10 of a unit.
SMALL = 7 * 2.0 ** -7 + 2.0 ** -10


def few_terms(seed, terms, batch, M, K):
    """A with `terms` non-zeros of 1 to 2 and either sign in every row."""
    A = uniform(seed, batch, M, K)
    A = torch.where(A < 0, A * 0.5 - 1.0, A * 0.5 + 1.0)
    A.scatter_(2, uniform(seed + 1, batch, M, K).argsort(2)[:, :, terms:], 0.0)
    return A


# the same of the A.B^T form, as (B, S, H, D) of scores that no other kernel takes (D is no multiple of four)
SCORES = {(128, 1): (4, 512, 12, 33), (128, 2): (2, 397, 8, 515), (64, 1): (4, 292, 8, 65), (64, 2): (2, 300, 8, 257),
          (64, 4): (1, 300, 8, 257)}


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("what", ["plain", "inf", "huge", "tiny", "denormal"])
def test_split_gemm_variants(anr, variant, what):
    batch, M, N, K = VARIANTS[variant]
    A, B = uniform(43, batch, M, K), uniform(44, batch, K, N)
    if what == "inf":                               # in the last row, column and k of a matrix
        A[batch // 2, M - 1, K - 1] = float("inf")
        B[0, K - 1, N - 1] = float("nan")
    elif what == "huge":
        A[batch - 1, M // 3, K // 2] = 3.4e38
        B[:, K // 2] = 0.25
    elif what == "tiny":                            # in the first chunk of some tiles, in the last of others
        A[:, ::301, 0] *= 2.0 ** -112
        A[:, 150::301, K - 1] *= 2.0 ** -130
    elif what == "denormal":
        A *= 2.0 ** -130
    buf = torch.full((batch * M * N + 128,), 7.0, device="cuda")
    C = buf[64:-64].view(batch, M, N)
    anr.gemm(A, B, C)
    assert_product(C, A, B)
    assert bool((buf[:64] == 7.0).all()) and bool((buf[-64:] == 7.0).all())


# A last chunk that is no whole one starts at K - 32 and passes over what was counted: values there are multiplied once,
# with their own partners alone, whichever operand and order of infinities
@pytest.mark.parametrize("batch,M,N,K", [*VARIANTS.values(), (1, 1100, 1000, 333), (1, 2000, 1900, 200), (2, 1040, 1050, 63)])
def test_split_gemm_infinities_in_the_last_chunks_overlap(anr, batch, M, N, K):
    A, B = uniform(51, batch, M, K), uniform(52, batch, K, N)
    B[0, K // 32 * 32 - 1, N - 1] = float("inf")
    B[batch - 1, K - 32, 0] = -float("inf")
    A[batch - 1, M // 2, max(K // 32 * 32 - 9, K - 32)] = float("inf")
    C = torch.empty(batch, M, N, device="cuda")
    anr.gemm(A, B, C)
    assert_product(C, A, B)


# ... and scores that the dispatch takes from the tile kernels: heads of 256 and more in whole chunks, parts of one
# (K below the 32 of a chunk) and a ragged last tile
@pytest.mark.parametrize("B,S,H,D", [*SCORES.values(), (16, 256, 8, 32), (16, 256, 8, 24), (16, 256, 8, 128), (16, 360, 8, 96)])
def test_split_scores_variants(anr, B, S, H, D):
    q, k = uniform(45, B, S, H, D), uniform(46, B, S, H, D)
    out, soft = torch.empty(2, B, H, S, S, device="cuda")
    for tiny in (False, True):
        if tiny:
            q[:, ::5, :, D - 1] *= 2.0 ** -115
        anr.tbg(q, k, out)
        assert_product(out, q.permute(0, 2, 1, 3).contiguous(), k.permute(0, 2, 3, 1).contiguous())
        # softmax over the same scores: an exponential and a division of a few units, at most 16 additions in a lane
        # and 6 between lanes, and the exponent, the distance from the row's maximum, rounded as it is subtracted and
        # as it is scaled to a power of two
        anr.tbs(q, k, soft)
        want, below = torch.softmax(out.double(), -1), out.amax(-1, keepdim=True).double() - out.double()
        assert bool(((soft.double() - want).abs() <= (32 + 2 * below) * 2.0 ** -24 * want + 2.0 ** -148).all())


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("terms", [1, 4])
def test_split_gemm_of_few_terms_is_rounded_once_per_term(anr, variant, terms):
    batch, M, N, K = VARIANTS[variant]
    A, B = few_terms(20, terms, batch, M, K), uniform(22, batch, K, N)
    B[:, :, : N // 2] = 1.0 + 2.0 ** -8 - 2.0 ** -17          # both small pieces as large as they get
    C = torch.empty(batch, M, N, device="cuda")
    anr.gemm(A, B, C)
    units = (C.double() - A.double() @ B.double()).abs() / (A.double().abs() @ B.double().abs()) * 2.0 ** 24
    # the first term's large product is exact; every further one and the small products' sum are a rounding each
    assert float(units.max()) <= terms + SMALL, float(units.max())


@pytest.mark.parametrize("variant", VARIANTS)
def test_split_gemm_of_one_sign_is_rounded_once_per_sixteen_terms(anr, variant):
    batch, M, N, K = VARIANTS[variant]
    A, B = uniform(24, batch, M, K).abs(), uniform(25, batch, K, N).abs()
    C = torch.empty(batch, M, N, device="cuda")
    anr.gemm(A, B, C)
    ref = A.double() @ B.double()
    rms = float(((C.double() - ref) / ref * 2.0 ** 24).square().mean().sqrt())
    # n roundings of a sum that grows evenly, each evenly spread over at most a unit of it: sqrt(n / 9); the last
    # chunk repeats up to half of its steps with zeros, which round nothing.  The fp32 instruction has 8 n.
    n = -(-K // 16) + 1
    assert rms <= 1.1 * (n / 9.0) ** 0.5 + SMALL, (rms, n)


@pytest.mark.parametrize("variant", VARIANTS)
def test_split_gemm_results_near_the_smallest_normal(anr, variant):
    batch, M, N, K = VARIANTS[variant]
    A, B = few_terms(27, 1, batch, M, K), uniform(29, batch, K, N)
    A *= 2.0 ** -64
    B = torch.where(B < 0, B * 0.5 - 1.0, B * 0.5 + 1.0) * 2.0 ** -60       # products of 2^-124 to 2^-122
    C = torch.empty(batch, M, N, device="cuda")
    anr.gemm(A, B, C)
    ref = A.double() @ B.double()
    units = (C.double() - ref).abs() / ref.abs() * 2.0 ** 24
    assert float(units.max()) <= 1.0 + SMALL, float(units.max())


@pytest.mark.parametrize("variant", VARIANTS)
def test_split_gemm_single_rows_near_the_smallest_normal(anr, variant):
    """The same where only some rows of a tile are that small: rows of every accumulator register."""
    batch, M, N, K = VARIANTS[variant]
    B = uniform(29, batch, K, N)
    B = torch.where(B < 0, B * 0.5 - 1.0, B * 0.5 + 1.0) * 2.0 ** -60
    C = torch.empty(batch, M, N, device="cuda")
    for first in (1, 6, 11, 16):
        A = few_terms(27, 1, batch, M, K)
        A[:, first::29] *= 2.0 ** -64
        anr.gemm(A, B, C)
        ref = A.double() @ B.double()
        units = ((C.double() - ref).abs() / ref.abs() * 2.0 ** 24)[:, first::29]
        assert float(units.max()) <= 1.0 + SMALL, float(units.max())


def conv_reference(x, w, stride, pad, dil=1, groups=1):
    """Convolution and the convolution of the absolute values, in 64 bits, tap by tap."""
    N, C, H, W = x.shape
    K, Cg, R, S = w.shape
    OH, OW = (H + 2 * pad - dil * (R - 1) - 1) // stride + 1, (W + 2 * pad - dil * (S - 1) - 1) // stride + 1
    out = []
    for f in (lambda t: t, torch.abs):
        xp = f(torch.nn.functional.pad(x.double(), (pad,) * 4))
        wd = f(w.double()).view(groups, K // groups, Cg, R, S)
        y = torch.zeros(N, groups, K // groups, OH * OW, dtype=torch.float64, device=x.device)
        for r in range(R):
            for s in range(S):
                tap = xp[:, :, r * dil:r * dil + stride * (OH - 1) + 1:stride, s * dil:s * dil + stride * (OW - 1) + 1:stride]
                y += wd[:, :, :, r, s].contiguous() @ tap.reshape(N, groups, Cg, OH * OW)
        out.append(y.view(N, K, OH, OW))
    return out[0], out[1], Cg * R * S


def assert_conv(y, x, w, stride, pad, dil=1, groups=1):
    ref, size, terms = conv_reference(x, w, stride, pad, dil, groups)
    got = y.double()
    finite = ref.abs() <= torch.finfo(torch.float32).max
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    inf = ~finite & ~torch.isnan(ref)
    assert torch.equal(got[inf], torch.sign(ref[inf]) * float("inf"))
    off = (got - ref).abs()[finite]
    bound = ((terms + 2) * 2.0 ** -24 * size + terms * 2.0 ** -149)[finite]
    assert bool((off <= bound).all()), float((off / bound).max())


# (N, C, H, W, K, R, stride, pad): two and three channels, ragged tiles, channels past a tile of 64, no padding
STEMS = [(64, 3, 64, 64, 64, 7, 2, 3), (11, 2, 129, 95, 100, 7, 2, 3), (4, 2, 131, 133, 64, 7, 1, 3), (4, 3, 130, 129, 49, 7, 1, 2),
         (3, 3, 225, 222, 190, 7, 2, 0), (33, 3, 40, 63, 64, 7, 1, 6)]
# the first four have too few tiles for the stem kernel; the same with more images, and two rounds with a ragged last one
STEMS += [(96, 3, 64, 64, 64, 7, 2, 3), (13, 2, 129, 95, 100, 7, 2, 3), (5, 2, 131, 133, 64, 7, 1, 3), (6, 3, 130, 129, 49, 7, 1, 2),
          (16, 3, 200, 224, 64, 7, 2, 3)]


@pytest.mark.parametrize("N,C,H,W,K,R,stride,pad", STEMS)
@pytest.mark.parametrize("what", ["plain", "inf", "tiny", "huge_weight"])
def test_stem_convolution(anr, N, C, H, W, K, R, stride, pad, what):
    x, w = uniform(7, N, C, H, W), uniform(8, K, C, R, R)
    if what == "inf":
        x[N - 1, C - 1, H // 2, W - 1] = float("inf")
        x[0, 0, 0, 0] = float("nan")
    elif what == "tiny":
        x[N // 2] *= 2.0 ** -125
    elif what == "huge_weight":
        w[K - 1, 0, R - 1, 0] = 3.4e38
        x *= 0.5
    r = anr.conv2d_route(anr.conv_desc(x.shape, K, R, R, (stride, stride), (pad, pad)))
    few = (N, C, H, W) in [c[:4] for c in STEMS[:4]]
    assert (r.kernel, r.tile_m == 256, r.ksplit) == (anr.ANR_CONV_KERNEL_BIGTAPS, not few, 1)
    OH, OW = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    buf = torch.full((N * K * OH * OW + 128,), 7.0, device="cuda")
    y = buf[64:-64].view(N, K, OH, OW)
    anr.conv2d(x, w, y, (stride, stride), (pad, pad))
    assert_conv(y, x, w, stride, pad)
    assert bool((buf[:64] == 7.0).all()) and bool((buf[-64:] == 7.0).all())


def test_stem_conv_bn_relu_on_strided_views(anr):
    N, C, H, W, K = 10, 3, 100, 110, 100
    x = uniform(9, N, C, H + 2, W + 5)[:, :, 1:H + 1, 2:W + 2]
    w, gamma, beta, mean = uniform(10, K, C, 7, 7), uniform(11, K), uniform(12, K), uniform(13, K)
    var = uniform(14, K) + 1.5
    OH, OW = (H - 1) // 2 + 1, (W - 1) // 2 + 1
    y = torch.empty(N, K, OH, OW + 3, device="cuda")[..., 1:OW + 1]
    anr.conv_bn_relu(x, w, gamma, beta, mean, var, 1e-5, y, (2, 2), (3, 3))
    ref, size, terms = conv_reference(x, w, 2, 3)
    c = lambda v: v.double().view(1, K, 1, 1)
    scale = c(gamma) / torch.sqrt(c(var) + 1e-5)
    want = torch.relu((ref - c(mean)) * scale + c(beta))
    # the sum's bound scaled, and a handful of roundings of the batch norm's own terms
    bound = (terms + 2) * 2.0 ** -24 * size * scale.abs() + 8 * 2.0 ** -24 * (ref.abs() * scale.abs() + (c(mean) * scale).abs() + c(beta).abs())
    assert bool(((y.double() - want).abs() <= bound).all())


# (N, C, H, W, K, pad): tiles of 64 and of 32 channels, patches of up to 512 and up to 1024 pixels, tiles that straddle
# images, channels past the last tile, a single chunk of sixteen channels
PATCHES = [(16, 64, 56, 56, 64, 1), (16, 16, 56, 56, 50, 1), (16, 48, 28, 28, 100, 1), (5, 32, 112, 112, 96, 1), (9, 32, 56, 60, 64, 0),
           (8, 16, 28, 56, 256, 2)]


def patch_case(anr, N, C, H, W, K, pad):
    x, w = uniform(15, N, C, H, W), uniform(16, K, C, 3, 3)
    r = anr.conv2d_route(anr.conv_desc(x.shape, K, 3, 3, (1, 1), (pad, pad), route=anr.ANR_CONV_ROUTE_PATCH))
    assert r.kernel == anr.ANR_CONV_KERNEL_PATCH and r.tile_m == 224, (r.kernel, r.tile_m)
    return x, w, torch.full((N, K, H + 2 * pad - 2, W + 2 * pad - 2), 7.0, device="cuda")


@pytest.mark.parametrize("N,C,H,W,K,pad", PATCHES)
@pytest.mark.parametrize("what", ["plain", "inf", "tiny", "huge_weight"])
def test_patch_convolution(anr, N, C, H, W, K, pad, what):
    x, w, y = patch_case(anr, N, C, H, W, K, pad)
    if what == "inf":
        x[N - 1, C - 1, H // 2, W - 1] = float("inf")
        x[0, 0, 0, 0] = float("nan")
    elif what == "tiny":
        x[N // 2] *= 2.0 ** -125
    elif what == "huge_weight":
        w[K - 1, 0, 2, 0] = 3.4e38
        x *= 0.5
    anr.conv2d(x, w, y, (1, 1), (pad, pad), route=anr.ANR_CONV_ROUTE_PATCH)
    assert_conv(y, x, w, 1, pad)
    desc, pack = anr.conv2d_pack_weights(x.shape, w, (1, 1), (pad, pad), route=anr.ANR_CONV_ROUTE_PATCH)
    z = torch.empty_like(y)
    anr.conv2d_packed(desc, x, pack, z)
    assert torch.equal(y.nan_to_num(1.5), z.nan_to_num(1.5))


@pytest.mark.parametrize("N,C,H,W,K,pad", PATCHES)
@pytest.mark.parametrize("terms", [1, 4])
def test_patch_convolution_of_few_terms_is_rounded_once_per_term(anr, N, C, H, W, K, pad, terms):
    x, _, y = patch_case(anr, N, C, H, W, K, pad)
    x[: N // 2] = 1.0 + 2.0 ** -8 - 2.0 ** -17          # both small pieces as large as they get
    w = few_terms(30, terms, 1, K, C * 9).view(K, C, 3, 3)
    w[: K // 2] *= (1.0 + 2.0 ** -8 - 2.0 ** -17) / w[: K // 2].abs().clamp_min(1.0)
    anr.conv2d(x, w, y, (1, 1), (pad, pad), route=anr.ANR_CONV_ROUTE_PATCH)
    ref, size, _ = conv_reference(x, w, 1, pad)
    units = ((y.double() - ref).abs() / size.clamp_min(1e-300) * 2.0 ** 24)[size > 0]
    assert float(units.max()) <= terms + SMALL, float(units.max())


@pytest.mark.parametrize("N,C,H,W,K,pad", PATCHES)
def test_patch_convolution_of_one_sign_is_rounded_nine_times_per_chunk(anr, N, C, H, W, K, pad):
    x, w, y = patch_case(anr, N, C, H, W, K, pad)
    sums = 3 if anr.conv2d_route(anr.conv_desc(x.shape, K, 3, 3, (1, 1), (pad, pad), route=anr.ANR_CONV_ROUTE_PATCH)).tile_n == 32 else 1
    x, w = x.abs(), w.abs()
    anr.conv2d(x, w, y, (1, 1), (pad, pad), route=anr.ANR_CONV_ROUTE_PATCH)
    ref = conv_reference(x, w, 1, pad)[0]
    units = ((y.double() - ref) / ref.clamp_min(1e-300) * 2.0 ** 24)[ref > 0]
    # n roundings of `sums` sums that grow evenly to that share of the result, each evenly spread over at most a unit
    # of its sum, and the additions of the sums
    n = 9 * C // 16
    ends = (sum((i + 1) ** 2 for i in range(sums)) / sums ** 2 / 3.0) ** 0.5
    assert float(units.square().mean().sqrt()) <= 1.1 * (n / 9.0) ** 0.5 / sums + ends + SMALL


@pytest.mark.parametrize("N,C,H,W,K,R,stride,pad", STEMS)
def test_stem_convolution_is_rounded_no_more_than_its_large_sum(anr, N, C, H, W, K, R, stride, pad):
    x, y = uniform(33, N, C, H, W), torch.empty(N, K, (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1, device="cuda")
    x[: N // 2] = 1.0 + 2.0 ** -8 - 2.0 ** -17          # both small pieces as large as they get
    for terms in (1, 4):
        w = few_terms(34, terms, 1, K, C * R * R).view(K, C, R, R)
        w[: K // 2] *= (1.0 + 2.0 ** -8 - 2.0 ** -17) / w[: K // 2].abs().clamp_min(1.0)
        anr.conv2d(x, w, y, (stride, stride), (pad, pad))
        ref, size, _ = conv_reference(x, w, stride, pad)
        units = ((y.double() - ref).abs() / size.clamp_min(1e-300) * 2.0 ** 24)[size > 0]
        assert float(units.max()) <= terms + SMALL, (terms, float(units.max()))
    x, w = uniform(35, N, C, H, W).abs(), uniform(36, K, C, R, R).abs()
    anr.conv2d(x, w, y, (stride, stride), (pad, pad))
    ref = conv_reference(x, w, stride, pad)[0]
    units = ((y.double() - ref) / ref.clamp_min(1e-300) * 2.0 ** 24)[ref > 0]
    # four roundings a channel of a sum that grows evenly, and the small products' sum (the fp32 instruction, which
    # runs the first four: 25 a channel)
    steps = 25 if (N, C, H, W) in [c[:4] for c in STEMS[:4]] else 4
    assert float(units.square().mean().sqrt()) <= 1.1 * (steps * C / 9.0) ** 0.5 + 3.0 ** -0.5 + SMALL


def microseconds(call):
    call()
    best = float("inf")
    for _ in range(5):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(4):
            call()
        end.record()
        end.synchronize()
        best = min(best, start.elapsed_time(end) * 250.0)
    return best


# Values the pieces cannot carry are redone with the fp32 instruction, at half the rate of the eight products; where
# the whole first try is lost as well the two take three times an ordinary call.
@pytest.mark.parametrize("batch,M,N,K", [(1, 2048, 2048, 2048), (16, 512, 512, 512), (1, 1024, 1024, 1024)])
def test_split_gemm_of_values_the_pieces_cannot_carry_takes_no_multiple(anr, batch, M, N, K):
    A, B, C = uniform(40, batch, M, K), uniform(41, batch, K, N), torch.empty(batch, M, N, device="cuda")
    usual = microseconds(lambda: anr.gemm(A, B, C))
    A[:, ::32, K - 1] = float("inf")
    assert microseconds(lambda: anr.gemm(A, B, C)) <= 3.0 * usual
    A = torch.softmax(200.0 * uniform(42, batch, M, K), -1)
    assert microseconds(lambda: anr.gemm(A, B, C)) <= 2.0 * usual


@pytest.mark.parametrize("C,H,K", [(64, 56, 64), (256, 28, 256)])
def test_patch_convolution_of_values_the_pieces_cannot_carry_takes_no_multiple(anr, C, H, K):
    x, w, y = patch_case(anr, 16, C, H, H, K, 1)
    call = lambda: anr.conv2d(x, w, y, (1, 1), (1, 1), route=anr.ANR_CONV_ROUTE_PATCH)
    usual = microseconds(call)
    x[:, 0, ::2] *= 2.0 ** -120
    assert microseconds(call) <= 3.0 * usual
    x.uniform_(-1.0, 1.0)
    w[::8] *= 2.0 ** -120
    assert microseconds(call) <= 3.0 * usual


def test_patch_convolution_results_near_the_smallest_normal(anr):
    x, _, y = patch_case(anr, 16, 64, 56, 56, 64, 1)
    x = torch.where(x < 0, x * 0.5 - 1.0, x * 0.5 + 1.0) * 2.0 ** -60
    w = few_terms(37, 1, 1, 64, 64 * 9).view(64, 64, 3, 3) * 2.0 ** -64
    anr.conv2d(x, w, y, (1, 1), (1, 1), route=anr.ANR_CONV_ROUTE_PATCH)
    ref = conv_reference(x, w, 1, 1)[0]
    units = ((y.double() - ref).abs() / ref.abs() * 2.0 ** 24)[ref != 0]
    assert float(units.max()) <= 1.0 + SMALL, float(units.max())


def test_stem_convolution_of_values_the_pieces_cannot_carry_takes_no_multiple(anr):
    x, w, y = uniform(47, 16, 3, 224, 224), uniform(48, 64, 3, 7, 7), torch.empty(16, 64, 112, 112, device="cuda")
    call = lambda: anr.conv2d(x, w, y, (2, 2), (3, 3))
    usual = microseconds(call)
    x[:, 0, ::8, ::8] *= 2.0 ** -120
    assert microseconds(call) <= 3.0 * usual
    x.uniform_(-1.0, 1.0)
    w[::8] *= 2.0 ** -120
    assert microseconds(call) <= 3.0 * usual
