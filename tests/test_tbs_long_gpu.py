"""The one-kernel TBS for 128 < S <= 512: edges of its key chunks (128) and query blocks (32), short and ragged
reductions, rows of every alignment, strided views, values that are not finite."""
import numpy as np
import pytest

import oracle
from paper_2006_06762_amd import inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GUARD = 12345.0
# probabilities: a score of standard deviation sqrt(D) s carries a few roundings of 2^-24 of its absolute sum, and the
# exponential turns an absolute error into a relative one; measured below 3e-6 of the row's largest for these
TOL = 2e-5


def check(got, ref, what):
    top = ref.max(-1, keepdims=True)
    err = float(np.max(np.abs(got.astype(np.float64) - ref) / top))
    assert err <= TOL, "%s: %.2e of the row's largest" % (what, err)


def heads_for(S, D):
    """As many heads as the one kernel asks for, and fewer than the split GEMM does."""
    chunks = (S + 127) // 128
    return 2 if D * chunks <= 64 else (36, 20, 14)[chunks - 2]


# (more than 512 floats of a row to walk, chunks times D, are left to two kernels)
EDGES = [(S, D, heads_for(S, D)) for S in (129, 160, 255, 256, 257, 384, 385, 389, 511, 512) for D in (8, 32, 40, 72, 128, 168, 256)
         if (S + 127) // 128 * D <= 512]
VIEW = (2, 192, 14, 64)
SMALL = [(160, 40), (256, 64), (300, 40), (511, 64), (512, 64)]
SMALL_HEADS = 24


@pytest.mark.parametrize("S,D,heads", EDGES)
def test_edges(S, D, heads):
    from paper_2006_06762_amd import binding as anr
    s = I.TbgShape(1, S, heads, D)
    q, k = I.tbg_inputs(s, 2000 + S + D)
    q = (q * (2.0 / D ** 0.5)).astype(np.float32)
    n = heads * S * S
    buf = torch.full((n + 128,), GUARD, device="cuda")
    out = buf[64:64 + n].view(1, heads, S, S)
    anr.tbs(torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda(), out)
    check(out.cpu().numpy(), oracle.tbs(q, k), "S %d D %d" % (S, D))
    assert bool((buf[:64] == GUARD).all()) and bool((buf[-64:] == GUARD).all())


@pytest.mark.parametrize("pad, start", [(0, 0), (32, 0), (4, 4), (3, 1)])
def test_views(pad, start):
    """q and k as slices of a projection that holds both, rows of the result further apart than they are long."""
    from paper_2006_06762_amd import binding as anr
    B, S, H, D = VIEW
    q, k = I.tbg_inputs(I.TbgShape(B, S, H, D), 2100)
    q = (q * 0.25).astype(np.float32)
    both = torch.zeros((B, S, 2, H, D), device="cuda")
    both[:, :, 0], both[:, :, 1] = torch.from_numpy(q), torch.from_numpy(k)
    buf = torch.full((B * H * S * (S + pad) + 8,), GUARD, device="cuda")
    wide = buf[start:start + B * H * S * (S + pad)].view(B, H, S, S + pad)
    anr.tbs(both[:, :, 0], both[:, :, 1], wide[..., :S])
    check(wide[..., :S].cpu().numpy(), oracle.tbs(q, k), "view %d %d" % (pad, start))
    assert bool((wide[..., S:] == GUARD).all())


def test_values_that_are_not_finite():
    """As a matrix product and torch's softmax give them: NaN and +inf spoil their query's row (a key's: every row),
    -inf gives probability zero."""
    from paper_2006_06762_amd import binding as anr
    S, D = 300, 16
    q = torch.ones((1, S, 1, D), device="cuda")
    k = torch.rand((1, S, 1, D), device="cuda", generator=torch.Generator(device="cuda").manual_seed(5))
    k[0, 290, 0, 3] = -float("inf")
    q[0, 7, 0, 2] = float("nan")
    q[0, 100, 0, 5] = 3e38
    q[0, 101, 0, :] = 0.0
    out = torch.empty((1, 1, S, S), device="cuda")
    anr.tbs(q, k, out)
    ref = torch.softmax((q[0, :, 0].cpu().double() @ k[0, :, 0].cpu().double().T).float(), -1)
    got = out[0, 0].cpu()
    assert torch.equal(got.isnan(), ref.isnan())
    ok = ~ref.isnan().any(-1)
    assert ok.sum() == S - 2 and bool((got[ok][:, 290] == 0).all())
    ok[100] = False                      # scores of 1e38: the largest alone survives
    assert float((got[ok] - ref[ok]).abs().max()) <= TOL
    assert got[100].argmax() == ref[100].argmax()


@pytest.mark.parametrize("S, D", SMALL)
def test_small_probabilities(S, D):
    """Whole numbers, so the scores and their distances from the row's maximum are exact: what is left is the exponential and
    the division (a few units), at most 16 + 3 additions in a lane and 5 between lanes, and half the smallest denormal."""
    from paper_2006_06762_amd import binding as anr
    gen = torch.Generator(device="cuda")
    gen.manual_seed(S)
    q, k = (torch.randint(-3, 4, (1, S, SMALL_HEADS, D), device="cuda", generator=gen).float() for _ in range(2))
    out = torch.empty((1, SMALL_HEADS, S, S), device="cuda")
    anr.tbs(q, k, out)
    scores = q.permute(0, 2, 1, 3).contiguous().double() @ k.permute(0, 2, 3, 1).contiguous().double()
    want = torch.softmax(scores, -1)
    assert bool(((want > 0) & (want < 2.0 ** -126)).any())
    assert bool(((out.double() - want).abs() <= 32 * 2.0 ** -24 * want + 2.0 ** -149).all())
