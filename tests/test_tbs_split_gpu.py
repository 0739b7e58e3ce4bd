"""TBS of 129 to 512 keys on bf16 pieces: edges of its key blocks (32), waves (8, 12, 16), query blocks (64) and steps of
16 floats, views and alignments of the result, values that the pieces cannot carry; and that its sizes reach it."""
import subprocess

import numpy as np
import pytest

import oracle
from paper_2006_06762_amd import inputs as I
from test_gemm_plan_cpu import CSRC

torch = pytest.importorskip("torch")
gpu = pytest.mark.gpu

GUARD = 12345.0
# The scores have a standard deviation of 2, so their partial sums stay below 16 and one rounding below 2^-21; the at most
# 16 steps of a sum, the small products' sum and q's, k's and the exponential's own roundings, 24 in all, add up at random
# to 2.4e-6, which the exponential turns into a relative error: eight times that
TOL = 2e-5

# (keys, floats, heads): two kernels, the one on fp32 products or the split GEMM would run these otherwise
EDGES = [(129, 80, 18), (160, 64, 172), (161, 64, 48), (192, 16, 48), (255, 32, 36), (256, 64, 36), (257, 80, 15), (257, 36, 18),
         (288, 256, 18), (320, 80, 20), (383, 64, 24), (384, 48, 24), (385, 100, 16), (385, 16, 24), (416, 252, 14), (511, 64, 18),
         (512, 80, 11), (512, 256, 12), (512, 132, 24), (512, 128, 34)]


def split_takes(tmp_path, cases):
    (tmp_path / "takes.cpp").write_text("""
#include <cstdio>
#include "tbg_dispatch.h"
using namespace anr;
int main()
{
    TbgProblem p{};
    long long S, D, batch;
    int softmax, aligned, offsets;
    while (scanf("%lld %lld %lld %d %d %d", &S, &D, &batch, &softmax, &aligned, &offsets) == 6) {
        p.S = S; p.D = D; p.batch = batch; p.softmax = softmax; p.aligned = aligned; p.offsets32 = offsets; p.out_offsets32 = true;
        printf("%d", (int)tbs_split_takes(p));
    }
}
""")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", CSRC, str(tmp_path / "takes.cpp"), "-o", str(tmp_path / "takes")], check=True)
    text = "\n".join(" ".join(str(int(x)) for x in c) for c in cases)
    return [d == "1" for d in subprocess.check_output([str(tmp_path / "takes")], input=text, text=True)]


def test_its_sizes_reach_it(tmp_path):
    assert all(split_takes(tmp_path, [(*e, 1, 1, 1) for e in EDGES]))
    lines = {(128, 64, 4096, 1, 1, 1): False, (513, 64, 4096, 1, 1, 1): False, (512, 260, 4096, 1, 1, 1): False,
             (512, 64, 4096, 0, 1, 1): False, (512, 64, 4096, 1, 0, 1): False, (512, 64, 4096, 1, 1, 0): False,
             (192, 64, 47, 1, 1, 1): False, (192, 64, 48, 1, 1, 1): True, (160, 64, 170, 1, 1, 1): False, (160, 64, 171, 1, 1, 1): True,
             (256, 56, 64, 1, 1, 1): False, (256, 96, 40, 1, 1, 1): False, (256, 80, 18, 1, 1, 1): True,
             (512, 256, 10, 1, 1, 1): False, (512, 256, 11, 1, 1, 1): True}
    assert split_takes(tmp_path, lines) == list(lines.values())


def run(q, k, out=None):
    from paper_2006_06762_amd import binding as anr
    return anr.tbs(q, k, torch.empty((q.shape[0], q.shape[2], q.shape[1], q.shape[1]), device="cuda") if out is None else out)


def check(got, ref, what):
    err = float(np.max(np.abs(got.astype(np.float64) - ref) / ref.max(-1, keepdims=True)))
    assert err <= TOL, "%s: %.2e of the row's largest" % (what, err)


@gpu
@pytest.mark.parametrize("S, D, heads", EDGES)
def test_edges(S, D, heads):
    s = I.TbgShape(1, S, heads, D)
    q, k = I.tbg_inputs(s, 2400 + S + D)
    q = (q * (2.0 / D ** 0.5)).astype(np.float32)
    n = heads * S * S
    buf = torch.full((n + 128,), GUARD, device="cuda")
    run(torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda(), buf[64:64 + n].view(1, heads, S, S))
    check(buf[64:64 + n].view(1, heads, S, S).cpu().numpy(), oracle.tbs(q, k), "S %d D %d" % (S, D))
    assert bool((buf[:64] == GUARD).all()) and bool((buf[-64:] == GUARD).all())


@gpu
@pytest.mark.parametrize("S", [224, 300, 416])
@pytest.mark.parametrize("pad, start", [(0, 0), (32, 0), (4, 4), (3, 1)])
def test_views(S, pad, start):
    """Two sequences, q and k as slices of a projection that holds both, rows of the result further apart than they are long."""
    B, H, D = 2, 18, 80
    q, k = I.tbg_inputs(I.TbgShape(B, S, H, D), 2500 + S)
    q = (q * 0.25).astype(np.float32)
    both = torch.full((B, S, 2, H, D + 4), GUARD, device="cuda")
    both[:, :, 0, :, :D], both[:, :, 1, :, :D] = torch.from_numpy(q), torch.from_numpy(k)
    buf = torch.full((B * H * S * (S + pad) + 8,), GUARD, device="cuda")
    wide = buf[start:start + B * H * S * (S + pad)].view(B, H, S, S + pad)
    run(both[:, :, 0, :, :D], both[:, :, 1, :, :D], wide[..., :S])
    check(wide[..., :S].cpu().numpy(), oracle.tbs(q, k), "view %d %d" % (pad, start))
    assert bool((wide[..., S:] == GUARD).all())


@gpu
@pytest.mark.parametrize("S", [200, 300, 500])
def test_values_the_pieces_cannot_carry(S):
    """Infinities, NaN, values near the largest and far below the smallest that three pieces hold: as a product in 64 bits and
    torch's softmax give them, and the head beside is what it is without them."""
    D, H = 80, 18
    gen = torch.Generator(device="cuda").manual_seed(S)
    q, k = (torch.randn((1, S, H, D), device="cuda", generator=gen) * 0.3 for _ in range(2))
    clean = run(q, k)
    q, k = q.clone(), k.clone()
    k[0, S - 1, 0, 3] = -float("inf")
    q[0, :, 0, 3] = 1.0
    q[0, 7, 0, 2] = float("nan")
    q[0, 64, 1, 5], k[0, 9, 1, 5] = 3e38, 1.0
    q[0, :, 2] *= 2.0 ** -126
    k[0, :, 2] *= 2.0 ** 126
    q[0, 130, 3, :] = 1e-39
    out = run(q, k)
    ref = torch.softmax(q[0].permute(1, 0, 2).contiguous().double() @ k[0].permute(1, 2, 0).contiguous().double(), -1)
    assert torch.equal(out[0].isnan(), ref.isnan()) and int(ref.isnan().any(-1).sum()) == 1
    assert bool((out[0, 0][~ref[0].isnan().any(-1)][:, S - 1] == 0).all())
    assert out[0, 1, 64].argmax() == 9 or ref[1, 64].argmax() != 9
    ok = ~ref.isnan().any(-1)
    ok[1, 64] = False                    # scores of 1e38: the largest alone survives
    assert float((out[0].double() - ref)[ok].abs().max()) <= TOL
    assert torch.equal(out[0, 4:], clean[0, 4:])


@gpu
@pytest.mark.parametrize("S, D", [(161, 80), (300, 64), (511, 48)])
def test_small_probabilities(S, D):
    """Whole numbers, so the scores and their distances from the row's maximum are exact: what is left is the exponential and
    the division (a few units), at most 4 additions in a lane and 6 between lanes, and half the smallest denormal."""
    gen = torch.Generator(device="cuda").manual_seed(S)
    q, k = (torch.randint(-3, 4, (1, S, 48, D), device="cuda", generator=gen).float() for _ in range(2))
    out = run(q, k)
    want = torch.softmax(q.permute(0, 2, 1, 3).contiguous().double() @ k.permute(0, 2, 3, 1).contiguous().double(), -1)
    assert bool(((want > 0) & (want < 2.0 ** -126)).any())
    assert bool(((out.double() - want).abs() <= 32 * 2.0 ** -24 * want + 2.0 ** -149).all())


# whole chunks of 32 floats, a last one that starts at D - 32 and counts part of itself, less than one
@gpu
@pytest.mark.parametrize("S, D, heads", [(256, 128, 128), (384, 48, 72), (250, 80, 150), (500, 100, 64), (256, 16, 192), (200, 252, 200), (320, 32, 128)])
def test_its_scores_are_those_of_the_scores_alone(S, D, heads):
    """Where the split GEMM takes those: softmax of the same bits, so equal queries of one key block give equal rows and the
    row's distances come out as the scores' own: log(p_i / p_max) against the difference, to the exponential's few units."""
    from paper_2006_06762_amd import binding as anr
    gen = torch.Generator(device="cuda").manual_seed(S + D)
    q, k = (torch.empty((1, S, heads, D), device="cuda").uniform_(-1, 1, generator=gen) for _ in range(2))
    scores = anr.tbg(q, k, torch.empty((1, heads, S, S), device="cuda"))
    below = (scores - scores.amax(-1, keepdim=True)).double()
    want = torch.softmax(scores.double(), -1)
    out = run(q, k).double()
    # the exponential 1.5 units, its argument's two roundings, the sum of up to 512 as a tree, the division; all of a few units
    assert bool(((out - want).abs() <= (16 - 2 * below) * 2.0 ** -24 * want + 2.0 ** -148).all())


# ------------------------------------------------------------------ every product of pieces that is formed
PAIRS = [("h", "m"), ("m", "h"), ("m", "m"), ("h", "l"), ("l", "h"), ("m", "l"), ("l", "m")]
PIECES = {"h": 1.0, "m": 2.0 ** -9, "l": 2.0 ** -18}


def up_to(piece):
    return sum(v for p, v in PIECES.items() if "hml".index(p) <= "hml".index(piece))


def one_product(pair, S, heads, D, at):
    """q and k whose scores are the product of one piece of each: three columns from `at` on, in which all else cancels and every
    partial sum is exact.  Both, and the factors that are left: +-1 a query, 0, +-1 or +-2 a key."""
    a, b = pair
    rng = np.random.default_rng(S + D + at)
    left, right = rng.choice([-1.0, 1.0], (S, heads)), rng.choice([-2.0, -1.0, 0.0, 1.0, 2.0], (S, heads))
    q, k = np.zeros((2, 1, S, heads, D))
    q[0, :, :, at:at + 3] = left[..., None] * [up_to(a), PIECES[a] - up_to(a), -PIECES[a]] / PIECES[a]
    k[0, :, :, at:at + 3] = right[..., None] * [up_to(b), up_to(b), up_to(b) - PIECES[b]] / PIECES[b]
    return q.astype(np.float32), k.astype(np.float32), left, right


def split(x):
    """The three bf16 pieces of a float32 array, each rounded to nearest, as float64."""
    t = torch.from_numpy(x)
    out = []
    for _ in range(3):
        piece = t.to(torch.bfloat16).float()
        out.append(piece.double().numpy())
        t = t - piece
    return out


@pytest.mark.parametrize("pair", PAIRS)
def test_one_product_tells_all(pair):
    """The model of the kernel's sum gives those scores, and none where that product is left out."""
    q, k, left, right = one_product(pair, 130, 2, 40, 33)
    pq, pk = split(q), split(k)
    want = np.einsum("ih,jh->hij", left, right)
    for left_out in (None, pair):
        s = sum(np.einsum("bihd,bjhd->hij", pq[i], pk[j]) for i, p in enumerate("hml") for j, r in enumerate("hml")
                if p + r != "ll" and (p, r) != left_out)
        assert np.array_equal(s, want if left_out is None else np.zeros_like(want))
    assert {-2.0, 0.0, 2.0} <= set(np.unique(want))


# (keys, floats, heads), and whether the scores alone are the split GEMM's
SUMS = [(257, 36, 18, 0), (257, 80, 15, 0), (385, 100, 16, 0), (416, 252, 14, 0), (192, 64, 48, 0), (512, 128, 34, 1), (250, 80, 150, 1)]


def test_sums_of_both_orders_are_among_them(tmp_path):
    text = (tmp_path / "takes.cpp")
    assert all(split_takes(tmp_path, [(*s[:3], 1, 1, 1) for s in SUMS]))
    text.write_text(text.read_text().replace("tbs_split_takes(p)", "tbg_split_takes(p)"))
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", CSRC, str(text), "-o", str(tmp_path / "takes")], check=True)
    lines = "\n".join("%d %d %d 1 1 1" % s[:3] for s in SUMS)
    assert subprocess.check_output([str(tmp_path / "takes")], input=lines, text=True) == "".join(str(s[3]) for s in SUMS)


@gpu
@pytest.mark.parametrize("S, D, heads, as_gemm", SUMS)
@pytest.mark.parametrize("pair", PAIRS)
def test_every_product_of_pieces_is_in_the_scores(S, D, heads, as_gemm, pair):
    """Columns of the first step, of one in the middle and of the last: the scores are exact, what is left is the exponential (a
    few units) and a tree of at most 512 equal-signed terms, 6 roundings of lanes and waves.  Not those of 2^-27 of the largest
    products in the last step of sums which have the small products' sum added ahead of its large ones: one instruction then
    adds both, with a rounding of 2^-24."""
    last = [D - 3] if as_gemm or pair not in (("m", "l"), ("l", "m")) else []
    for at in (0, D // 2 // 16 * 16 + 5, *last):
        q, k, left, right = one_product(pair, S, heads, D, at)
        out = run(torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda())[0]
        scores = torch.from_numpy(np.einsum("ih,jh->hij", left, right)).cuda()
        want = torch.softmax(scores, -1)
        assert bool(((out.double() - want).abs() <= 32 * 2.0 ** -24 * want).all()), at
