"""Timed cases of the fp32 operator library: what its callers have it do, through the public binding.

Each case is one operator call (or, for the ConvLayer, the packed call an inference program makes) on
tensors the caller already holds.  Shapes are those of the operator and subgraph lists of arXiv 2006.06762
(Appendix C: batch 1 and 16) and of this repository's own benchmark step and tests, plus ragged ones of the
same ranges.  Everything is float32: the library has no other type.
"""
import math

import torch

from paper_2006_06762_amd import binding as anr

EPS = 1e-5


def _conv(name, op, N, C, H, W, K, R, stride, pad, dil=1, groups=1):
    case = {"op": op, "N": N, "C": C, "H": H, "W": W, "K": K, "R": R, "stride": stride, "pad": pad, "dil": dil,
            "groups": groups}
    return dict(case, name=name) if name else case


def _gemm(name, batch, M, N, K):
    case = {"op": "gemm", "batch": batch, "M": M, "N": N, "K": K}
    return dict(case, name=name) if name else case


def _scores(name, op, B, S, H, D):
    case = {"op": op, "B": B, "S": S, "H": H, "D": D}
    return dict(case, name=name) if name else case


def _nrm(name, batch, N, M):
    case = {"op": "nrm", "batch": batch, "N": N, "M": M}
    return dict(case, name=name) if name else case


def listed():
    return [
        # A single small product, as one request through a small dense layer: latency of one launch.
        _gemm("gemm_128", 1, 128, 128, 128),
        # The paper's middle GMM at its larger batch: sixteen independent ordinary products in one call.
        _gemm("gemm_512_x16", 16, 512, 512, 512),
        # Sizes that are no multiple of anything, as vocabularies and padded-free batches have them.
        _gemm("gemm_ragged", 3, 1009, 1531, 771),
        # The largest product: a dense layer of a large model.
        _gemm("gemm_4096", 1, 4096, 4096, 4096),
        # Stem of an image network: three input channels, 7x7, stride 2, the largest maps.
        _conv("conv_stem_7x7", "conv2d", 16, 3, 224, 224, 64, 7, 2, 3),
        # The 3x3 layer of a residual network's first stage, the repository's benchmark convolution.
        _conv("conv_3x3_56", "conv2d", 16, 64, 56, 56, 64, 3, 1, 1),
        # ConvLayer as inference runs it (constants packed once, batch norm and ReLU fused): third stage.
        _conv("convlayer_packed_14", "convlayer_packed", 16, 256, 14, 14, 256, 3, 1, 1),
        # The last stage's 3x3 layer for a single image: small maps, a long reduction, latency counts.
        _conv("conv_7x7map_b1", "conv2d", 1, 512, 7, 7, 512, 3, 1, 1),
        # The pointwise layer that starts a bottleneck.
        _conv("convlayer_1x1_56", "convlayer", 16, 64, 56, 56, 64, 1, 1, 0),
        # Depthwise 3x3 of a mobile network's early stage with its down-sampling: a stream over memory.
        _conv("dwconv_s2_112", "dwconv", 16, 64, 112, 112, 64, 3, 2, 1),
        # Attention scores with softmax, twelve heads, sequence 128, batch 16.
        _scores("tbs_128", "tbs", 16, 128, 12, 64),
        # Norm of sixteen large matrices: one reduction over a gigabyte.
        _nrm("nrm_4096_x16", 16, 4096, 4096),
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


_MOST_FLOPS = 40e9      # a drawn convolution or product stays under a third of gemm_4096
_MOST_BYTES = 600e6     # and under the bytes of nrm_4096_x16


def draw(rng):
    while True:
        op = rng.choice(["gemm", "gemm", "conv2d", "conv2d", "convlayer", "convlayer_packed", "dwconv", "tbg", "tbs",
                         "nrm"])
        if op == "gemm":
            def size():
                n = _log(rng, 32, 4096)
                return n if rng.random() < 0.3 else max(32, n // 32 * 32)
            case = _gemm(None, rng.choice([1, 1, 3, 16]), size(), size(), size())
        elif op in ("conv2d", "convlayer", "convlayer_packed"):
            R = rng.choice([1, 1, 3, 3, 3, 5, 7])
            C = rng.choice([3, 16, 32, 48, 64, 100, 128, 192, 256, 512])
            K = rng.choice([32, 64, 96, 128, 160, 256, 384, 512])
            H = _log(rng, 7, 224)
            W = H if rng.random() < 0.8 else _log(rng, 7, 224)
            groups = 4 if C % 4 == 0 and rng.random() < 0.15 else 1
            dil = 2 if rng.random() < 0.15 else 1
            case = _conv(None, op, rng.choice([1, 1, 4, 7, 16, 16, 32]), C, H, W, K, R, rng.choice([1, 1, 2]),
                         R // 2 * dil, dil, groups)
        elif op == "dwconv":
            H = _log(rng, 7, 224)
            W = H if rng.random() < 0.8 else _log(rng, 7, 224)
            R = rng.choice([3, 3, 3, 5])
            C = _log(rng, 32, 1024)
            case = _conv(None, op, rng.choice([1, 4, 16, 32]), C, H, W, C, R, rng.choice([1, 2]), R // 2)
        elif op in ("tbg", "tbs"):
            case = _scores(None, op, rng.choice([1, 4, 16, 32]), _log(rng, 32, 512), rng.choice([8, 12, 16]),
                           rng.choice([32, 64, 80, 128]))
        else:
            case = _nrm(None, rng.choice([1, 4, 16]), _log(rng, 64, 4096), _log(rng, 64, 4096))
        need = work(case)
        if need["flops"] <= _MOST_FLOPS and need["bytes"] <= _MOST_BYTES:
            return case


def _out_hw(c):
    span = c["dil"] * (c["R"] - 1) + 1
    return ((c["H"] + 2 * c["pad"] - span) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - span) // c["stride"] + 1)


def _tensors(case, seed):
    """The inputs of a case, from the seed alone, with the distributions of the repository's benchmark."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def uniform(*shape, lo=-1.0, hi=1.0):
        return torch.empty(shape, device="cuda", dtype=torch.float32).uniform_(lo, hi, generator=gen)

    def normal(*shape, sigma=1.0):
        return torch.empty(shape, device="cuda", dtype=torch.float32).normal_(0.0, sigma, generator=gen)

    c, op = case, case["op"]
    if op == "gemm":
        lead = (c["batch"],) if c["batch"] > 1 else ()
        return {"A": uniform(*lead, c["M"], c["K"]), "B": uniform(*lead, c["K"], c["N"])}
    if op in ("tbg", "tbs"):
        dims = (c["B"], c["S"], c["H"], c["D"])
        return {"q": normal(*dims), "k": normal(*dims)}
    if op == "nrm":
        return {"x": uniform(c["batch"], c["N"], c["M"])}
    per = 1 if op == "dwconv" else c["C"] // c["groups"]
    t = {"x": uniform(c["N"], c["C"], c["H"], c["W"]), "w": normal(c["K"], per, c["R"], c["R"], sigma=0.05)}
    if op.startswith("convlayer"):
        K = c["K"]
        t["bn"] = (uniform(K, lo=0.5, hi=1.5), uniform(K, lo=-0.1, hi=0.1), normal(K, sigma=0.1),
                   uniform(K, lo=0.5, hi=2.0))
    return t


def prepare(case, seed):
    t, c, op = _tensors(case, seed), case, case["op"]
    state = dict(t, op=op)
    if op == "gemm":
        lead = (c["batch"],) if c["batch"] > 1 else ()
        state["C"] = torch.empty(*lead, c["M"], c["N"], device="cuda")
    elif op in ("tbg", "tbs"):
        state["out"] = torch.empty(c["B"], c["H"], c["S"], c["S"], device="cuda")
    elif op == "nrm":
        state["out"] = torch.empty(c["batch"], device="cuda")
    else:
        state["y"] = torch.empty(c["N"], c["K"], *_out_hw(c), device="cuda")
        state["stride"] = (c["stride"], c["stride"])
        state["pad"] = (c["pad"], c["pad"])
        state["dil"] = (c["dil"], c["dil"])
        state["groups"] = c["groups"]
        if op == "convlayer_packed":
            state["desc"], state["pack"] = anr.conv2d_pack_weights(t["x"].shape, t["w"], state["stride"], state["pad"],
                                                                   bn=t["bn"], eps=EPS, dil=state["dil"],
                                                                   groups=c["groups"])
    return state


def run(s):
    op = s["op"]
    if op == "gemm":
        return anr.gemm(s["A"], s["B"], s["C"])
    if op == "conv2d":
        return anr.conv2d(s["x"], s["w"], s["y"], s["stride"], s["pad"], dil=s["dil"], groups=s["groups"])
    if op == "convlayer":
        return anr.conv_bn_relu(s["x"], s["w"], *s["bn"], EPS, s["y"], s["stride"], s["pad"], dil=s["dil"],
                                groups=s["groups"])
    if op == "convlayer_packed":
        return anr.conv_bn_relu_packed(s["desc"], s["x"], s["pack"], s["y"])
    if op == "dwconv":
        return anr.dwconv(s["x"], s["w"], s["y"], s["stride"], s["pad"], s["dil"])
    if op == "tbg":
        return anr.tbg(s["q"], s["k"], s["out"])
    if op == "tbs":
        return anr.tbs(s["q"], s["k"], s["out"])
    return anr.nrm(s["x"], s["out"])


def work(case):
    c, op = case, case["op"]
    if op == "gemm":
        return {"bytes": 4 * c["batch"] * (c["M"] * c["K"] + c["K"] * c["N"] + c["M"] * c["N"]),
                "flops": 2 * c["batch"] * c["M"] * c["N"] * c["K"]}
    if op in ("tbg", "tbs"):
        heads = c["B"] * c["H"]
        return {"bytes": 4 * heads * (2 * c["S"] * c["D"] + c["S"] * c["S"]), "flops": 2 * heads * c["S"] ** 2 * c["D"]}
    if op == "nrm":
        n = c["batch"] * c["N"] * c["M"]
        return {"bytes": 4 * n, "flops": 2 * n}
    OH, OW = _out_hw(c)
    per = 1 if op == "dwconv" else c["C"] // c["groups"]
    out = c["N"] * c["K"] * OH * OW
    return {"bytes": 4 * (c["N"] * c["C"] * c["H"] * c["W"] + c["K"] * per * c["R"] ** 2 + out),
            "flops": 2 * out * per * c["R"] ** 2}


def tolerance(case):
    """Four times the distance from the 64-bit results measured for 32-bit sums of the case's length: 4.0e-7 at 512
    terms, 4.9e-7 at 771, 1.1e-6 at 4096, so 1.75e-8 per square root of a term."""
    op = case["op"]
    if op == "nrm":
        return {"rel": 2e-7}        # 4.1e-8 measured
    if op == "dwconv":
        return {"rel": 3e-7}        # 5.0e-8 and, for 5x5, 7e-8 measured
    if op == "tbs":
        return {"rel": 4e-6}        # 8.2e-7 measured: a score's rounding error e changes its exponential by 1 + e
    if op == "tbg":
        terms = case["D"]
    elif op == "gemm":
        terms = case["K"]
    else:
        terms = case["C"] // case["groups"] * case["R"] ** 2
    return {"rel": max(4e-7, 7e-8 * math.sqrt(terms))}


def exact(case, seed):
    t, c, op = _tensors(case, seed), case, case["op"]
    if op == "gemm":
        return t["A"].double() @ t["B"].double()
    if op in ("tbg", "tbs"):
        q = t["q"].double().permute(0, 2, 1, 3).contiguous()
        k = t["k"].double().permute(0, 2, 3, 1).contiguous()
        s = q @ k
        return torch.softmax(s, -1) if op == "tbs" else s
    if op == "nrm":
        return t["x"].double().square().sum((1, 2)).sqrt()
    OH, OW = _out_hw(c)
    x = torch.nn.functional.pad(t["x"].double(), (c["pad"],) * 4)
    w = t["w"].double()
    G = c["C"] if op == "dwconv" else c["groups"]
    Cg, Kg, st, dil = c["C"] // G, c["K"] // G, c["stride"], c["dil"]
    y = torch.zeros(c["N"], G, Kg, OH * OW, device="cuda", dtype=torch.float64)
    for r in range(c["R"]):
        for s in range(c["R"]):
            tap = x[:, :, r * dil:r * dil + st * (OH - 1) + 1:st, s * dil:s * dil + st * (OW - 1) + 1:st]
            tap = tap.reshape(c["N"], G, Cg, OH * OW)
            wt = w[:, :, r, s].reshape(G, Kg, Cg)
            y += tap * wt.reshape(1, G, 1, 1) if op == "dwconv" else wt @ tap
    y = y.reshape(c["N"], c["K"], OH, OW)
    if op.startswith("convlayer"):
        gamma, beta, mean, var = (v.double().reshape(1, -1, 1, 1) for v in t["bn"])
        y = torch.relu(gamma * (y - mean) / torch.sqrt(var + EPS) + beta)
    return y
