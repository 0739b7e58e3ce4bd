"""The bf16-split GEMM's staging, walked thread by thread on the CPU with the kernel's own index arithmetic: every
load inside its matrix (or past the extent by the lane's part of the offset alone), every k counted once.  And the
rules by which products and attention scores choose their kernels."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2006_06762_amd", "csrc")


@pytest.fixture(scope="module")
def staging(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "staging")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, os.path.join(HERE, "gemm_split_staging.cpp"), "-o", exe],
                   check=True)
    return lambda *args: subprocess.run([exe, *map(str, args)], capture_output=True, text=True)


# tails of K of every kind (below a chunk, one past, one short), odd and even N, one pair of columns, single rows
@pytest.mark.parametrize("tile,groups", [(64, 1), (64, 2), (64, 4), (128, 1), (128, 2), (256, 1)])
@pytest.mark.parametrize("M,N,K,nt", [(*s, nt) for s in [(65, 3, 33), (1, 2, 31), (70, 129, 1), (63, 66, 95), (3, 65, 64), (66, 64, 17), (2, 67, 161)]
                                      for nt in (0, 1) if nt or s[2] >= 32])
@pytest.mark.parametrize("pad", [0, 3])
def test_split_gemm_staging_stays_inside_and_counts_once(staging, tile, groups, M, N, K, nt, pad):
    res = staging(tile, groups, M, N, K, pad, nt)
    assert res.returncode == 0, res.stdout + res.stderr


@pytest.fixture(scope="module")
def dispatch(tmp_path_factory):
    """What launch_gemm runs for a product in packed tensors (all of them 16-byte aligned): kernel, tile and wave groups of
    the split GEMM, and how many such variants there are."""
    where = tmp_path_factory.mktemp("dispatch")
    (where / "choose.cpp").write_text("""
#include <cstdio>
#include <cstdlib>
#include "gemm_dispatch.h"
using namespace anr;
int main(int, char** v)
{
    GemmProblem p{};
    p.batch = atoi(v[1]); p.M = atoi(v[2]); p.N = atoi(v[3]); p.K = atoi(v[4]); p.nk = atoi(v[5]);
    p.one_level = !p.nk;
    p.offsets32 = true;
    p.lines = p.K % 4 == 0 && p.N % 4 == 0;
    p.vec = p.K % 4 == 0 && p.N % 4 == 0;
    const char* const names[] = {"ksplit", "rows32", "pipe", "split", "plain"};
    const auto& c = gsplit::kVariants[gsplit::choose_variant(p.M, p.N, p.K, p.batch)];
    printf("%s %d %d %d", names[(int)choose_gemm(p)], c.tile, c.groups, gsplit::kVariantCount);
}
""")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", CSRC, str(where / "choose.cpp"), "-o", str(where / "choose")], check=True)

    def choose(batch, M, N, K, nk=0):
        kernel, *rest = subprocess.check_output([str(where / "choose"), *map(str, (batch, M, N, K, nk))], text=True).split()
        return (kernel, *map(int, rest))
    return choose


def test_shapes_of_the_gpu_tests_run_what_they_are_listed_for(dispatch):
    """Kernel, tile and wave groups, and every variant of the split GEMM has a shape."""
    split = pytest.importorskip("test_split_gpu")
    rows32 = pytest.importorskip("test_gemm_rows32_gpu")
    for variant, shape in split.VARIANTS.items():
        assert dispatch(*shape) == ("split", *variant, len(split.VARIANTS)), shape
    for variant, (B, S, H, D) in split.SCORES.items():
        assert dispatch(B * H, S, S, D, 1) == ("split", *variant, len(split.SCORES)) and D % 4 != 0
    # (views of odd strides: never aligned, here by their odd extents; 700 x 700 x 545 has 484 tiles)
    assert [dispatch(1, *shape)[0] for shape in split.UNALIGNED] == ["rows32", "rows32", "split", "split", "split"]
    assert {dispatch(1, *shape)[1:3] for shape in split.UNALIGNED[2:]} >= {(64, 4), (128, 2)}
    for M, N in rows32.EDGES:
        for K in rows32.EDGES_K:
            # past 256 tiles it starts at 97: those two lengths are the other side of the line
            want = "ksplit" if (M, N, K) == (32, 32, 128) else "plain" if M == 129 and K < 97 else "rows32"
            assert dispatch(1, M, N, K)[0] == want, (M, N, K)
    for shape in rows32.VIEWS:
        assert dispatch(*shape)[0] == "rows32"


def test_dispatch_at_its_lines(dispatch):
    """256 and 512 tiles of 32 x 32, the shortest reductions on either side."""
    for (M, N, K), want in {(511, 512 - 1, 65): "rows32", (511, 511, 64): "plain", (512, 512, 96): "pipe", (512, 512, 100): "rows32",
                            (511, 1023, 97): "rows32", (511, 1023, 96): "plain", (511, 1025, 333): "split", (512, 1028, 300): "pipe",
                            (512, 1024, 128): "ksplit", (1024, 1024, 256): "ksplit", (1024, 1056, 256): "split"}.items():
        assert dispatch(1, M, N, K)[0] == want, (M, N, K)


@pytest.fixture(scope="module")
def scores(tmp_path_factory):
    """What launch_tbg runs for packed tensors."""
    where = tmp_path_factory.mktemp("scores")
    (where / "choose.cpp").write_text("""
#include <cstdio>
#include <cstdlib>
#include "tbg_dispatch.h"
using namespace anr;
int main(int, char** v)
{
    TbgProblem p{};
    p.S = atoi(v[1]); p.D = atoi(v[2]); p.batch = atoi(v[3]); p.softmax = atoi(v[4]);
    p.aligned = p.D % 4 == 0;
    p.offsets32 = p.out_offsets32 = true;
    const char* const names[] = {"rows32", "rows_long", "tile64", "tile", "gemm"};
    printf("%s", names[(int)choose_tbg(p)]);
}
""")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", CSRC, str(where / "choose.cpp"), "-o", str(where / "choose")], check=True)
    return lambda *args: subprocess.check_output([str(where / "choose"), *map(str, args)], text=True)


def test_long_scores_of_the_gpu_tests_run_the_one_kernel(scores):
    long = pytest.importorskip("test_tbs_long_gpu")
    for S, D, heads in long.EDGES:
        assert scores(S, D, heads, 1) == "rows_long", (S, D, heads)
    assert {((S + 127) // 128, D) for S, D, heads in long.EDGES} >= {(2, 256), (3, 168), (4, 128)}
    B, S, H, D = long.VIEW
    assert scores(S, D, B * H, 1) == "rows_long"
    for S, D in long.SMALL:
        assert scores(S, D, long.SMALL_HEADS, 1) == "rows_long"
    assert scores(300, 16, 1, 1) == "rows_long"          # values that are not finite


def test_scores_dispatch_at_its_lines(scores):
    """128 and 512 keys, few and enough work-groups, long walks, the split GEMM's sizes; scores alone never."""
    for (S, D, heads, softmax), want in {(128, 64, 200, 1): "rows32", (129, 64, 16, 1): "rows_long", (129, 64, 12, 1): "tile",
                                         (384, 104, 14, 1): "tile", (384, 104, 15, 1): "rows_long", (136, 80, 17, 1): "tile", (136, 80, 18, 1): "rows_long", (384, 128, 24, 1): "rows_long",
                                         (320, 192, 48, 1): "tile64", (512, 256, 24, 1): "tile64", (512, 64, 48, 1): "rows_long",
                                         (513, 64, 20, 1): "tile", (512, 128, 32, 1): "gemm", (384, 128, 57, 1): "gemm", (256, 64, 100, 0): "tile64",
                                         (300, 36, 40, 1): "tile", (300, 33, 40, 1): "gemm"}.items():
        assert scores(S, D, heads, softmax) == want, (S, D, heads, softmax)


def test_pointwise_route_reports_the_gemm_it_runs(dispatch):
    """Tile, wave groups and work-groups of a pointwise layer that runs as a GEMM: the variant of weights times image."""
    from paper_2006_06762_amd import binding as B
    gpu = pytest.importorskip("test_conv_pointwise_gemm_gpu")
    seen = set()
    for N, C, H, W, K in [*gpu.SHAPES, (16, 512, 45, 45, 256), (1, 2000, 57, 57, 512), (2, 700, 61, 61, 200), (32, 64, 85, 85, 384)]:
        r = B.conv2d_route(B.conv_desc((N, C, H, W), K, 1, 1))
        _, tile, groups, _ = dispatch(N, K, H * W, C)
        assert r.kernel == B.ANR_CONV_KERNEL_POINTWISE
        assert (r.tile_m, r.tile_n, r.wave_groups) == (tile, tile, groups)
        assert r.work_groups == N * -(-K // tile) * -(-H * W // tile)
        seen.add((tile, groups))
    assert len(seen) >= 4 and max(g for _, g in seen) > 1
