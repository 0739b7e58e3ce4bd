"""The bf16-split GEMM's staging, walked thread by thread on the CPU with the kernel's own index arithmetic: every
load inside its matrix (or past the extent by the lane's part of the offset alone), every k counted once."""
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


def test_variant_shapes_select_their_variants(tmp_path):
    """The GPU tests' shapes run the tile and wave groups they are listed for, and every variant has one."""
    torch_tests = pytest.importorskip("test_split_gpu")
    src = tmp_path / "choose.cpp"
    src.write_text("""
#include <cstdio>
#include <cstdlib>
#include "gemm_split_plan.h"
int main(int, char** v)
{
    const auto& c = anr::gsplit::kVariants[anr::gsplit::choose_variant(atoi(v[2]), atoi(v[3]), atoi(v[4]), atoi(v[1]))];
    printf("%d %d %d", c.tile, c.groups, anr::gsplit::kVariantCount);
}
""")
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(tmp_path / "choose")], check=True)
    choose = lambda shape: tuple(map(int, subprocess.check_output([str(tmp_path / "choose"), *map(str, shape)]).split()))
    for variant, shape in torch_tests.VARIANTS.items():
        assert choose(shape) == (*variant, len(torch_tests.VARIANTS))
    for variant, (B, S, H, D) in torch_tests.SCORES.items():
        assert choose((B * H, S, S, D)) == (*variant, len(torch_tests.SCORES)) and D % 4 != 0
