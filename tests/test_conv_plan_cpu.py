"""Host arithmetic of the patch-staging convolution's plan against the definition it shortens."""
import random
import subprocess

from paper_2006_06762_amd import binding as B
from test_gemm_plan_cpu import CSRC


def test_virtual_rows_of_a_tile(tmp_path):
    (tmp_path / "rows.cpp").write_text("""
#include <cstdio>
#include "conv_igemm_plan.h"
int main()
{
    int N, OH, OW, stride, R, bm, hv;
    while (scanf("%d %d %d %d %d %d %d", &N, &OH, &OW, &stride, &R, &bm, &hv) == 7)
        printf("%d ", anr::igemm::max_virtual_rows(N, OH, OW, stride, R, bm, hv));
}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(tmp_path / "rows.cpp"), "-o", str(tmp_path / "rows")], check=True)
    rng = random.Random(5)
    cases = [(1, 1, 1, 1, 3, 64, 3), (1, 1, 300, 1, 3, 64, 3), (300, 1, 1, 2, 3, 224, 3), (7, 132, 132, 1, 3, 224, 134), (1, 8, 8, 1, 3, 64, 10), (3, 8, 8, 5, 3, 64, 38)]
    for _ in range(600):
        OH, stride = rng.choice([1, 2, 3, 7, 14, rng.randint(1, 60)]), rng.choice([1, 1, 2, 3, 4])
        cases.append((rng.randint(1, 9), OH, rng.choice([1, 2, 7, 14, 28, 56, rng.randint(1, 90)]), stride, 3, rng.choice([64, 128, 224]), (OH - 1) * stride + 3))
    want = []
    for N, OH, OW, stride, R, bm, hv in cases:
        total, most = N * OH * OW, 0
        row = lambda m: m // OW // OH * hv + m // OW % OH * stride
        for m in range(0, total, bm):
            most = max(most, row(min(m + bm, total) - 1) - row(m))
        want.append(most + R)
    text = "\n".join(" ".join(map(str, c)) for c in cases)
    assert list(map(int, subprocess.check_output([str(tmp_path / "rows")], input=text, text=True).split())) == want


def test_layers_that_the_pieces_would_slow_down():
    """Few rounds for each of four groups of waves and a split reduction: with the pieces 19.0 -> 23.3, 20.0 -> 23.7, 17.2 -> 19.8 and
    23.6 -> 25.3 us, so these are not given room for them; one with more rounds (37.8 -> 33.9) and one without a split
    (20.0 -> 18.2) are."""
    def more(x, K, R, groups=1):
        d = B.conv_desc(x, K, R, R, (1, 1), (R // 2, R // 2), groups=groups)
        return B.conv2d_fast_workspace_size(d) - B.workspace_size(B.ANR_OP_CONV2D, d)
    assert [more((4, 256, 8, 123), 32, 3), more((1, 512, 45, 45), 32, 3), more((16, 100, 12, 41), 32, 3), more((1, 256, 21, 99), 96, 3)] == [0] * 4
    assert more((32, 512, 7, 7), 160, 3) > 0 and more((3, 32, 40, 40), 128, 7, 4) > 0
