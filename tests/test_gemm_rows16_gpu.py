"""The GEMM by 16 x 16 tiles: edges of its tiles, of the 64-wide chunks and of the 16 k of a lane, fewer chunks than waves, both
kinds of run; and 32 x 32 tiles past its line, which the same edges no longer reach."""
import subprocess

import pytest

from test_gemm_plan_cpu import CSRC

torch = pytest.importorskip("torch")
gpu = pytest.mark.gpu

EDGES = [(1, 1, 2), (1, 15, 17), (1, 16, 16), (1, 33, 64), (3, 47, 130), (1, 256, 255), (1, 9, 2040), (16, 17, 60)]
EDGES_K = [97, 112, 113, 127, 191, 193, 511, 513, 577, 799, 801, 1023, 1027, 3001]
PAST = [(1, 300, 260), (3, 129, 161)]
PAST_K = [97, 287, 289, 511, 799, 801, 865, 1025]


def rows16(tmp_path, cases):
    (tmp_path / "takes.cpp").write_text("""
#include <cstdio>
#include "gemm_dispatch.h"
using namespace anr;
int main()
{
    GemmProblem p{};
    long long b, M, N, K;
    while (scanf("%lld %lld %lld %lld", &b, &M, &N, &K) == 4) {
        p.batch = b; p.M = M; p.N = N; p.K = K; p.one_level = p.offsets32 = true;
        p.lines = p.vec = K % 4 == 0 && N % 4 == 0;
        printf("%d", choose_gemm(p) == GemmKernel::rows32 ? 1 + (int)gemm_rows16_takes(p) : 0);
    }
}
""")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", CSRC, str(tmp_path / "takes.cpp"), "-o", str(tmp_path / "takes")], check=True)
    return subprocess.check_output([str(tmp_path / "takes")], input="\n".join(" ".join(map(str, c)) for c in cases), text=True)


def test_its_sizes_reach_it(tmp_path):
    assert set(rows16(tmp_path, [(*e, K) for e in EDGES for K in EDGES_K])) == {"2"}
    assert set(rows16(tmp_path, [(*e, K) for e in PAST for K in PAST_K])) == {"1"}
    assert rows16(tmp_path, [(1, 256, 256, 333), (1, 257, 256, 333), (64, 32, 32, 333), (65, 32, 32, 333), (1, 256, 256, 512), (1, 256, 256, 64)]) == "212100"


@gpu
@pytest.mark.parametrize("batch, M, N, K", [(*e, K) for e in EDGES for K in EDGES_K] + [(*e, K) for e in PAST for K in PAST_K])
def test_edges(batch, M, N, K):
    """Odd distances between rows, NaN and infinities around that must not be multiplied, guards around the result."""
    from paper_2006_06762_amd import binding as anr
    from test_split_gpu import assert_product, uniform
    A = torch.full((batch, M, K + 5), float("nan"), device="cuda")[:, :, 3:K + 3]
    B = torch.full((batch, K, N + 7), float("inf"), device="cuda")[:, :, 1:N + 1]
    A.copy_(uniform(M + K, batch, M, K))
    B.copy_(uniform(N + K, batch, K, N))
    wide = torch.full((batch, M, N + 3), 7.0, device="cuda")
    anr.gemm(A, B, wide[:, :, 1:N + 1])
    assert_product(wide[:, :, 1:N + 1], A.contiguous(), B.contiguous())
    assert bool((wide[:, :, 0] == 7.0).all()) and bool((wide[:, :, N + 1:] == 7.0).all())
    # whole numbers: every partial sum is exact
    A, B = (A * 4).round().contiguous(), (B * 4).round().contiguous()
    C = torch.empty(batch, M, N, device="cuda")
    anr.gemm(A, B, C)
    assert torch.equal(C.double(), A.double() @ B.double())


@gpu
@pytest.mark.parametrize("K", [200, 900])
def test_values(K):
    """Infinities and NaN spoil their own sums alone, a sum near the largest float keeps its compensation."""
    from paper_2006_06762_amd import binding as anr
    from test_split_gpu import assert_product, uniform
    A, B = uniform(3, 1, 70, K), uniform(4, 1, K, 50)
    A[0, 20, K - 1], A[0, 30, 5] = float("inf"), float("nan")
    B[0, 0, 7], B[0, K - 1, 49] = -float("inf"), 0.0
    A[0, 40], A[0, 40, K // 2] = 1e30, 3.2e38
    B[0, K // 2, 9] = 1.0
    C = torch.empty(1, 70, 50, device="cuda")
    anr.gemm(A, B, C)
    assert_product(C, A, B)
