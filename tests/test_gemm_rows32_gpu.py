"""The GEMM of few 32 x 32 tiles: edges of its tiles and 32-wide chunks, fewer chunks than waves, every number of folds,
views of any alignment, batches; values that are not finite; an error that does not grow with K."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_split_gpu import assert_product, uniform


# (32 x 32 x 128 is another kernel's, and so is K below 97 with more than 256 tiles: the other sides of two lines)
EDGES = [(1, 2), (31, 33), (32, 32), (33, 64), (65, 95), (200, 130), (129, 3000)]
EDGES_K = [65, 95, 97, 128, 159, 287, 288, 290, 511, 799, 801, 1023, 1025, 2049]
VIEWS = [(1, 70, 50, 333), (3, 45, 101, 700), (16, 33, 31, 1100)]


@pytest.mark.parametrize("M,N", EDGES)
@pytest.mark.parametrize("K", EDGES_K)
def test_edges(M, N, K):
    from paper_2006_06762_amd import binding as anr
    A, B = uniform(M + K, M, K), uniform(N + K, K, N)
    buf = torch.full((M * N + 128,), 7.0, device="cuda")
    C = buf[64:-64].view(M, N)
    anr.gemm(A, B, C)
    assert_product(C, A, B)
    assert bool((buf[:64] == 7.0).all()) and bool((buf[-64:] == 7.0).all())
    # whole numbers: every partial sum is exact
    A, B = (A * 4).round(), (B * 4).round()
    anr.gemm(A, B, C)
    assert torch.equal(C.double(), A.double() @ B.double())


@pytest.mark.parametrize("batch,M,N,K", VIEWS)
def test_views(batch, M, N, K):
    """Rows that lie apart at odd distances, behind NaN and infinities that must not be multiplied."""
    from paper_2006_06762_amd import binding as anr
    A = torch.full((batch, M, K + 5), float("nan"), device="cuda")[:, :, 3:K + 3]
    B = torch.full((batch, K, N + 7), float("inf"), device="cuda")[:, :, 1:N + 1]
    A.copy_(uniform(1, batch, M, K))
    B.copy_(uniform(2, batch, K, N))
    wide = torch.full((batch, M, N + 3), 7.0, device="cuda")
    anr.gemm(A, B, wide[:, :, 1:N + 1])
    assert_product(wide[:, :, 1:N + 1], A.contiguous(), B.contiguous())
    assert bool((wide[:, :, 0] == 7.0).all()) and bool((wide[:, :, N + 1:] == 7.0).all())


@pytest.mark.parametrize("K", [200, 500, 1500])
@pytest.mark.parametrize("what", ["inf", "nan", "huge", "overflow", "denormal"])
def test_values(K, what):
    from paper_2006_06762_amd import binding as anr
    M, N = 100, 90
    A, B = uniform(3, M, K), uniform(4, K, N)
    if what == "inf":                               # on its own, with the other sign, times zero
        A[M // 2, K - 1] = float("inf")
        B[0, N // 3] = -float("inf")
        B[K - 1, N - 1] = 0.0
    elif what == "nan":
        A[M - 1, 0] = float("nan")
    elif what == "huge":                            # a sum near the largest float keeps its compensation
        A[M // 3], A[M // 3, K // 2] = 1e30, 3.2e38
        B[K // 2] = 1.0
    elif what == "overflow":
        A[1] = 1e20
        B[:, 2] = 1e20
    elif what == "denormal":
        A *= 2.0 ** -130
    C = torch.empty(M, N, device="cuda")
    anr.gemm(A, B, C)
    assert_product(C, A, B)


@pytest.mark.parametrize("K", [256 + 3, 601, 1601, 4001])
def test_error_does_not_grow_with_the_reduction(K):
    """A run adds at most eight instructions of two terms to each of two sums, and those are added once; the result is
    rounded once more: rms 2^-24 / sqrt(3) each, of a part of the sum that grows to the whole only within the run."""
    from paper_2006_06762_amd import binding as anr
    A, B = uniform(5, 96, K), uniform(6, K, 96)
    C = torch.empty(96, 96, device="cuda")
    anr.gemm(A, B, C)
    ref = A.double() @ B.double()
    assert float((C.double() - ref).norm() / ref.norm()) <= 1.1e-7          # sqrt(6.5 / 3) * 2^-24 = 8.8e-8


@pytest.mark.parametrize("batch,M,N,K,steps", [(1, 256, 259, 97, 2), (1, 256, 259, 165, 2), (1, 256, 259, 287, 2), (1, 256, 259, 289, 4),
                                               (1, 256, 259, 513, 4), (1, 256, 259, 801, 8), (1, 256, 259, 861, 8), (1, 256, 259, 865, 8),
                                               (300, 29, 31, 97, 1), (300, 29, 31, 127, 1), (300, 29, 31, 129, 2)])
def test_error_by_the_length_of_a_run(batch, M, N, K, steps):
    """A run adds `steps` instructions of two products to each of two sums: in units of a rounding of the result, the squares
    of these roundings (each of a part of the run's half that grows to the whole) make steps + 1/2 in all, the term that
    enters the compensated sum one, the result itself one, and from K = 864 on, where the two halves are added first,
    that addition one.  A rounding is evenly spread over 2^-24 of a number's power of two, 0.541 of the square of its own
    size on average.  The split GEMM, which took the products of K = 801 and 861 and the many small ones before, is at
    8.3e-8, 8.5e-8 and, for K = 97, 5.0e-8."""
    from paper_2006_06762_amd import binding as anr
    A, B = uniform(7, batch, M, K), uniform(8, batch, K, N)
    C = torch.empty(batch, M, N, device="cuda")
    anr.gemm(A, B, C)
    ref = A.double() @ B.double()
    roundings = steps + 2.5 + (K >= 864)
    assert float((C.double() - ref).norm() / ref.norm()) <= (0.541 * roundings / 3) ** 0.5 * 2.0 ** -24
