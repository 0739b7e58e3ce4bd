// Walks what every thread of a work-group of the bf16-split GEMM loads, tile by tile and chunk by chunk, with
// the arithmetic the kernel itself uses, and multiplies what it stages.  Prints one line and exits non-zero if
// a load touches an element outside its matrix, the products are not those of whole numbers, or something that is
// not counted is multiplied.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "gemm_split_plan.h"

using namespace anr::gsplit;

static long outside = 0;

// Element i of a matrix: zero where the lane's part of the offset alone is past the extent (which the hardware
// guarantees), counted where it is not and the whole offset is.
static int load(const std::vector<int>& m, int64_t lane, int64_t scalar)
{
    if (lane >= (int64_t)m.size()) return 0;
    if (lane < 0 || lane + scalar >= (int64_t)m.size()) {
        ++outside;
        return 0;
    }
    return m[lane + scalar];
}

int main(int argc, char** argv)
{
    if (argc != 8) return 2;
    const int tile = atoi(argv[1]), groups = atoi(argv[2]), M = atoi(argv[3]), N = atoi(argv[4]), K = atoi(argv[5]);
    const int pad = atoi(argv[6]);
    const bool nt = atoi(argv[7]) != 0;
    const int lda = K + pad, ldb = (nt ? K : N) + pad;
    std::vector<int> A((size_t)(M - 1) * lda + K, 1000003), B(nt ? (size_t)(N - 1) * ldb + K : (size_t)(K - 1) * ldb + N, 1000003);
    for (int i = 0; i < M; ++i)
        for (int k = 0; k < K; ++k) A[(size_t)i * lda + k] = (i * 31 + k * 17) % 23 - 11;
    for (int j = 0; j < N; ++j)
        for (int k = 0; k < K; ++k) B[nt ? (size_t)j * ldb + k : (size_t)k * ldb + j] = (j * 13 + k * 7) % 19 - 9;

    const int nchunks = (K + KC - 1) / KC, iters = (nchunks + groups - 1) / groups;
    long wrong = 0, kept = 0;
    std::vector<int> sa((size_t)tile * KC), sb((size_t)tile * KC);          // [row or column position][k of a chunk]
    std::vector<long> acc((size_t)tile * tile);
    for (int m0 = 0; m0 < M; m0 += tile)
        for (int n0 = 0; n0 < N; n0 += tile) {
            for (auto& v : acc) v = 0;
            for (int g = 0; g < groups; ++g)
                for (int i = 0; i <= iters + 1; ++i) {                        // two chunks of look-ahead past the last
                    const int c = g + i * groups, k0 = chunk_k0(c, K);
                    for (int tid = 0; tid < 2 * tile; ++tid) {
                        const int at = tid & 1, row = tid >> 1, bt = row / (tile / 2), pair = row % (tile / 2);
                        for (int f = 0; f < 2; ++f) {
                            for (int e = 0; e < 8; ++e) {
                                const int64_t past = c < nchunks ? 0 : (int64_t)1 << 40;
                                // the offset inside a chunk belongs to the lane
                                const int off = unit_k(at, f, e);
                                const bool in = c * KC + KC <= K || counts(c, k0 + off, K);
                                int v = load(A, (int64_t)unit_row(m0 + row, M) * lda + off + past, k0);
                                sa[(size_t)row * KC + off] = in ? v : 0;
                                if (nt) {
                                    v = load(B, (int64_t)unit_row(n0 + row, N) * ldb + off + past, k0);
                                    sb[(size_t)row * KC + off] = in ? v : 0;
                                }
                            }
                            for (int e = 0; !nt && e < 4; ++e)
                                for (int b = 0; b < 2; ++b) {
                                    const int64_t lane = (int64_t)piece_k(bt, at) * ldb + piece_col(n0 + 2 * pair, N) + b;
                                    const int step = k0 + piece_step(f, e);
                                    const int v = load(B, lane + (c < nchunks ? 0 : (int64_t)1 << 40), (int64_t)step * ldb);
                                    const int off = piece_k(bt, at) + piece_step(f, e);
                                    const bool in = c * KC + KC <= K || counts(c, k0 + off, K);
                                    sb[(size_t)(2 * pair + b) * KC + off] = in ? v : 0;
                                }
                        }
                    }
                    // as the try with the fp32 instruction stages it, whatever is not counted is zero on both sides: one of
                    // them may hold an infinity
                    for (int r = 0; r < tile; ++r)
                        for (int k = 0; k < KC; ++k)
                            if (c < nchunks && !counts(c, k0 + k, K)) kept += (sa[(size_t)r * KC + k] != 0) + (sb[(size_t)r * KC + k] != 0);
                    for (int r = 0; r < tile; ++r)
                        for (int j = 0; j < tile; ++j)
                            for (int k = 0; k < KC; ++k) acc[(size_t)r * tile + j] += (long)sa[(size_t)r * KC + k] * sb[(size_t)j * KC + k];
                }
            for (int r = m0; r < M && r < m0 + tile; ++r)
                for (int j = n0; j < N && j < n0 + tile; ++j) {
                    long want = 0;
                    for (int k = 0; k < K; ++k) want += (long)A[(size_t)r * lda + k] * B[nt ? (size_t)j * ldb + k : (size_t)k * ldb + j];
                    // a lane holds the sums of a pair of columns
                    const int even = j - (j - n0) % 2;
                    const int held = nt || j != even ? j : even + second_of_pair(even, N);
                    wrong += acc[(size_t)(r - m0) * tile + (held - n0)] != want;
                }
        }
    printf("%ld outside, %ld wrong, %ld kept\n", outside, wrong, kept);
    return outside != 0 || wrong != 0 || kept != 0;
}
