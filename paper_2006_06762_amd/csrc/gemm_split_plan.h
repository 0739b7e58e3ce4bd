// What gemm_split_kernel.h stages where: plain arithmetic without a device in it, so that a CPU program can
// walk every thread's loads.  No load may lean on the range check with its scalar offset: the lane's part of an
// offset alone decides what is past the extent, and every other load lies inside its matrix.
#pragma once
#include <cstdint>

namespace anr {
namespace gsplit {

constexpr int KC = 32;                               // k of a global load round; LDS buffers hold half of it
constexpr uint32_t kOutOfRange = 0x80000000u;        // byte offset beyond any descriptor extent

constexpr int smaller(int a, int b) { return a < b ? a : b; }

// First k that chunk c loads.  The last chunk of a K that is no multiple of 32 starts at K - 32, inside the
// matrix, and what an earlier chunk has counted is cleared in A (`counts`), in the A.B^T form and in the fp32
// instruction's try in B too.  A K below 32 comes in the A.B^T form only: the chunk starts at zero, and what its rows
// read past K is cleared in both operands.
constexpr int chunk_k0(int c, int K) { return K < KC ? 0 : smaller(c * KC, K - KC); }
constexpr bool counts(int c, int k, int K) { return k >= c * KC && k < K; }

// Element e (0..7) of half f of a staging unit of A, or of B in the A.B^T form: offset from the chunk's start.
constexpr int unit_k(int at, int f, int e) { return 16 * f + 4 * at + (e < 4 ? e : 4 + e); }

// The row such a unit reads: rows past the end repeat the last one (loaded, never stored).
constexpr int unit_row(int row, int rows) { return smaller(row, rows - 1); }

// Row e (0..3) of half f of a staging piece of k-major B (K >= 32), offset from the chunk's start: the part that differs
// between lanes and the part that rides in the scalar offset.
constexpr int piece_k(int bt, int at) { return 4 * bt + 8 * at; }
constexpr int piece_step(int f, int e) { return 16 * f + e; }

// First of the two columns such a piece reads (N >= 2): pairs past the end repeat the last two columns.  In an
// odd N the last pair is N - 2, N - 1 where the tile's place for it is N - 1, N: the sums of column N - 1 are
// then those of the pair's second column (`second_of_pair`).
constexpr int piece_col(int col, int N) { return smaller(col, N - 2); }
constexpr bool second_of_pair(int col, int N) { return col == N - 1; }

// Tile and wave groups: the variant with the shortest estimated time.  `base` is the launch, `round` the time in
// which each group of a work-group alone on its CU gets one 32-wide chunk done (load latency, staging, two
// barriers), `busy` a CU's time per chunk and work-group once several fill it, `ends` its time for a work-group's
// first loads and stores.  Large tiles read fewer operand bytes per FLOP, small ones spread a small product over
// more CUs, and wave groups shorten the chain of chunks where there are not enough tiles even so.  The figures
// are those that chose best among all five variants timed on 550 products of 32 to 4096 (0.2 % slower than the
// best one on average, 12 % at most), near a least-squares fit of the estimate itself.
// 128 with two groups is the form whose second group of waves stages what the first one multiplies.
struct Variant {
    int tile, groups;
    double base, round, busy, ends;      // us
};
constexpr Variant kVariants[] = {{128, 1, 5.5, 2.64, 1.49, 1.36}, {128, 2, 3.8, 1.56, 1.555, 3.2}, {64, 1, 4.9, 1.88, 0.46, 0.42},
                                 {64, 2, 6.3, 1.48, 0.44, 0.94}, {64, 4, 2.4, 1.79, 0.44, 6.24}};
constexpr int kVariantCount = sizeof(kVariants) / sizeof(kVariants[0]);

constexpr double estimate_us(const Variant& t, int64_t M, int64_t N, int64_t K, int64_t batch)
{
    const int64_t chunks = (K + KC - 1) / KC;
    const int64_t tiles = ((M + t.tile - 1) / t.tile) * ((N + t.tile - 1) / t.tile) * batch;
    const double chain = (double)((chunks + t.groups - 1) / t.groups) * t.round;
    const double work = (double)((tiles + 255) / 256) * ((double)chunks * t.busy + t.ends);
    return t.base + (work > chain ? work : chain);
}

constexpr int choose_variant(int64_t M, int64_t N, int64_t K, int64_t batch)
{
    int best = 0;
    for (int v = 1; v < kVariantCount; ++v)
        if (estimate_us(kVariants[v], M, N, K, batch) < estimate_us(kVariants[best], M, N, K, batch)) best = v;
    return best;
}

}  // namespace gsplit
}  // namespace anr
