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
// matrix, and what an earlier chunk has counted is cleared in A (`counts`); of a K below 32 the only chunk
// starts at zero and rows and columns past K are kept out lane by lane.
constexpr int chunk_k0(int c, int K) { return K < KC ? 0 : smaller(c * KC, K - KC); }
constexpr bool counts(int c, int k, int K) { return k >= c * KC && k < K; }

// Element e (0..7) of half f of a staging unit of A, or of B in the A.B^T form: offset from the chunk's start.
constexpr int unit_k(int at, int f, int e) { return 16 * f + 4 * at + (e < 4 ? e : 4 + e); }

// The row such a unit reads: rows past the end repeat the last one (loaded, never stored).
constexpr int unit_row(int row, int rows) { return smaller(row, rows - 1); }

// Row e (0..3) of half f of a staging piece of k-major B, offset from the chunk's start: the part that differs
// between lanes and the part that rides in the scalar offset.
constexpr int piece_k(int bt, int at) { return 4 * bt + 8 * at; }
constexpr int piece_step(int f, int e) { return 16 * f + e; }

// First of the two columns such a piece reads (N >= 2): pairs past the end repeat the last two columns.  In an
// odd N the last pair is N - 2, N - 1 where the tile's place for it is N - 1, N: the sums of column N - 1 are
// then those of the pair's second column (`second_of_pair`).
constexpr int piece_col(int col, int N) { return smaller(col, N - 2); }
constexpr bool second_of_pair(int col, int N) { return col == N - 1; }

}  // namespace gsplit
}  // namespace anr
