// Which kernel takes C = A.B: the rule of launch_gemm, plain arithmetic without a device in it, so that a CPU program can
// ask it too.
#pragma once
#include <cstdint>

#include "gemm_split_plan.h"

namespace anr {

enum class GemmKernel { ksplit, rows32, pipe, split, plain };

struct GemmProblem {
    int64_t M, N, K, batch;
    bool nk;              // the A.B^T form
    bool one_level;       // no inner batch, no softmax behind it
    bool lines;           // rows of A and B are whole 16-byte units, and so are the steps of the batch
    bool vec;             // of C as well, and all extents multiples of four
    bool offsets32;       // byte offsets inside one matrix below 2^31
};

constexpr int64_t gemm_tiles(const GemmProblem& p, int edge) { return ((p.M + edge - 1) / edge) * ((p.N + edge - 1) / edge) * p.batch; }

// The pipelined fp32 kernel where it is the faster one: a short reduction over few 64 x 64 tiles, so that the
// time is a chain of latencies (splitting adds an LDS round trip to every chunk).  At most one tile per CU:
// 512^2 x 96 5.1 against 7.3 us, 1024^2 x 480 12.8 against 13.9, x 608 15.3 against 16.2 (past 704 four
// wave groups of the split kernel come level, and only they keep up with a longer chain).  Up to three tiles
// per CU and the seven chunks of one wave group: 1536 x 1024 x 160 9.2 against 10.7, 1536^2 x 224 15.3 against
// 16.1; x 256 18.6 against 17.1, and 16 x 512^2 x 128 14.3 against 12.7.  Up to four and two chunks: 2048^2 x 64
// 10.6 against 12.7.  The split kernel starts at one chunk.
constexpr bool gemm_pipe_takes(const GemmProblem& p)
{
    const int64_t tiles = gemm_tiles(p, 64);
    return p.offsets32 && p.vec && !p.nk && (tiles <= 256 ? p.K <= 704 : tiles <= 768 ? p.K <= 7 * 32 : tiles <= 1024 ? p.K <= 64 : p.K < gsplit::KC);
}

// A k-major B is read a whole chunk of rows and a pair of columns at a time.  Operands the pipelined kernel
// cannot load, few tiles and a short reduction: the plain kernel's prologue is the shortest (up to a tile per
// CU K = 32 to 47 0.73 of the split kernel's time, 81 to 96 0.82, 129 to 160 0.94, 161 to 224 1.11; up to two
// 48 to 80 0.89, 81 to 96 0.97, 129 to 160 1.16; three to four tiles per CU 48 to 64 1.13).
constexpr bool gemm_split_takes(const GemmProblem& p)
{
    const int64_t tiles = gemm_tiles(p, 64);
    return p.offsets32 && (p.nk || (p.N >= 2 && p.K >= gsplit::KC)) && p.K > (tiles <= 256 ? 160 : tiles <= 512 ? 96 : 0);
}

// Few 32 x 32 tiles: gemm_rows32_kernel, whatever the alignment.  Up to a tile per CU from K = 65 on (283 x 821 x 83
// 6.9 -> 5.6 us, 449 x 450 x 1920 36 -> 16), or from 97 where the pipelined kernel can load the operands (2560 x 32 x
// 96 5.1 -> 5.5), up to two from 97 (1422 x 200 x 510 14.7 -> 12.5, 192 x 2464 x 320 10.1 -> 10.0); past that each CU has
// more work than its own chain and larger tiles reuse more (520 tiles, K = 384, 11.6 -> 13.3).  Where the pipelined kernel
// could load them, products of 257 to 512 tiles are level at K = 100 to 128, slower up to 288 (3 x 120 x 784 x 144 6.7 ->
// 8.4, 624 x 672 x 228 8.6 -> 9.5) and faster from 330 on (1861 x 160 x 452 12.9 -> 11.4): they stay here for their sums, 5.2e-8
// of the exact results where the pipelined kernel's are 1.8e-7 (K = 97) to 3.4e-7 (704).
constexpr bool gemm_rows32_takes(const GemmProblem& p)
{
    const int64_t tiles = gemm_tiles(p, 32);
    return p.offsets32 && !p.nk && p.one_level && tiles <= 512 && p.K > (tiles <= 256 && !p.vec ? 64 : 96);
}

// Of these the fewest, by 16 x 16 tiles (gemm_rows16_kernel): to 64 tiles of 32 x 32 every CU has at most one of 16 x 16.
// Of 400 products of 1 to 256 tiles, new / old time: to 64 tiles 0.47 to 0.90 (64 x 64 x 2720 19.9 / 10.0 us, 200 x 130 x 300
// 6.3 / 4.6), 65 to 128 0.61 to 1.13, then 0.75 to 1.34, past 192 1.12 to 1.76: the matrix cores of all CUs are busy then, and larger
// tiles read less.
constexpr bool gemm_rows16_takes(const GemmProblem& p) { return gemm_rows32_takes(p) && gemm_tiles(p, 32) <= 64; }

constexpr GemmKernel choose_gemm(const GemmProblem& p)
{
    // few whole tiles and a reduction of 128, 256 or 512: one 32x32 tile per work-group, K split over its waves
    if (!p.nk && p.one_level && p.lines && p.M % 32 == 0 && p.N % 32 == 0 && gemm_tiles(p, 32) <= 1024 && (p.K == 128 || p.K == 256 || p.K == 512))
        return GemmKernel::ksplit;
    if (gemm_rows32_takes(p)) return GemmKernel::rows32;
    if (gemm_pipe_takes(p)) return GemmKernel::pipe;
    return gemm_split_takes(p) ? GemmKernel::split : GemmKernel::plain;
}

}  // namespace anr
