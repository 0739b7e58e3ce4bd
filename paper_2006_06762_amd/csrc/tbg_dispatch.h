// Which kernel takes the scores q.k^T of S queries and keys of D floats, with or without the softmax: the rule of
// launch_tbg, plain arithmetic without a device in it, so that a CPU program can ask it too.
#pragma once
#include <cstdint>

namespace anr {

enum class TbgKernel { rows32, rows_long, tile64, tile, gemm };

struct TbgProblem {
    int64_t S, D, batch;      // batch: heads of all sequences
    bool softmax;
    bool aligned;             // D a multiple of four, rows of q and k whole 16-byte units
    bool offsets32;           // byte offsets inside one (b, h) view of q and of k below 2^31
    bool out_offsets32;       // and of the result
};

constexpr int64_t kTbgMaxKeys = 128;      // of the fused kernel of a single pass
constexpr int64_t kTbgLongKeys = 512, kTbgLongD = 256;

constexpr bool tbs_rows32_takes(const TbgProblem& p) { return p.softmax && p.S <= kTbgMaxKeys && p.D <= 1024 && p.D % 8 == 0; }

// whole tiles, whole chunks and 32-bit byte offsets inside one (b, h) view: the lean form
constexpr bool tbg_whole(const TbgProblem& p) { return p.S % 64 == 0 && p.D % 64 == 0 && p.offsets32 && p.out_offsets32; }

// Enough 128 x 128 tiles to fill the chip twice, mostly full: the bf16-split GEMM (32 x 12 heads of 512 x
// 512 x 128 231 -> 200 us, 16 x 12 of 200 x 200 x 80 36 -> 26).  With fewer or half-empty tiles the other kernels
// are the faster ones (8 x 8 of 312 x 312 x 64 15.0 against 16.5 us), and so they are with a single
// chunk in the lean form (24 x 8 of 256 x 256 x 64 18.4 against 20.6, 48 x 8 of 512 x 512 x 64 129.7 against
// 128.7).  The fused softmax of a single pass keeps its sizes.
constexpr bool tbg_split_takes(const TbgProblem& p)
{
    const int64_t t = (p.S + 127) / 128;
    return p.S > kTbgMaxKeys && p.offsets32 && t * t * p.batch >= 512 && (double)p.S * p.S >= 0.6 * t * t * 128 * 128 &&
           (double)p.S * p.S * p.batch >= 384.0 * 128 * 128 && (p.D >= 48 || p.S % 64 == 0) && !(tbg_whole(p) && p.D <= 64);
}

// What is left with a softmax and up to 512 keys: one kernel that keeps the scores on the chip (16 x 16 heads, two
// kernels / one: 160 x 160 x 64 52 / 28 us, 256 x 256 x 64 74 / 42, 481 x 481 x 32 193 / 131, 512 x 512 x 64 198 /
// 158).  The split GEMM keeps its sizes: its scores are the closer ones, and those tbg gives for them.  A work-group
// walks `walk` floats of every key row of a chunk of 128 in a row, so with few work-groups or a long walk the two
// kernels are faster (8 heads of 300 x 300 x 128 11.4 / 16.9, 24 of 512 x 512 x 256 43.6 / 55.2).  Of 826 shapes of 136 to 512
// keys, 32 to 256 floats and 4 to 128 heads this line costs 0.4 % against the faster of both on average and 17 % at
// most; the next ones to it: 24 heads of 256 x 256 x 104 17.9 / 11.9, 16 of 384 x 384 x 104 21.7 / 16.4, 24 of 384 x 384 x
// 128 23.5 / 24.9, 48 of 320 x 320 x 192 36.4 / 34.4.
constexpr bool tbs_long_takes(const TbgProblem& p)
{
    const int64_t chunks = (p.S + 127) / 128, walk = chunks * p.D, items = p.batch * ((p.S + 31) / 32);
    return p.softmax && p.S > kTbgMaxKeys && p.S <= kTbgLongKeys && p.D <= kTbgLongD && p.D % 8 == 0 && p.offsets32 && !tbg_split_takes(p) &&
           (walk <= 64 || (walk <= 512 && items >= (walk < 320 ? 11 * walk / 20 : 176)));
}

// Softmax, 129 to 512 keys: the kernel on bf16 pieces that keeps 64 rows of scores on the chip (tbs_split_kernel.h),
// in place of whichever of the three above would run.  Lines from 900 shapes of 129 to 512 keys, 16 to 256 floats and
// 8 to 512 heads, new / old time:
//  - split GEMM and softmax kernel: always (0.33 to 0.91; 16 x 8 heads of 484 x 484 x 80 129 / 77 us);
//  - one kernel on fp32 products: its sums of more than 80 floats, or of a number that is no whole step of 16, are
//    the closer ones (error against 64 bits new / old 0.72 at 16 floats, 0.98 at 64, 1.00 at 80, 1.015 at 56, 1.07
//    at 96), so it keeps those.  Up to 64 floats it also keeps few work-groups (to 128 of them 0.92 to 1.09, from 144
//    0.73 to 0.97; to 160 keys a third block of queries and three waves idle: to 288 of them 1.06 to 1.23, 768 0.72 to
//    0.80); longer rows are always faster here (0.59 to 0.98);
//  - two kernels: from 88 work-groups (0.56 to 0.97; 60 to 84 0.78 to 1.31).
constexpr bool tbs_split_takes(const TbgProblem& p)
{
    if (!p.softmax || !p.aligned || !p.offsets32 || p.S <= kTbgMaxKeys || p.S > kTbgLongKeys || p.D > kTbgLongD) return false;
    if (tbg_split_takes(p)) return true;
    const int64_t groups = p.batch * ((p.S + 63) / 64);
    if (!tbs_long_takes(p)) return groups >= 88;
    return p.D % 16 == 0 && p.D <= 80 && (p.D > 64 || groups >= (p.S > 160 ? 144 : 512));
}

constexpr TbgKernel choose_tbg(const TbgProblem& p)
{
    const int64_t tiles = (p.S + 63) / 64;
    if (!p.aligned || tbg_split_takes(p) || p.batch * tiles * tiles >= ((int64_t)1 << 31)) return TbgKernel::gemm;
    if (tbs_rows32_takes(p)) return TbgKernel::rows32;
    if (tbs_long_takes(p)) return TbgKernel::rows_long;
    return tbg_whole(p) ? TbgKernel::tile64 : TbgKernel::tile;
}

}  // namespace anr
