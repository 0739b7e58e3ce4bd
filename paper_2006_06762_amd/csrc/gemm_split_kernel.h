// GMM (C = A.B, Sec. 4.1 and Appendix C of arXiv 2006.06762) on the bf16 matrix pipes, each fp32
// operand split into three bf16 pieces (split_bf16.h): any M, N, K, any alignment.
//
// Work-group tile BM x BN, WM x WN waves of MB x 2 blocks of 32 x 32, NWG such groups of waves that
// share the chunks of the reduction.  Operands travel global -> registers -> (split) -> LDS, so a float
// is split once per work-group and not once per wave that reads it.  The LDS image is in operand order:
// plane (h, m, l), then unit of eight k, then row, 16 bytes each: a wave's operand read is 32 consecutive
// 16-byte pieces per half (no bank conflict).  A half chunk of 16 k has two units; unit t holds k = 4t ..
// 4t+3 and 8+4t .. 8+4t+3, so that the two lanes that stage a row read 32 contiguous bytes at a time (any
// order of k is a valid reduction order as long as both operands use it).  Units are 64 bytes further
// apart than their rows need: those two lanes then write to different banks.
//
// SPEC, for products with about one tile of 128 x 128 per CU: four waves only load, split and store, four only multiply,
// and a chunk has a buffer to itself, so there is one barrier per 32 k.  Vector-ALU and matrix instructions of
// different waves run side by side (probe: 256 us of matrix instructions with 232 us of splitting in the other waves take
// 306), and a work-group alone on its CU has no second one whose products cover its splitting.  Two groups that
// took turns at both, each with a barrier per 16 k, against it: 512^3 x16 37.2 -> 31.8 us, 512 x 512 x 2048 x16 122 -> 106,
// 2048^3 119 -> 104, 2038 x 1861 x 473 33.9 -> 28.4.  With several tiles per CU two work-groups of the other form cover
// each other (4096^2 x 512 109 against 116).  Two chunks of loads in flight: 3 to 8 % slower.
//
// B is k-major in memory.  A staging piece is four k of two neighbouring columns: 8-byte loads (the
// address unit takes a load instruction's 64 lanes in 16 cycles whatever their width, and 4-byte loads
// cost a quarter of the time of a work-group alone on its CU), and packing pairs of k transposes for
// free.  Column 2p + b sits at position b*BN/2 + p, so that a lane's two accumulator blocks are
// neighbouring columns of C.  Which rows, columns and k a thread reads at the edges: gemm_split_plan.h.
//
// Bound: large products by the matrix pipes' power (eight bf16 products per fp32 one at 181 TFLOP/s are
// 1.45 PFLOP/s, what a large bf16 product of the library reaches on the card is 1.3); work-groups alone on their
// CU by the chain load - split - LDS - multiply.  Measured against the fp32 kernels this one took over from:
// 4096^3 976 -> 765-889 us (by card), 2048^3 133 -> 104, 1024^3 x16 257 -> 204, 512^3 x16 38.6 -> 31.8,
// 1009 x 1531 x 771 x3 (4-byte aligned rows) 167 -> 70, 1024^3 22.7 -> 22.4.  Tried and dropped: the split
// between the matrix instructions, v_dot2 for its subtractions, wave groups in opposite order (all slower);
// 256 x 256 tiles, which leave no registers for the second set of sums (six products in one set, 4096^3 in
// 600 us, but up to five full-size roundings where a single non-zero term needs one).
#pragma once
#include <type_traits>

#include "anr_kernels.h"
#include "gemm_split_plan.h"
#include "split_bf16.h"

namespace anr {
namespace gsplit {

template <int ROWS>
struct Plane {
    static constexpr int UNIT = ROWS * 16 + 64;      // bytes between units of eight k
    static constexpr int BYTES = 2 * UNIT;
};

// SPEC: whole chunks in two buffers, four halves, for one group of waves that multiplies.
template <int BM, int BN, int NWG, bool SPEC>
constexpr size_t lds_bytes()
{
    return (SPEC ? 2 : NWG) * 2 * 3 * (size_t)(Plane<BM>::BYTES + Plane<BN>::BYTES) + 16;      // and flags
}

// Chunk-invariant description of a launch (what the host works out once).
struct Grid {
    int tiles_m, tiles_n;
    int group_m;          // tiles are walked in bands of group_m rows of tiles
};

// One tile of a work-group: as bf16 pieces, or PLAIN, with the fp32 instruction.  False if it met a value that the
// pieces cannot carry: then nothing is stored.
template <int BM, int BN, int WM, int WN, int NWG, bool SPEC, bool NT, bool FUSED, bool PLAIN>
__device__ __forceinline__ bool compute_tile(const GemmArgs& p, const Grid& g, const int thread)
{
    constexpr int T = 64 * WM * WN;                  // threads of a wave group
    constexpr int MB = BM / (32 * WM);
    static_assert(BN == 64 * WN && BM == BN && T == 2 * BM,
                  "two blocks of columns per wave; per half chunk every thread stages one unit of A and one piece of B");
    constexpr int PA = Plane<BM>::BYTES, PB = Plane<BN>::BYTES;
    constexpr int BUF = 3 * (PA + PB);
    constexpr int RED = BM * BN * 4;                 // a group's accumulators
    static_assert(BM <= T, "a thread per row");
    static_assert(NWG == 1 || (NWG - 1) * RED <= NWG * 2 * BUF, "the groups' sums meet in the staging buffers");

    extern __shared__ __attribute__((aligned(16))) char slds[];

    static_assert(!SPEC || NWG == 1, "one group multiplies, the other one stages");
    const int wgrp = NWG > 1 ? __builtin_amdgcn_readfirstlane(thread / T) : 0;
    const bool stager = SPEC && __builtin_amdgcn_readfirstlane(thread / T) != 0;
    char* const region = slds + wgrp * 2 * BUF;
    int* const flag = reinterpret_cast<int*>(slds + (SPEC ? 2 : NWG) * 2 * BUF);     // a value was met that the pieces cannot carry
    const int tid = thread % T;
    const int lane = tid & 63, wave = tid >> 6;
    const int r32 = lane & 31, h = lane >> 5;
    const int wm = wave / WN, wn = wave % WN;

    // Work-group ids are dealt round-robin over the 8 XCDs, each with its own L2: every XCD gets a
    // contiguous run of the batch's tiles, each matrix walked in bands of group_m tile rows, column by
    // column (512^3 x16: whole matrices stay on one XCD)
    const int tiles = g.tiles_m * g.tiles_n;
    int id = blockIdx.x;
    {
        const int all = (int)gridDim.x, per = all >> 3, rest = all & 7, xcd = id & 7, slot = id >> 3;
        id = xcd * per + (xcd < rest ? xcd : rest) + slot;
    }
    const int mat = id / tiles;
    id -= mat * tiles;
    const int band = id / (g.group_m * g.tiles_n);
    const int band_rows = min(g.group_m, g.tiles_m - band * g.group_m);
    const int in_band = id - band * g.group_m * g.tiles_n;
    const int tile_m = band * g.group_m + in_band % band_rows, tile_n = in_band / band_rows;
    const int m0 = tile_m * BM, n0 = tile_n * BN;

    const int zo = mat / p.batch_inner, zi = mat - zo * p.batch_inner;
    const float* A = p.A + zo * p.sAo + zi * p.sAi;
    const float* B = p.B + zo * p.sBo + zi * p.sBi;
    float* __restrict__ C = p.C + zo * p.sCo + zi * p.sCi;
    const int M = p.M, N = p.N, K = p.K;

    const uint32_t a_bytes = 4u * (uint32_t)((int64_t)(M - 1) * p.lda + K);
    const uint32_t b_bytes = NT ? 4u * (uint32_t)((int64_t)(N - 1) * p.ldb + K) : 4u * (uint32_t)((int64_t)(K - 1) * p.ldb + N);
    const __amdgpu_buffer_rsrc_t arsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(A), 0, (int)a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t brsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(B), 0, (int)b_bytes, 0x00020000);

    // Staging of A: row tid/2, unit tid%2.  Of B: four k 4t + 8 (tid%2) .. +3 of the column pair
    // (tid/2) % (BN/2), unit t = (tid/2) / (BN/2); of the k-contiguous B of the A.B^T form like A.
    const int at = tid & 1, arow = tid >> 1;
    const int bt = arow / (BN / 2), bpair = arow % (BN / 2);
    const uint32_t aoff = 4u * (uint32_t)((int64_t)unit_row(m0 + arow, M) * p.lda + unit_k(at, 0, 0));
    const uint32_t boff = NT ? 4u * (uint32_t)((int64_t)unit_row(n0 + arow, N) * p.ldb + unit_k(at, 0, 0))
                             : 4u * (uint32_t)((int64_t)piece_k(bt, at) * p.ldb + piece_col(n0 + 2 * bpair, N));

    float ra[2][8], rb[2][8];                        // rb: four k of the first column, then of the second (NT: as ra)
    const uint32_t ldb4 = 4u * (uint32_t)p.ldb;
    auto load_unit = [&](__amdgpu_buffer_rsrc_t rsrc, uint32_t off, int k0, int f, float (&r)[8]) {
        const f32x4 lo = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off + 64 * f, 4 * k0, 0));
        const f32x4 hi = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off + 64 * f + 32, 4 * k0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) { r[e] = lo[e]; r[4 + e] = hi[e]; }
    };
    // Chunks past the last one read zeros: their offset is out of range (a branch around the loads would make
    // the compiler wait for them where it ends)
    const int nchunks = (K + KC - 1) / KC;
    auto load_a = [&](int c, auto f_c) {             // half f of chunk c
        constexpr int f = decltype(f_c)::value;
        const uint32_t past = c < nchunks ? 0u : kOutOfRange;
        load_unit(arsrc, aoff | past, chunk_k0(c, K), f, ra[f]);
    };
    auto load_b = [&](int c, auto f_c) {
        constexpr int f = decltype(f_c)::value;
        const uint32_t past = c < nchunks ? 0u : kOutOfRange;
        const int k0 = chunk_k0(c, K);
        if (NT) {
            load_unit(brsrc, boff | past, k0, f, rb[f]);
            return;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // the row's part of the offset is uniform and rides in the load's scalar offset
            const f32x2 v = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(brsrc, (int)(boff | past), (int)((uint32_t)(k0 + piece_step(f, e)) * ldb4), 0));
            rb[f][e] = v[0];
            rb[f][4 + e] = v[1];
        }
    };
    // Half f goes to buffer f: eight pairs of floats are split (0-3: the unit of A, 4-5 and 6-7: the
    // columns of B) and written as soon as a 16- or 8-byte store is complete.
    uint32_t lost = 0;
    uint32_t sp[3][8];
    char* const wa = region + at * Plane<BM>::UNIT + arow * 16;
    char* const wb = region + 3 * PA + (NT ? at * Plane<BN>::UNIT + ((arow & 1) * (BN / 2) + (arow >> 1)) * 16
                                           : bt * Plane<BN>::UNIT + bpair * 16 + 8 * at);
    // k that an earlier chunk has counted and, of a K below 32, k past the end (in B's rows too: they run on into
    // the next one).  Zeros in A leave the NaN of an infinity in B, which ends the first try; the second one has zeros in
    // both (in the first they cost the 64-wide tiles a sixth: 1009 x 1531 x 771 x3 74.5 against 87.4 us)
    auto clear_uncounted = [&](auto f_c, int c) {
        constexpr int f = decltype(f_c)::value;
        const int k0 = chunk_k0(c, K);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const bool in = counts(c, k0 + unit_k(at, f, e), K);
            ra[f][e] = in ? ra[f][e] : 0.f;
            if (NT) rb[f][e] = in ? rb[f][e] : 0.f;
        }
        if (PLAIN && !NT) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool in = counts(c, k0 + piece_k(bt, at) + piece_step(f, e), K);
                rb[f][e] = in ? rb[f][e] : 0.f;
                rb[f][4 + e] = in ? rb[f][4 + e] : 0.f;
            }
        }
    };
    int at_buf = 0;                                  // SPEC: the chunk's buffer, bytes
    auto split_pair = [&](auto f_c, int i) {
        constexpr int f = decltype(f_c)::value;
        if (i < 4) split2(ra[f][2 * i], ra[f][2 * i + 1], sp[0][i], sp[1][i], sp[2][i], lost);
        else split2(rb[f][2 * (i - 4)], rb[f][2 * (i - 4) + 1], sp[0][i], sp[1][i], sp[2][i], lost);
        if (i == 3) {
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(wa + at_buf + f * BUF + q * PA) = u32x4{sp[q][0], sp[q][1], sp[q][2], sp[q][3]};
        }
        if (NT && i == 7) {
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(wb + at_buf + f * BUF + q * PB) = u32x4{sp[q][4], sp[q][5], sp[q][6], sp[q][7]};
        }
        if (!NT && (i == 5 || i == 7)) {
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x2*>(wb + at_buf + f * BUF + q * PB + (i == 7 ? BN * 8 : 0)) = u32x2{sp[q][i - 1], sp[q][i]};
        }
    };
    // For the fp32 instruction the half goes as it is: units of four k, 16 bytes a row
    constexpr int QA = BM * 16 + 64, QB = BN * 16 + 64;
    static_assert(4 * QA <= 3 * PA && 4 * QB <= 3 * PB, "fits the room of the pieces");
    char* const fa = region + at * QA + arow * 16;
    char* const fb = region + 3 * PA + (NT ? at * QB + ((arow & 1) * (BN / 2) + (arow >> 1)) * 16 : (bt + 2 * at) * QB + bpair * 16);
    auto store_half = [&](auto f_c, int c) {         // half f of chunk c
        constexpr int f = decltype(f_c)::value;
        if (c * KC + KC > K) clear_uncounted(f_c, c);
        if constexpr (PLAIN) {
            const float* const x = ra[f];
            const float* const y = rb[f];
            *reinterpret_cast<f32x4*>(fa + at_buf + f * BUF) = f32x4{x[0], x[1], x[2], x[3]};
            *reinterpret_cast<f32x4*>(fa + at_buf + f * BUF + 2 * QA) = f32x4{x[4], x[5], x[6], x[7]};
            *reinterpret_cast<f32x4*>(fb + at_buf + f * BUF) = f32x4{y[0], y[1], y[2], y[3]};
            *reinterpret_cast<f32x4*>(fb + at_buf + f * BUF + (NT ? 2 * QB : BN * 8)) = f32x4{y[4], y[5], y[6], y[7]};
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) split_pair(f_c, i);
        }
    };

    // the products of the first pieces (or of the floats themselves), with SPEC a sum for each half of the chunks as two
    // groups would have, and the other seven
    constexpr int SUMS = SPEC ? 2 : 1;
    f32x16 sums_of[SUMS][MB][2], low[MB][2];
    f32x16 (&acc)[MB][2] = sums_of[0];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                low[mb][nb][r] = 0.f;
#pragma unroll
                for (int i = 0; i < SUMS; ++i) sums_of[i][mb][nb][r] = 0.f;
            }

    auto multiply = [&](auto f_c) {
        constexpr int f = decltype(f_c)::value;
        if constexpr (PLAIN) {
            // the wave's half h takes the units 2q + h, element by element
            const char* a = region + at_buf + f * BUF + h * QA + (wm * MB * 32 + r32) * 16;
            const char* b = region + at_buf + f * BUF + 3 * PA + h * QB + (wn * 32 + r32) * 16;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                f32x4 av[MB], bv[2];
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) av[mb] = *reinterpret_cast<const f32x4*>(a + 2 * q * QA + mb * 512);
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) bv[nb] = *reinterpret_cast<const f32x4*>(b + 2 * q * QB + nb * BN * 8);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                        for (int nb = 0; nb < 2; ++nb) sums_of[f % SUMS][mb][nb] = mfma32(av[mb][e], bv[nb][e], sums_of[f % SUMS][mb][nb]);
            }
        } else {
            const char* a = region + at_buf + f * BUF + h * Plane<BM>::UNIT + (wm * MB * 32 + r32) * 16;
            const char* b = region + at_buf + f * BUF + 3 * PA + h * Plane<BN>::UNIT + (wn * 32 + r32) * 16;
            u32x4 bv[3][2];
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) bv[q][nb] = *reinterpret_cast<const u32x4*>(b + q * PB + nb * BN * 8);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                u32x4 av[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) av[q] = *reinterpret_cast<const u32x4*>(a + q * PA + mb * 512);
#pragma unroll
                for (int t = 0; t < kProducts; ++t)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) {
                        f32x16& sum = t < kProducts - 1 ? low[mb][nb] : sums_of[f % SUMS][mb][nb];
                        sum = mfma_bf16(av[kPieceA[t]], bv[kPieceB[t]][nb], sum);
                    }
            }
        }
    };

    // Half f of every chunk goes through buffer f: between two barriers one buffer is multiplied, the other filled
    // with the loaded half of the next chunk and that half's loads of the chunk after it sent.  Group w takes every
    // NWG-th chunk.
    using F0 = std::integral_constant<int, 0>;
    using F1 = std::integral_constant<int, 1>;
    auto half = [&](auto f_c, int c_fill, int c_load) {
        using G = std::integral_constant<int, decltype(f_c)::value ^ 1>;
        multiply(f_c);
        store_half(G{}, c_fill);
        load_a(c_load, G{});
        load_b(c_load, G{});
    };
    if constexpr (SPEC) {
        // Barrier c: chunk c is staged and chunk c - 1 multiplied.  A value that the pieces cannot carry is noted before it,
        // in the chunk's flag, and every wave leaves before the next one.
        if (stager) {
            load_a(0, F0{});
            load_b(0, F0{});
            load_a(0, F1{});
            load_b(0, F1{});
        } else if (!PLAIN && thread == 0) {
            flag[0] = flag[1] = 0;
        }
        if (!PLAIN) __syncthreads();
        if (stager) {
#pragma unroll 1
            for (int c = 0, stop = 0; c < nchunks; ++c) {
                at_buf = (c & 1) * 2 * BUF;
                store_half(F0{}, c);
                load_a(c + 1, F0{});
                load_b(c + 1, F0{});
                store_half(F1{}, c);
                load_a(c + 1, F1{});
                load_b(c + 1, F1{});
                __builtin_amdgcn_sched_barrier(0);
                if (!PLAIN) {
                    if (__builtin_amdgcn_readfirstlane(stop)) break;
                    if (lost_bits(lost)) flag[c & 1] = 1;
                }
                __syncthreads();
                if (!PLAIN) stop = flag[c & 1];
            }
        } else {
#pragma unroll 1
            for (int c = 0, stop = 0; c < nchunks; ++c) {
                if (!PLAIN && __builtin_amdgcn_readfirstlane(stop)) break;
                __syncthreads();
                at_buf = (c & 1) * 2 * BUF;
                if (!PLAIN) stop = flag[c & 1];
                multiply(F0{});
                multiply(F1{});
            }
        }
    } else {
        if (!PLAIN && thread == 0) *flag = 0;
        load_a(wgrp, F0{});
        load_b(wgrp, F0{});
        load_a(wgrp, F1{});
        load_b(wgrp, F1{});
        store_half(F0{}, wgrp);
        load_a(wgrp + NWG, F0{});
        load_b(wgrp + NWG, F0{});
        int end = (nchunks + NWG - 1) / NWG * NWG;       // the barriers are the work-group's
#pragma unroll 1
        for (int c = wgrp; c < end; c += NWG) {
            __syncthreads();
            // set between the barriers of a round and read behind the second, so every wave reads the same
            if (!PLAIN && lost_bits(lost)) *flag = 1;
            half(F0{}, c, c + NWG);
            __syncthreads();
            const int stop = PLAIN ? 0 : *flag;
            half(F1{}, c + NWG, c + 2 * NWG);
            if (!PLAIN && __builtin_amdgcn_readfirstlane(stop)) end = 0;
        }
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (!PLAIN) acc[mb][nb][r] += low[mb][nb][r];
                if (SPEC) acc[mb][nb][r] += sums_of[SUMS - 1][mb][nb][r];
            }
    if (NWG > 1) {
        // every staging buffer is free: groups 1 .. NWG-1 leave their accumulators there, group 0 adds
        // them in group order
        __syncthreads();
        if (wgrp > 0) {
            float* red = reinterpret_cast<float*>(slds + (wgrp - 1) * RED) + wave * (MB * 2 * 16 * 64) + lane;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) red[((mb * 2 + nb) * 16 + r) * 64] = acc[mb][nb][r];
        }
        __syncthreads();
        if (wgrp == 0) {
#pragma unroll
            for (int o = 1; o < NWG; ++o) {
                const float* red = reinterpret_cast<const float*>(slds + (o - 1) * RED) + wave * (MB * 2 * 16 * 64) + lane;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[mb][nb][r] += red[((mb * 2 + nb) * 16 + r) * 64];
            }
        }
    }

    if (!PLAIN) {
        SumCheck sums;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) sums.check(acc[mb][nb]);
        if (__syncthreads_or(lost_bits(lost) || sums.refused())) return false;
    }
    // scale and shift of the tile's rows
    float* const row_scale = reinterpret_cast<float*>(slds);
    if (FUSED) {
        __syncthreads();                             // the staging buffers are free
        if (thread < BM) {
            const int row = min(m0 + thread, M - 1);
            const float scale = p.scale_shift ? p.scale_shift[row] : p.gamma[row] / sqrtf(p.var[row] + p.eps);
            row_scale[thread] = scale;
            row_scale[BM + thread] = p.scale_shift ? p.scale_shift[M + row] : p.beta[row] - p.mean[row] * scale;
        }
        __syncthreads();
    }
    if (stager || (NWG > 1 && wgrp > 0)) return true;

    // accumulator register r of lane (h, r32): row 8*(r/4) + 4*h + r%4 of block mb, columns 2*(wn*32 + r32) + nb:
    // 32 lanes write 256 contiguous bytes of a row, and C is not read again (non-temporal)
    auto store_tile = [&](auto whole_c) {
        constexpr bool whole = decltype(whole_c)::value;
        typedef float pair __attribute__((ext_vector_type(2), aligned(4)));
        const int col = n0 + 2 * (wn * 32 + r32);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int row0 = m0 + (wm * MB + mb) * 32 + 4 * h;
            float* const c = C + (int64_t)row0 * p.ldc + col;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int dr = 8 * (r / 4) + (r % 4);
                float* const d = c + (int64_t)dr * p.ldc;
                pair v = {acc[mb][0][r], acc[mb][1][r]};
                if (FUSED) {
                    const float scale = row_scale[row0 - m0 + dr], shift = row_scale[BM + row0 - m0 + dr];
                    v[0] = fmaxf(fmaf(v[0], scale, shift), 0.f);
                    v[1] = fmaxf(fmaf(v[1], scale, shift), 0.f);
                }
                if (whole || (row0 + dr < M && col + 1 < N)) __builtin_nontemporal_store(v, reinterpret_cast<pair*>(d));
                else if (row0 + dr < M && col < N) *d = v[!NT && second_of_pair(col, N)];
            }
        }
    };
    if (m0 + BM <= M && n0 + BN <= N) store_tile(std::true_type{});
    else store_tile(std::false_type{});
    return true;
}

// Values the pieces cannot carry: the tile again with the fp32 instruction, staged the same way.  A lost low piece
// ends the first try a chunk or two after it is met, so a product full of them takes little more than the fp32
// kernels did (4096^3, probabilities of a steep softmax: 1050 to 1080 us against 1003); infinities, NaN and a last
// chunk's lost pieces cost both tries (1870).  Operand by operand, without staging, it was 5020.  The flag costs an
// ordinary product 1.4 % (set at the end of a round instead, where it cuts the schedule in two, 6 %).
// FUSED: batch norm and ReLU per row of C (a pointwise convolution's).  Forms of their own: asked of every product, they
// cost short reductions 3 to 5 % (3 x 1312 x 384 x 151 11.1 -> 11.7 us, 192 heads of 249 x 249 x 80 67.9 -> 70.7).
template <int BM, int BN, int WM, int WN, int NWG, bool SPEC, int MINW, bool NT, bool FUSED>
__global__ __launch_bounds__(64 * WM * WN * (SPEC ? 2 : NWG), MINW) void gemm_split_kernel(const GemmArgs p, const Grid g)
{
    int thread = threadIdx.x;
    if (compute_tile<BM, BN, WM, WN, NWG, SPEC, NT, FUSED, false>(p, g, thread)) return;
    asm("" : "+v"(thread));                          // nothing of the second try is held through the first
    compute_tile<BM, BN, WM, WN, NWG, SPEC, NT, FUSED, true>(p, g, thread);
}

}  // namespace gsplit
}  // namespace anr
