// Full TBS for 128 < S <= 512 on the bf16 matrix pipes, each fp32 operand split into three bf16 pieces (split_bf16.h):
// scores, softmax and probabilities in one launch, so that the scores never go to memory.
//
// Work-group = 64 queries x all keys of one (b, h), a wave for 32 keys: 8, 12 or 16 of them (two blocks of keys to a wave
// cost 241 registers and left a SIMD two waves: 16 x 16 heads of 384 x 384 x 64 88 us against 80 with twelve waves of one).
// A wave computes its block transposed, keys x
// queries: a lane then holds 16 keys of one query and a softmax row reduces inside the lane, across the two half-waves and,
// through LDS, across the waves.  q is split once into LDS, in operand order (step of 16 columns, piece, half, row, 16 bytes); a
// key is used by one wave alone, so it goes from memory to registers and is split there: no barrier stands between the
// first product and the last, and the waves of a SIMD split and multiply in turn.  (Keys two steps ahead, whole lines of
// them, spill: 16 x 8 heads of 484 x 484 x 80 138 us against 83.)
//
// Where scores alone would be the split GEMM's (as_gemm), these are the same products in the same order, in the same sums.
// (Otherwise two roundings are saved, see `step`.)  A value that the pieces cannot carry has 64 queries x all keys done again
// with the fp32 instruction here, the GEMM's own tile there.
//
// The heads of a sequence go round fastest among the work-groups: all query blocks of one head at a time would ask one
// channel of the L2 for their keys where rows are whole multiples of its interleaving (4 x 16 heads of 512 x 512 x 64 54 us
// against 45).
//
// Bound: the phases of a work-group follow each other (q's way into LDS, the products with the splitting of the keys
// between them, the softmax, the stores), and one or two work-groups of a CU cover that in part: 16 x 8 heads of
// 484 x 484 x 80 take 23 us of memory traffic and 77 in all.  The kernel of 32 queries on the fp32 instruction
// (tbs_long_kernel), against this one (us): 16 x 16 heads of 256 x 256 x 64 40.7 / 30.2, 16 x 16 of 512 x 512 x 64 159.5 / 132.8,
// 16 x 12 of 176 x 176 x 80 37.0 / 25.2; the split GEMM with a softmax behind it: 16 x 8 of 484 x 484 x 80 129 / 77, 32 x 12
// of 470 x 470 x 128 385 / 279 (78 TFLOP/s), 32 x 12 of 256 x 256 x 48 106.6 / 41.6.
#pragma once
#include <type_traits>

#include "split_bf16.h"
#include "tbg_kernel.h"

namespace anr {
namespace tbg {

constexpr int kSplitQueries = 64;
constexpr uint32_t kPastExtent = 0x80000000u;        // byte offset beyond any extent here
constexpr int kStepBytes = 3 * 2 * kSplitQueries * 16;
constexpr int kCornerBytes = 32 * 36 * 4;            // a wave's block on its way out

constexpr size_t split_lds_bytes(int D, int waves)
{
    const size_t q = (size_t)((D + 15) / 16) * kStepBytes;
    const size_t corners = (size_t)waves * kCornerBytes;
    return q > corners ? q : corners;
}

// The scores of the work-group's queries, from the pieces or, PLAIN, with the fp32 instruction.  False if a value was met that
// the pieces cannot carry, the same for all waves.
template <int W, bool PLAIN>
__device__ __forceinline__ bool split_scores(const Args& p, char* const panel, const int thread, const float* qb, const float* kb, int i0, bool as_gemm, f32x16 (&acc)[2])
{
    const int lane = thread & 63, wave = __builtin_amdgcn_readfirstlane(thread >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const int steps = (p.D + 15) / 16;
    // As the split GEMM counts: the last chunk of 32 columns starts at D - 32, what an earlier one has counted is left out, and
    // so is a step of nothing else.
    const int back_from = as_gemm && p.D > 32 ? (steps - 1) & ~1 : steps, back = 16 * steps - p.D;
    auto column = [&](int s) { return 16 * s - (s >= back_from ? back : 0); };          // first one of a step
    uint32_t lost = 0;

    // a unit is the columns 4t .. 4t+3 and 8+4t .. 8+4t+3 of a step (any order of columns is one as long as both operands use it)
    auto split_unit = [&](const f32x4& lo, const f32x4& hi, u32x4 (&out)[3]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint32_t a, b, c;
            split2(lo[2 * i], lo[2 * i + 1], a, b, c, lost);
            out[0][i] = a; out[1][i] = b; out[2][i] = c;
            split2(hi[2 * i], hi[2 * i + 1], a, b, c, lost);
            out[0][2 + i] = a; out[1][2 + i] = b; out[2][2 + i] = c;
        }
    };
    // D is a multiple of four: a quad of columns is inside a row or past its end (zero)
    const __amdgpu_buffer_rsrc_t qrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(qb), 0, (int)(4 * ((p.S - 1) * (int)p.qs_s + p.D)), 0x00020000);
    const __amdgpu_buffer_rsrc_t krsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(kb), 0, (int)(4 * ((p.S - 1) * (int)p.ks_s + p.D)), 0x00020000);
    auto quad = [&](const __amdgpu_buffer_rsrc_t& rsrc, uint32_t row, int s, int at) {
        const int col = column(s) + at;
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(col >= 16 * (s & ~1) && col < p.D ? row + 4u * (uint32_t)col : kPastExtent), 0, 0));
    };
    for (int u = thread; u < steps * 2 * kSplitQueries; u += 64 * W) {
        const int t = u & 1, row = (u >> 1) % kSplitQueries, s = (u >> 1) / kSplitQueries;
        const uint32_t at = 4u * (uint32_t)(min(i0 + row, p.S - 1) * (int)p.qs_s);
        const f32x4 lo = quad(qrsrc, at, s, 4 * t), hi = quad(qrsrc, at, s, 8 + 4 * t);
        char* const to = panel + s * kStepBytes + t * (kSplitQueries * 16) + row * 16;
        if constexpr (PLAIN) {
            *reinterpret_cast<f32x4*>(to) = lo;
            *reinterpret_cast<f32x4*>(to + 2 * kSplitQueries * 16) = hi;
        } else {
            u32x4 pieces[3];
            split_unit(lo, hi, pieces);
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(to + q * (2 * kSplitQueries * 16)) = pieces[q];
        }
    }

    const uint32_t krow = 4u * (uint32_t)(min(32 * wave + r32, p.S - 1) * (int)p.ks_s);          // keys past S repeat the last one and are masked
    f32x4 raw[2];
    auto load = [&](int s) {
#pragma unroll
        for (int e = 0; e < 2; ++e) raw[e] = quad(krsrc, krow, s, 8 * e + 4 * h);
    };
    // the products of the first pieces, and the other seven
    f32x16 low[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[nb][r] = low[nb][r] = 0.f;
    load(0);
    __syncthreads();                                 // q is staged

    const char* const qrow = panel + h * (kSplitQueries * 16) + r32 * 16;
    // The next step's keys are on their way while this one's are multiplied.  The last step adds the small products' sum ahead
    // of its large products, where the sum is not yet as large as it gets, or behind them, as the split GEMM does.
    auto step = [&](int s, auto last_c) {
        constexpr bool last = decltype(last_c)::value;
        u32x4 a[3];
        f32x4 plain[2];
        if constexpr (PLAIN) {
            plain[0] = raw[0];
            plain[1] = raw[1];
        } else {
            split_unit(raw[0], raw[1], a);
        }
        if (!last) load(s + 1);
        const char* const from = qrow + s * kStepBytes;
        if constexpr (PLAIN) {
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) {
                    const f32x4 q = *reinterpret_cast<const f32x4*>(from + e * (2 * kSplitQueries * 16) + nb * 512);
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[nb] = mfma32(plain[e][i], q[i], acc[nb]);
                }
        } else {
            u32x4 q[2][3];
#pragma unroll
            for (int piece = 0; piece < 3; ++piece)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) q[nb][piece] = *reinterpret_cast<const u32x4*>(from + piece * (2 * kSplitQueries * 16) + nb * 512);
#pragma unroll
            for (int t = 0; t < kProducts; ++t)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) {
                    if (last && t == kProducts - 1 && !as_gemm)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[nb][r] += low[nb][r];
                    f32x16& sum = t < kProducts - 1 ? low[nb] : acc[nb];
                    sum = mfma_bf16(a[kPieceB[t]], q[nb][kPieceA[t]], sum);
                }
        }
    };
    if (32 * wave < p.S) {                           // uniform over the wave: one past the last key has nothing to multiply
#pragma unroll 1
        for (int s = 0; s + 1 < steps; ++s) step(s, std::false_type{});
        step(steps - 1, std::true_type{});
    }
    if constexpr (!PLAIN) {
        if (as_gemm)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[nb][r] += low[nb][r];
        SumCheck sums;
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) sums.check(acc[nb]);
        return !__syncthreads_or(lost_bits(lost) || sums.refused());
    }
    return true;
}

template <int W>
__global__ __launch_bounds__(64 * W, 4) void tbs_split_kernel(const Args p, int vec_store, int as_gemm)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ float red[2][W][kSplitQueries];
    int thread = threadIdx.x;
    // every XCD gets a contiguous range of items: the query blocks of a head share its keys in one L2
    int item = blockIdx.x;
    if (p.xcd_chunk > 0) item = (item & 7) * p.xcd_chunk + (item >> 3);
    const int row = p.d_h.div(item), hh = item - row * p.H;
    const int b = p.d_tiles_i.div(row), ti = row - b * p.tiles_i;
    const int i0 = ti * kSplitQueries;
    const float* const qb = p.q + b * p.qs_b + hh * p.qs_h;
    const float* const kb = p.k + b * p.ks_b + hh * p.ks_h;

    f32x16 sc[2];
    if (!split_scores<W, false>(p, lds, thread, qb, kb, i0, as_gemm != 0, sc)) {
        // values the pieces cannot carry: again with the fp32 instruction
        asm("" : "+v"(thread));
        split_scores<W, true>(p, lds, thread, qb, kb, i0, as_gemm != 0, sc);
    }

    // register r of lane (h, r32), block nb: key 32*wave + 8*(r/4) + 4*h + r%4, query i0 + 32*nb + r32
    const int lane = thread & 63, wave = __builtin_amdgcn_readfirstlane(thread >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    float mx[2], sum[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        mx[nb] = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            sc[nb][r] = 32 * wave + 4 * h + 8 * (r / 4) + r % 4 < p.S ? sc[nb][r] : -INFINITY;
            mx[nb] = fmaxf(mx[nb], sc[nb][r]);
        }
        mx[nb] = fmaxf(mx[nb], __shfl_xor(mx[nb], 32));
        if (h == 0) red[0][wave][32 * nb + r32] = mx[nb];
    }
    __syncthreads();
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
#pragma unroll
        for (int w = 0; w < W; ++w) mx[nb] = fmaxf(mx[nb], red[0][w][32 * nb + r32]);
        // the sum as a tree: as few roundings as softmax_rows_kernel's
        float quarter[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
#pragma unroll
            for (int e = 0; e < 4; ++e) sc[nb][4 * g + e] = exp_nonpositive(sc[nb][4 * g + e] - mx[nb]);          // 0 for masked keys
            quarter[g] = (sc[nb][4 * g] + sc[nb][4 * g + 1]) + (sc[nb][4 * g + 2] + sc[nb][4 * g + 3]);
            __builtin_amdgcn_sched_barrier(0);       // (a few exponentials at a time: all at once they spill)
        }
        sum[nb] = (quarter[0] + quarter[1]) + (quarter[2] + quarter[3]);
        sum[nb] += __shfl_xor(sum[nb], 32);
        if (h == 0) red[1][wave][32 * nb + r32] = sum[nb];
    }
    __syncthreads();
    // every wave is done with q: each takes 32 rows of 36 floats of its room
    float* const ps = reinterpret_cast<float*>(lds) + wave * (32 * 36);
    float* __restrict__ const ob = p.out + b * p.os_b + hh * p.os_h;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        float total[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < W; ++w) total[w % 4] += red[1][w][32 * nb + r32];
        const float inv = 1.0f / ((total[0] + total[1]) + (total[2] + total[3]));
        const int q0 = i0 + 32 * nb, k0 = 32 * wave;
        if (q0 >= p.S || k0 >= p.S) break;           // uniform over the wave, and no barrier follows
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 v = {sc[nb][4 * g] * inv, sc[nb][4 * g + 1] * inv, sc[nb][4 * g + 2] * inv, sc[nb][4 * g + 3] * inv};
            *reinterpret_cast<f32x4*>(&ps[r32 * 36 + 8 * g + 4 * h]) = v;
        }
        // the region is the wave's own and its LDS accesses run in order; the fences only hold the compiler
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (vec_store && k0 + 32 <= p.S) {
            const int col = 4 * (lane & 7);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 8 * i + (lane >> 3);
                const f32x4 v = *reinterpret_cast<const f32x4*>(&ps[row * 36 + col]);
                if (q0 + row < p.S) {
                    float* const o = ob + (q0 + row) * p.os_i + k0 + col;
                    if (vec_store == 2) stg4_nt(o, v);
                    else stg4(o, v);
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int row = 2 * i + h;
                const float v = ps[row * 36 + r32];
                if (q0 + row < p.S && k0 + r32 < p.S) ob[(q0 + row) * p.os_i + k0 + r32] = v;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

}  // namespace tbg
}  // namespace anr
