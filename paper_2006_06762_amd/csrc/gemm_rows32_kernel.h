// GMM for few output tiles (more than 64: gemm_rows16_kernel has the fewest) and a long reduction, any M, N, K and
// alignment: a work-group owns one 32 x 32 tile of C
// and its NW waves share the reduction, wave w taking the 32-wide chunks w, w + NW, ...  As in
// gemm_tile32_ksplit_kernel (whole tiles, one chunk per wave) a wave stages its chunk of A and B through a region of
// LDS of its own, so that there is no barrier before the sums meet; here the next chunk's loads are in flight while
// this one is multiplied.
//
// Bound: a chain of latencies per wave (load, LDS, sixteen matrix instructions) with the waves of a SIMD in
// different places of theirs.  The kernels with 64-wide tiles, which these products took before, leave most CUs idle and
// walk the chunks with a barrier each: 96 x 1088 x 3648 63 -> 26 us, 553 x 420 x 1298 29 -> 14, 16 x
// 130 x 68 x 3577 62 -> 28, 192 x 1408 x 864 20 -> 14.
//
// The sums of short runs of k meet in a compensated one, so the error does not grow with K: relative to the exact
// results 4.55e-8 (eight runs a chunk), 5.15e-8 (four), 6.3e-8 (two), 8.05e-8 (one), 8.5e-8 (one, both accumulators
// added up first).  The split GEMM has 5.0e-8 at K = 97, 5.3e-8 at 129, 5.7e-8 at 161, 6.35e-8 at 289, 8.3e-8 at 801, 8.5e-8
// at 864 and 9.9e-8 at 1281, the fp32 kernels 18e-8 at 97 and 34e-8 at 704.  Sixteen waves gained 3 % at K above 3000
// and lost 5 to 30 below; sums in fp64 instead took up to 1.2 times as long.
#pragma once
#include "anr_device.h"
#include "anr_kernels.h"

namespace anr {
namespace grows {

constexpr int KC = 32;
constexpr int LD = 36;                          // LDS row stride, floats
constexpr int kStage = 2 * 32 * LD;             // floats of a wave: A block, then B block
constexpr uint32_t kOutOfRange = 0x80000000u;   // byte offset beyond any descriptor extent

// A compensated sum: what an addition rounds off is taken from the next term.  Infinite sums leave the compensation
// undefined; clamped (it is at most 2^103) it does not turn them into NaN.
struct Sum16 {
    float s[16], c[16];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = c[r] = 0.f;
    }
    __device__ __forceinline__ void add(int r, float x)
    {
        const float y = x - c[r], t = s[r] + y;
        c[r] = __builtin_amdgcn_fmed3f((t - s[r]) - y, -0x1p104f, 0x1p104f);
        s[r] = t;
    }
};

// FOLDS 8, 4, 2, 1: both accumulators join the sum every 4, 8, 16 or 32 k; 0: their sum does every 32.
template <int NW, int FOLDS>
__global__ __launch_bounds__(64 * NW) void gemm_rows32_kernel(const GemmArgs p, int tiles_m, int tiles_n)
{
    static_assert(16 % NW == 0, "a wave finishes 16 / NW accumulator registers");
    extern __shared__ __attribute__((aligned(16))) float lds[];   // [NW waves][kStage]
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;

    // every XCD gets a contiguous run of the batch's tiles (ids are dealt round-robin over the eight)
    int id = blockIdx.x;
    {
        const int all = (int)gridDim.x, per = all >> 3, rest = all & 7, xcd = id & 7, slot = id >> 3;
        id = xcd * per + (xcd < rest ? xcd : rest) + slot;
    }
    const int tiles = tiles_m * tiles_n;
    const int mat = id / tiles;
    id -= mat * tiles;
    const int tn = id / tiles_m, tm = id - tn * tiles_m;
    const int m0 = 32 * tm, n0 = 32 * tn;
    const float* const A = p.A + mat * p.sAo;
    const float* const B = p.B + mat * p.sBo;
    float* __restrict__ C = p.C + mat * p.sCo;
    const int M = p.M, N = p.N, K = p.K;
    const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(A), 0, (int)(4u * (uint32_t)((int64_t)(M - 1) * p.lda + K)), 0x00020000);
    const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(B), 0, (int)(4u * (uint32_t)((int64_t)(K - 1) * p.ldb + N)), 0x00020000);

    // staging unit of a lane: row lane/8 (+ 8 t) of the block, 16 bytes at column 4 (lane % 8).  Rows of A past the end
    // repeat the last one; columns of B past the end are the next row's or past the extent, and not stored.
    const int srow = lane >> 3, sq = (lane & 7) * 4;
    uint32_t aoff[4], boff[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int row = min(m0 + srow + 8 * t, M - 1);
        aoff[t] = 4u * (uint32_t)((int64_t)row * p.lda + wave * KC + sq);
        boff[t] = 4u * (uint32_t)((int64_t)(wave * KC + srow + 8 * t) * p.ldb + n0 + sq);
    }
    const uint32_t astep = 4u * NW * KC, bstep = 4u * NW * KC * (uint32_t)p.ldb;
    const int nchunks = (K + KC - 1) / KC;
    f32x4 ra[4], rb[4];
    int k0 = wave * KC;                          // of the chunk in ra, rb
    // a chunk past the end reads nothing, k past the end of the last one come as zeros in both operands
    auto load = [&](int c) {
        const bool past = c >= nchunks;
        const int kl = c * KC;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            ra[t] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(arsrc, (int)(past ? kOutOfRange : aoff[t]), 0, 0));
            const bool in = kl + srow + 8 * t < K;
            rb[t] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(brsrc, (int)(in ? boff[t] : kOutOfRange), 0, 0));
            aoff[t] += astep;
            boff[t] += bstep;
        }
    };
    load(wave);
    float* const st = lds + wave * kStage;
    Sum16 sum;
    sum.clear();
#pragma unroll 1
    for (int c = wave; c < nchunks; c += NW) {
        if (k0 + KC > K) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) ra[t][e] = k0 + sq + e < K ? ra[t][e] : 0.f;
        }
        k0 += NW * KC;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            *reinterpret_cast<f32x4*>(&st[(srow + 8 * t) * LD + sq]) = ra[t];
            *reinterpret_cast<f32x4*>(&st[32 * LD + (srow + 8 * t) * LD + sq]) = rb[t];
        }
        load(c + NW);
        // the region is the wave's own and its LDS accesses run in order; the fences only hold the compiler
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_sched_barrier(0);       // the loads stay ahead of the products
        f32x16 acc, acc2;
        auto clear = [&] {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = acc2[r] = 0.f;
        };
        auto fold = [&] {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                sum.add(r, acc[r]);
                sum.add(r, acc2[r]);
            }
        };
        constexpr int kRun = FOLDS == 0 ? 4 : FOLDS > 4 ? 1 : 4 / FOLDS;      // steps of eight k
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            if (kk % kRun == 0) clear();
            const f32x4 av = *reinterpret_cast<const f32x4*>(&st[r32 * LD + kk * 8 + 4 * h]);
            float bv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) bv[e] = st[32 * LD + (kk * 8 + 4 * h + e) * LD + r32];
            acc = mfma32(av[0], bv[0], acc);
            acc2 = mfma32(av[1], bv[1], acc2);
            if (FOLDS == 8) {
                fold();
                clear();
            }
            acc = mfma32(av[2], bv[2], acc);
            acc2 = mfma32(av[3], bv[3], acc2);
            if (FOLDS > 0 && (kk + 1) % kRun == 0) fold();
        }
        if (FOLDS == 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) sum.add(r, acc[r] + acc2[r]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    __syncthreads();
    double* const red = reinterpret_cast<double*>(lds);
    static_assert(16 * 64 * sizeof(double) <= kStage * sizeof(float), "a wave's sums fit its region");
#pragma unroll
    for (int r = 0; r < 16; ++r) red[(wave * 16 + r) * 64 + lane] = (double)sum.s[r] - (double)sum.c[r];
    __syncthreads();
    // wave w finishes accumulator registers (16 / NW) w ...: register r is row 8 (r / 4) + 4 h + r % 4
    const int col = n0 + r32;
#pragma unroll
    for (int q = 0; q < 16 / NW; ++q) {
        const int r = wave * (16 / NW) + q;
        double v = 0.0;
#pragma unroll
        for (int o = 0; o < NW; ++o) v += red[(o * 16 + r) * 64 + lane];
        const int row = m0 + 8 * (r / 4) + 4 * h + (r % 4);
        if (row < M && col < N) C[(int64_t)row * p.ldc + col] = (float)v;
    }
}

}  // namespace grows
}  // namespace anr
