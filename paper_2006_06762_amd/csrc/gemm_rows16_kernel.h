// GMM for very few output tiles and a long reduction, any M, N, K and alignment: a work-group owns one 16 x 16 tile of C and
// its NW waves share the reduction, wave w taking the 64-wide chunks w, w + NW, ...
//
// Bound: the fp32 matrix instruction.  A 32 x 32 tile (gemm_rows32_kernel) keeps the matrix cores of its CU busy for K / 2 x 64
// cycles over four SIMDs, 9 us at K = 2720 with everything else hidden, while most CUs have no tile at all; a quarter of the
// tile on four times the CUs takes a quarter of that, and a load's latency for each of a wave's few chunks.  The lanes of
// v_mfma_f32_16x16x4 may share out k in any way that is the same for both operands: a lane takes 16 k in a row, so its part
// of A is 64 contiguous bytes and goes from memory to registers, as B does (64 bytes of 4 rows an instruction), and no LDS is
// needed before the waves' sums meet.  64 x 64 x 2720 19.9 -> 10.0 us, 3 x 96 x 96 x 3828 27.0 -> 13.8, 200 x 130 x 300
// 6.3 -> 4.6, 48 x 1000 x 700 9.1 -> 5.7.  Sixteen waves instead of eight: 10.3, 14.8, 4.7.
//
// The sums of runs of RUN instructions (4 RUN k) meet in a compensated one: relative to the exact
// results 5.2e-8 (RUN 1) and 8.1e-8 (4), where the kernel of 32 x 32 tiles has 5.2e-8 below K = 288, 6.3e-8 below 800 and 8.5e-8
// from there.
#pragma once
#include "gemm_rows32_kernel.h"

namespace anr {
namespace grows {

constexpr int KC16 = 64;

template <int NW, int RUN>
__global__ __launch_bounds__(64 * NW) void gemm_rows16_kernel(const GemmArgs p, int tiles_m, int tiles_n)
{
    __shared__ double red[NW * 4 * 64];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, kq = lane >> 4;

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
    const int m0 = 16 * tm, n0 = 16 * tn;
    const float* const A = p.A + mat * p.sAo;
    const float* const B = p.B + mat * p.sBo;
    float* __restrict__ C = p.C + mat * p.sCo;
    const int M = p.M, N = p.N, K = p.K;
    const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(A), 0, (int)(4u * (uint32_t)((int64_t)(M - 1) * p.lda + K)), 0x00020000);
    const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(B), 0, (int)(4u * (uint32_t)((int64_t)(K - 1) * p.ldb + N)), 0x00020000);

    // rows and columns past the end repeat the last one and are not stored
    int k = wave * KC16 + 16 * kq;                   // the lane's first of the chunk to load
    uint32_t aoff = 4u * (uint32_t)((int64_t)min(m0 + r16, M - 1) * p.lda + k);
    uint32_t boff = 4u * (uint32_t)((int64_t)k * p.ldb + min(n0 + r16, N - 1));
    const uint32_t ldb4 = 4u * (uint32_t)p.ldb, bstep = NW * KC16 * ldb4;
    f32x4 ra[4];
    float rb[16];
    // k past the end comes as zeros in both operands (in A all but the end of a unit, cleared below)
    auto load = [&] {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            ra[q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(arsrc, (int)(k + 4 * q < K ? aoff + 16 * q : kOutOfRange), 0, 0));
#pragma unroll
        for (int t = 0; t < 16; ++t)
            rb[t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(brsrc, (int)(k + t < K ? boff + t * ldb4 : kOutOfRange), 0, 0));
        k += NW * KC16;
        aoff += 4u * NW * KC16;
        boff += bstep;
    };
    load();
    float s[4] = {0.f, 0.f, 0.f, 0.f}, c[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int k0 = wave * KC16; k0 < K; k0 += NW * KC16) {
        f32x4 a[4];
        float b[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) a[q] = ra[q];
#pragma unroll
        for (int t = 0; t < 16; ++t) b[t] = rb[t];
        if (k0 + KC16 > K) {
#pragma unroll
            for (int t = 0; t < 16; ++t) a[t / 4][t % 4] = k0 + 16 * kq + t < K ? a[t / 4][t % 4] : 0.f;
        }
        load();
        __builtin_amdgcn_sched_barrier(0);           // the loads stay ahead of the products
#pragma unroll
        for (int t = 0; t < 16; t += RUN) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < RUN; ++i) acc = mfma16(a[(t + i) / 4][(t + i) % 4], b[t + i], acc);
            // what an addition rounds off is taken from the next term, as in Sum16
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float y = acc[r] - c[r], sum = s[r] + y;
                c[r] = __builtin_amdgcn_fmed3f((sum - s[r]) - y, -0x1p104f, 0x1p104f);
                s[r] = sum;
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) red[(wave * 4 + r) * 64 + lane] = (double)s[r] - (double)c[r];
    __syncthreads();
    // wave w < 4 finishes accumulator register w: row 4 kq + w
    if (wave < 4) {
        double v = 0.0;
#pragma unroll
        for (int o = 0; o < NW; ++o) v += red[(o * 4 + wave) * 64 + lane];
        const int row = m0 + 4 * kq + wave, col = n0 + r16;
        if (row < M && col < N) C[(int64_t)row * p.ldc + col] = (float)v;
    }
}

}  // namespace grows
}  // namespace anr
