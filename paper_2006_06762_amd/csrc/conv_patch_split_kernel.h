// The 3 x 3 patch kernel on the bf16 matrix pipes, fp32 as three bf16 pieces (split_bf16.h): the tile of
// conv_igemm_kernel's 224-pixel variants, planned by the same code, and at stride 1 the tile of 224 pixels x 64 channels for
// any width (plan_wide in conv_igemm.hip).
//
// Splitting costs vector-ALU time beside the matrix instructions, so it pays where a split float is used
// often: an input element of the staged patch serves nine taps, a weight 224 pixels.  A chunk is sixteen
// input channels.  The patch (virtual rows with their padding, as in conv_igemm_kernel.h) is staged as
// [piece][eight channels][patch pixel], sixteen bytes each: the operand of a pixel at tap (r, s) is one
// 16-byte read at the pixel's place plus the tap's offset.  Weights are staged as
// [piece][tap][eight channels][output channel].
//
// Rows of the result are channels, columns pixels, so that 32 lanes store one whole 128-byte run of a
// channel.  Eight waves: with 64 channels two halves of them by four groups of two blocks of 32 pixels (the
// last group has one: seven blocks), with 32 channels a block of pixels each (one wave only stages).
//
// Bound: a chunk takes 5.3 us (56x56, 64 and 256 channels to 64) where its matrix instructions take 3.8; the
// rest is the split of the next chunk (about 240 vector-ALU instructions per wave, and they hold up the matrix
// pipe) and its LDS stores, which one staging buffer keeps apart from the products.  Against the fp32 form,
// batch 16: 56x56 64 -> 64 34.0 -> 29.7 us, 28x28 256 -> 256 133 -> 100, 112x112 128 -> 64 251 -> 225, 28x28
// 16 -> 128 11.1 -> 8.5; 28x28 128 -> 128 and 512 -> 128 come out level (37, 121).  Dealing the taps to the
// waves instead of the blocks (all waves on all blocks, sums meeting in LDS) was slower.
#pragma once
#include "conv_igemm_kernel.h"
#include "conv_internal.h"
#include "split_bf16.h"

namespace anr {
namespace psplit {

constexpr uint32_t kPastExtent = 0x80000000u;       // byte offset beyond any descriptor extent
constexpr int T = 512;
constexpr int MB = 7, BM = 32 * MB;

// BN output channels (64 or 32), CAP patch pixels (a multiple of 64).
template <int BN, int CAP>
struct Lds {
    static constexpr int XKQ = CAP * 16, XPLANE = 2 * XKQ;      // bytes
    // the six lanes that stage one channel's unit rows, and three channels, fall on different banks
    static constexpr int WKQ = BN * 16 + 48, WTAP = (2 * WKQ + 255) / 256 * 256 + 32, WPLANE = 9 * WTAP;
    static constexpr size_t kStaging = 3 * XPLANE + 3 * WPLANE;
    static constexpr size_t kBytes = kStaging + 2 * BN * sizeof(float);                // and the batch norm
    // the floats themselves: units of four channels in the room of the pieces
    static constexpr int FTAP = 2 * WTAP;
    static_assert(4 * WKQ <= FTAP && 9 * FTAP <= 3 * WPLANE && 4 * XKQ <= 3 * XPLANE, "fits the room of the pieces");
    static_assert(kBytes <= 160 * 1024, "LDS");
};

// One tile of a work-group: as bf16 pieces, or PLAIN, with the fp32 instruction.  False if it met a value that the
// pieces cannot carry: then nothing is stored.
template <int BN, int CAP, bool PACKED, bool PLAIN>
__device__ __forceinline__ bool compute_tile(const ConvArgs& p, const igemm::Geom& g, const int wp, const int tid)
{
    using L = Lds<BN, CAP>;
    constexpr int XKQ = L::XKQ, XPLANE = L::XPLANE, WKQ = L::WKQ, WTAP = L::WTAP, WPLANE = L::WPLANE;
    constexpr int NB = BN / 32, MG = 8 / NB, BLK = MG == 4 ? 2 : 1;      // blocks of 32 pixels of a wave
    constexpr int PX = (CAP + T - 1) / T;                                // patch pixels of a thread
    extern __shared__ __attribute__((aligned(16))) char plds[];
    char* const lx = plds;
    char* const lw = plds + 3 * XPLANE;
    float* const lbn = reinterpret_cast<float*>(plds + L::kStaging);

    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const int wn = wave % NB, mg = wave / NB;
    int tile_m, tile_n;
    {
        const int w = blockIdx.x;
        if (g.xcd_n) {        // the tile grid splits eight ways (xcd_n is a power of two)
            const int xcd = w & 7, slot = w >> 3;
            const int lm = g.d_sub_n.div(slot);
            tile_m = (xcd >> g.xcd_n_shift) * g.sub_m + lm;
            tile_n = (xcd & (g.xcd_n - 1)) * g.sub_n + (slot - lm * g.sub_n);
        } else {
            tile_n = g.d_tiles_m.div(w);
            tile_m = w - tile_n * g.tiles_m;
        }
    }
    const int m0 = tile_m * BM, co0 = tile_n * BN;
    const int g0 = g.d_ow.div(m0);
    const int n_first = g.d_oh.div(g0);
    const int v0 = n_first * g.HV + (g0 - n_first * p.OH) * p.stride_h;

    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.x), 0, (int)g.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(PACKED ? p.wpack : p.w), 0,
                                                                           (int)(PACKED ? g.wpack_bytes : g.w_bytes), 0x00020000);

    // ---- staging: patch pixel of this thread (the waves without weights to stage take the first ones) and
    //      its input offset; weight unit (row r of the kernel, eight channels, output channel)
    const int px0 = (tid + T - 6 * BN) & (T - 1);
    uint32_t xoff[PX];
    bool stages[PX];                               // (uniform over the wave) it has pixels of the patch there
#pragma unroll
    for (int i = 0; i < PX; ++i) {
        const int px = px0 + T * i;
        stages[i] = (CAP % T == 0 || i + 1 < PX || px < CAP) && (i == 0 || __builtin_amdgcn_readfirstlane(px) < g.VR * wp);
        const int vr = px / wp, col = px - vr * wp;
        const int v = v0 + vr;
        const int n = g.d_hv.div(v), ih = v - n * g.HV - p.pad_h, iw = col - p.pad_w;
        const bool in = (vr < g.VR) & (n < p.N) & ((unsigned)ih < (unsigned)p.H) & ((unsigned)iw < (unsigned)p.W);
        xoff[i] = in ? 4u * (uint32_t)(n * p.xs[0] + ih * p.xs[2] + iw) : kPastExtent;
    }
    const int wr = tid % 3, wk = tid / 3 & 1, wc = tid / 6;
    const bool has_w = wc < BN;
    uint32_t woff, wstep;                          // bytes; wstep: from one chunk to the next
    if (PACKED) {
        // images of eight input channels: BN rows of 72 weights and four floats of padding
        woff = 4u * (uint32_t)(((tile_n * (p.C / 8) + wk) * BN + (has_w ? wc : 0)) * 76 + 3 * wr);
        wstep = 4u * 2 * BN * 76;
    } else {
        woff = 4u * (uint32_t)((min(co0 + wc, p.K - 1) * p.C + 8 * wk) * 9 + 3 * wr);
        wstep = 4u * 16 * 9;
    }
    char* const dx = lx + px0 * 16;
    char* const dw = PLAIN ? lw + 3 * wr * L::FTAP + 2 * wk * WKQ + wc * 16 : lw + 3 * wr * WTAP + wk * WKQ + wc * 16;

    float rx[PX][2][8], rw[8][3];
    const uint32_t xs1b = 4u * (uint32_t)p.xs[1];
    auto load_chunk = [&](int ck) {
#pragma unroll
        for (int i = 0; i < PX; ++i)
            if (i == 0 || stages[i]) {
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        rx[i][k][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xrsrc, (int)xoff[i], (int)((uint32_t)(16 * ck + 8 * k + e) * xs1b), 0));
            }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            typedef float f32x3 __attribute__((ext_vector_type(3)));
            const f32x3 v = __builtin_bit_cast(f32x3, __builtin_amdgcn_raw_buffer_load_b96(wrsrc, (int)woff + 36 * e, (int)((uint32_t)ck * wstep), 0));
#pragma unroll
            for (int s = 0; s < 3; ++s) rw[e][s] = v[s];
        }
    };
    uint32_t lost = 0;
    auto store_chunk = [&] {
        if constexpr (PLAIN) {
            // units of four channels
#pragma unroll
            for (int i = 0; i < PX; ++i)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (i > 0 && !stages[i]) break;
                    const float* const v = rx[i][u / 2] + 4 * (u % 2);
                    *reinterpret_cast<f32x4*>(dx + u * XKQ + T * 16 * i) = f32x4{v[0], v[1], v[2], v[3]};
                }
            if (has_w) {
#pragma unroll
                for (int t = 0; t < 3; ++t)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        *reinterpret_cast<f32x4*>(dw + t * L::FTAP + u * WKQ) = f32x4{rw[4 * u][t], rw[4 * u + 1][t], rw[4 * u + 2][t], rw[4 * u + 3][t]};
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < PX; ++i)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if (i > 0 && !stages[i]) break;
                u32x4 s[3];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t hh, mm, ll;
                    split2(rx[i][k][2 * e], rx[i][k][2 * e + 1], hh, mm, ll, lost);
                    s[0][e] = hh; s[1][e] = mm; s[2][e] = ll;
                }
#pragma unroll
                for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(dx + q * XPLANE + k * XKQ + T * 16 * i) = s[q];
            }
        if (has_w) {
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                u32x4 s[3];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t hh, mm, ll;
                    split2(rw[2 * e][t], rw[2 * e + 1][t], hh, mm, ll, lost);
                    s[0][e] = hh; s[1][e] = mm; s[2][e] = ll;
                }
#pragma unroll
                for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(dw + q * WPLANE + t * WTAP) = s[q];
            }
        }
    };
    load_chunk(0);
    __builtin_amdgcn_sched_barrier(0);

    if (tid < BN) {
        const int co = min(co0 + tid, p.K - 1);
        float scale = 1.f, shift = 0.f;
        if (p.scale_shift) {
            scale = p.scale_shift[co];
            shift = p.scale_shift[p.K + co];
        } else if (p.gamma) {
            scale = p.gamma[co] / sqrtf(p.var[co] + p.eps);
            shift = p.beta[co] - p.mean[co] * scale;
        }
        lbn[tid] = scale;
        lbn[BN + tid] = shift;
    }

    // operand addresses: the pixel of the wave's blocks at tap (0, 0) (a block past the seventh repeats it)
    uint32_t xa[BLK];
#pragma unroll
    for (int b = 0; b < BLK; ++b) {
        const int m = min(m0 + 32 * min(BLK * mg + b, MB - 1) + r32, g.Mtot - 1);
        const int gr = g.d_ow.div(m), ow = m - gr * p.OW;
        const int n = g.d_oh.div(gr), oh = gr - n * p.OH;
        xa[b] = (uint32_t)(((n * g.HV + oh * p.stride_h - v0) * wp + ow * p.stride_w) * 16 + h * XKQ);
    }
    const char* const wa = lw + h * WKQ + (32 * wn + r32) * 16;
    // The products of the first pieces, and the other seven, at most 2^-7 of those: a chunk rounds the large sum
    // nine times.  Tiles of 32 channels, whose fp32 kernel adds up four parts, have registers for a large sum per
    // kernel row (28x28, 128 -> 128, inputs and weights of one sign: 1.2 units of 2^-24 rms; 3.0 with one sum, 2.2
    // with the fp32 kernel.  Tiles of 64, one sum: 56x56, 64 -> 64 2.2 against 3.0).
    constexpr int SUMS = BLK == 1 ? 3 : 1;
    f32x16 acc[BLK][SUMS], low[BLK];
#pragma unroll
    for (int b = 0; b < BLK; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            low[b][r] = 0.f;
#pragma unroll
            for (int i = 0; i < SUMS; ++i) acc[b][i][r] = 0.f;
        }

    auto multiply = [&](auto blocks_c) {
        constexpr int blocks = decltype(blocks_c)::value;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const char* const xt = lx + ((t / 3) * wp + t % 3) * 16;
            if constexpr (PLAIN) {
                // the wave's half h takes the units 2u + h, channel by channel
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const f32x4 wv = *reinterpret_cast<const f32x4*>(wa + t * L::FTAP + 2 * u * WKQ);
                    f32x4 xv[blocks];
#pragma unroll
                    for (int b = 0; b < blocks; ++b) xv[b] = *reinterpret_cast<const f32x4*>(xt + xa[b] + 2 * u * XKQ);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int b = 0; b < blocks; ++b) acc[b][t / 3 % SUMS] = mfma32(wv[e], xv[b][e], acc[b][t / 3 % SUMS]);
                }
                continue;
            }
            u32x4 wv[3], xv[3][blocks];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                wv[q] = *reinterpret_cast<const u32x4*>(wa + q * WPLANE + t * WTAP);
#pragma unroll
                for (int b = 0; b < blocks; ++b) xv[q][b] = *reinterpret_cast<const u32x4*>(xt + xa[b] + q * XPLANE);
            }
#pragma unroll
            for (int i = 0; i < kProducts; ++i)
#pragma unroll
                for (int b = 0; b < blocks; ++b) {
                    f32x16& sum = i < kProducts - 1 ? low[b] : acc[b][t / 3 % SUMS];
                    sum = mfma_bf16(wv[kPieceA[i]], xv[kPieceB[i]][b], sum);
                }
        }
    };
    const int chunks = p.C / 16;
    for (int ck = 0; ck < chunks; ++ck) {
        store_chunk();
        __syncthreads();
        load_chunk(ck + 1 < chunks ? ck + 1 : ck);
        __builtin_amdgcn_sched_barrier(0);
        if (BLK * mg + BLK <= MB) multiply(std::integral_constant<int, BLK>{});
        else if (BLK * mg < MB) multiply(std::integral_constant<int, 1>{});
        __syncthreads();
    }

    SumCheck sums;
#pragma unroll
    for (int b = 0; b < BLK; ++b) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int i = 0; i < SUMS; ++i) low[b][r] += acc[b][i][r];
        if (BLK * mg + b < MB) sums.check(low[b]);
    }
    if (!PLAIN && __syncthreads_or(lost_bits(lost) || sums.refused())) return false;

    // register r of lane (h, r32): channel 8*(r/4) + 4*h + r%4 of the half, pixel r32 of the block
    auto store_block = [&](int mb, f32x16 v, bool runs) {
        const int m = m0 + 32 * mb + r32;
        const int gr = g.d_ow.div(m), ow = m - gr * p.OW;
        const int n = g.d_oh.div(gr), oh = gr - n * p.OH;
        const int ch0 = 32 * wn + 4 * h;
        if (p.gamma) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int ch = ch0 + 8 * (r / 4) + (r % 4);
                v[r] = fmaxf(fmaf(v[r], lbn[ch], lbn[BN + ch]), 0.f);
            }
        }
        if (m >= g.Mtot) return;
        float* const y = p.y + n * p.ys[0] + (co0 + ch0) * p.ys[1] + oh * p.ys[2] + ow;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int ch = 8 * (r / 4) + (r % 4);
            if (co0 + ch0 + ch < p.K) {
                if (runs) __builtin_nontemporal_store(v[r], y + ch * p.ys[1]);
                else y[ch * p.ys[1]] = v[r];
            }
        }
    };
#pragma unroll
    for (int b = 0; b < BLK; ++b)
        if (BLK * mg + b < MB) store_block(BLK * mg + b, low[b], g.vec_store != 0);
    return true;
}

// Values the pieces cannot carry: the tile again with the fp32 instruction, staged the same way.  The two tries
// take 71 us for 56x56, 64 -> 64, batch 16, with such a value in every tile (without 30 to 34; element by element,
// without staging, 168), and 250 us for 28x28, 256 -> 256 (105; 685).  Ending the first try early, as the GEMM
// does, costs ordinary values 2 %.
template <int BN, int CAP, bool PACKED>
__global__ __launch_bounds__(T, 2) void conv_patch_split_kernel(const ConvArgs p, const igemm::Geom g, int wp)
{
    int tid = threadIdx.x;
    if (compute_tile<BN, CAP, PACKED, false>(p, g, wp, tid)) return;
    asm("" : "+v"(tid));                             // nothing of the second try is held through the first
    compute_tile<BN, CAP, PACKED, true>(p, g, wp, tid);
}

}  // namespace psplit
}  // namespace anr
