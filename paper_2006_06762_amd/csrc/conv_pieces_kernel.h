// General convolution (kernels of 9 to 49 taps of any form, any stride, padding, dilation, groups, channel count, width, strided view) on
// the bf16 matrix pipes, each fp32 operand split into three bf16 pieces (split_bf16.h) once per call: split_operands_kernel
// writes the pieces of x and w to the workspace in the order in which conv_pieces_kernel reads them.
//
// What bounds the forms on the fp32 instruction is its rate; a form that splits what each tile loads is bound by the vector
// ALUs: 64 x 64 tiles split a float for every 64 products, which takes them as long as the products take the matrix pipes,
// and a float of x once per tap and column tile.  (Measured as a kernel of its own, on the tiles of gemm_split_kernel.h:
// 14 x 14, 256 -> 256, batch 16, no faster than the fp32 form.)  Here the loop holds loads, LDS traffic and matrix instructions
// only, so small tiles, which fill the chip with the layers of small maps, cost no more per product than large ones.
// Both kernels together against the forms without, in turn on one card, batch 16 unless stated (us): 14 x 14, 256 -> 256, 3 x 3 44.1 ->
// 41.2; 25 x 25, 64 -> 64, 5 x 5 35.6 -> 31.0; 80 x 80, 64 -> 96, 5 x 5, stride 2 139 -> 91.5; 87 x 87, 48 -> 32, 7 x 7, stride 2 115 ->
// 56.5; 12 x 12, 192 -> 512, 5 x 5, batch 32 307 -> 170; 123 x 123, 64 -> 256, 7 x 7, batch 1 251 -> 171; 56 x 56, 128 -> 128, 5 x 5 445 ->
// 316.  The products alone run at 124 to 130 TFLOP/s in the last two, matrix pipes 39 % busy (170 and 77 % in the largest GEMM): a
// barrier and 35 scalar instructions for sixteen of the matrix.
//
// A unit is eight input channels (of one group) at one tap, 16 bytes a piece; units are ordered (channels / 8, tap), so
// that the taps of the same channels follow each other and find their pixels in L1.  A step is two units, sixteen k, one
// matrix instruction deep.
//   x: plane (h, m, l), then image and unit of eight channels, then pixel: 16 bytes.  Taps outside the image have an
//      offset past the extent, which loads zero.
//   w: block of 32 output channels, step, piece, unit, channel: a wave's operand of a step is 3 KB in a row and goes
//      straight to registers (its waves divide the channels of a tile, so nothing is loaded twice).
// Channels past the last one of a group, output channels past the last one and units past the last one are zero.
// A float that the pieces cannot carry leaves a NaN as its last piece: every sum it reaches is refused, and the tile is
// computed again with the fp32 instruction from x and w themselves.
//
// Columns of a wave's two blocks are interleaved (block nb holds pixels 2 r + nb), so that a lane ends up with two
// neighbouring pixels of a channel and 32 lanes write 256 contiguous bytes, whatever the width or alignment of y.
#pragma once
#include <type_traits>

#include "conv_gather_kernel.h"
#include "split_bf16.h"

namespace anr {
namespace cpieces {

using gconv::kOutOfRange;
using gconv::Plan;

constexpr int BP = 64;               // pixels of a tile
constexpr int kMaxTaps = 49;

// Where the pieces lie, and where w is read from (host side: plan and launch_conv2d_pieces in conv_pieces.hip).
struct Pieces {
    char* at;                    // in the workspace, behind the partial tiles
    const float* w;              // row of output channel co: w + (co / w_tile) * w_tile_step + co % w_tile * w_row
    int w_tile, w_tile_step, w_row;
    int w_unit;                  // floats between a row's units of eight channels (the channels of a unit are RS apart)
    uint32_t w_in_bytes;
    int cg8;                     // units of eight channels per group
    int units;                   // cg8 * taps
    int steps;                   // units / 2, rounded up
    uint32_t plane;              // bytes of a plane of x
    uint32_t x_bytes;            // of the three planes: the pieces of w start there
    uint32_t w_bytes;
    int x_units, x_groups_of_256;
    uint32_t rs_mul;             // 2^31 / RS, rounded up
    FastDiv d_hw, d_w, d_cg8g, d_cg8;
};

// Eight floats as pieces, 16 bytes each; a lost one leaves a NaN as its last piece.
__device__ __forceinline__ void split_unit(const float (&v)[8], u32x4 (&out)[3])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t ph, pm, pl, lost = 0;
        split2(v[2 * i], v[2 * i + 1], ph, pm, pl, lost);
        out[0][i] = ph;
        out[1][i] = pm;
        out[2][i] = lost_bits(lost) ? 0x7fc07fc0u : pl;
    }
}

// One launch for both operands: the first work-groups take eight output channels and eight input channels of w each, with all
// their taps, through LDS (rows of w are contiguous in taps, units in channels), the others 256 units of x.  Bound by
// latency: 8 us for 1.4 million floats (14 MB read and written), of which a launch and two memory round trips are 4.
__global__ __launch_bounds__(256) void split_operands_kernel(const ConvArgs p, const Plan g, const Pieces z)
{
    char* const ws = z.at;
    const int tid = threadIdx.x;
    u32x4 out[3];
    const int w_groups = (int)gridDim.x - z.x_groups_of_256;
    if ((int)blockIdx.x >= w_groups) {
        const int i = ((int)blockIdx.x - w_groups) * 256 + tid;
        if (i >= z.x_units) return;
        const int img = z.d_hw.div(i), px = i - img * (p.H * p.W);
        const int n = z.d_cg8g.div(img), cu = img - n * (g.groups * z.cg8);
        const int grp = z.d_cg8.div(cu), c0 = 8 * (cu - grp * z.cg8);
        const int ih = z.d_w.div(px), iw = px - ih * p.W;
        const float* const x = p.x + n * p.xs[0] + (int64_t)(grp * g.Cg + c0) * p.xs[1] + ih * p.xs[2] + iw;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = x[(c0 + e < g.Cg ? e : 0) * p.xs[1]];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = c0 + e < g.Cg ? v[e] : 0.f;
        split_unit(v, out);
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(ws + (size_t)q * z.plane + (size_t)i * 16) = out[q];
        return;
    }
    // eight rows (output channels) of w, 32 threads each
    __shared__ float rows[8 * (8 * kMaxTaps + 1)];
    int b = (int)blockIdx.x;
    const int part = b & 3;
    b >>= 2;
    const int block = z.d_cg8.div(b), c8 = b - block * z.cg8;
    const int blocks_ng = g.tiles_ng * (g.bn / 32);                        // per group of channels
    const int grp = block / blocks_ng;
    const int RS = g.RS, len = 8 * RS, have = min(8, g.Cg - 8 * c8) * RS;
    {
        const int row = tid >> 5, kg = (block - grp * blocks_ng) * 32 + part * 8 + row;
        const bool row_in = kg < g.Kg;
        const int co = grp * g.Kg + (row_in ? kg : 0);
        const float* const w = z.w + (int64_t)(co / z.w_tile) * z.w_tile_step + (int64_t)(co % z.w_tile) * z.w_row + (int64_t)c8 * z.w_unit;
        for (int j0 = tid & 31; j0 < len; j0 += 32 * 7) {
            float v[7];                                                    // (all in flight at once)
#pragma unroll
            for (int i = 0; i < 7; ++i) v[i] = w[min(j0 + 32 * i, have - 1)];
#pragma unroll
            for (int i = 0; i < 7; ++i)
                if (j0 + 32 * i < len) rows[row * (len + 1) + j0 + 32 * i] = row_in && j0 + 32 * i < have ? v[i] : 0.f;
        }
    }
    __syncthreads();
    char* const wp = ws + z.x_bytes + (size_t)block * z.steps * 3072 + part * 128;
    for (int i = tid; i < 8 * RS; i += 256) {
        const int tap = i >> 3, row = i & 7, u = c8 * RS + tap;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = rows[row * (len + 1) + e * RS + tap];
        split_unit(v, out);
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(wp + (size_t)(u >> 1) * 3072 + q * 1024 + (u & 1) * 512 + row * 16) = out[q];
    }
    if ((z.units & 1) && c8 == z.cg8 - 1 && tid < 8) {
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(wp + (size_t)(z.steps - 1) * 3072 + q * 1024 + 512 + tid * 16) = u32x4{0, 0, 0, 0};
    }
}

// Tile of BC channels x 64 pixels, a wave per 32 channels, NWG groups of waves that take every NWG-th step.
template <int BC, int NWG>
struct Shape {
    static constexpr int T = 2 * BC, UB = 2 * BP / T;   // threads of a group; units of x that each stages per step
    static constexpr int BLOCK = 512 + 64;              // 32 pixels; 64 bytes apart, so that neighbouring pixels go to different banks
    static constexpr int UNIT = 2 * BLOCK + 64, PLANE = 2 * UNIT, BUF = 3 * PLANE;
    static constexpr int RED = BC * BP * 4;             // a group's accumulators
    static constexpr int kStaging = NWG * 2 * BUF;
    static constexpr int kRoom = kStaging > (NWG - 1) * RED ? kStaging : (NWG - 1) * RED;
    static_assert(UB * T == 2 * BP && (T == 2 * BP || T == BP), "whole units per thread, one of a step's two per wave");
    static constexpr size_t lds_bytes(int taps) { return (size_t)kRoom + 4 * (size_t)taps * BP; }
    // where pixel px of the tile lies in a unit
    static constexpr int slot(int px) { return (px & 1) * BLOCK + (px >> 1) * 16; }
};

// What follows the loop of a tile: the groups' sums are added, looked over (not if PLAIN: false then if one is refused, with
// nothing stored) and stored, with batch norm and ReLU where the call has them.
template <int BC, int NWG, bool PLAIN>
__device__ __forceinline__ bool store_tile(const ConvArgs& p, const Plan& g, f32x16 (&acc)[2], char* lds, int thread, int split, int tile_n,
                                           int p0, int cl0, int cog)
{
    using S = Shape<BC, NWG>;
    const int wgrp = NWG > 1 ? __builtin_amdgcn_readfirstlane(thread / S::T) : 0;
    const int tid = thread % S::T, lane = tid & 63, wave = tid >> 6;
    const int r32 = lane & 31, h = lane >> 5;
    if (NWG > 1) {
        // groups 1 .. NWG-1 leave their accumulators in the staging buffers, group 0 adds them in group order
        __syncthreads();
        if (wgrp > 0) {
            float* red = reinterpret_cast<float*>(lds + (wgrp - 1) * S::RED) + wave * (2 * 16 * 64) + lane;
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r) red[(nb * 16 + r) * 64] = acc[nb][r];
        }
        __syncthreads();
        if (wgrp == 0) {
#pragma unroll
            for (int o = 1; o < NWG; ++o) {
                const float* red = reinterpret_cast<const float*>(lds + (o - 1) * S::RED) + wave * (2 * 16 * 64) + lane;
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[nb][r] += red[(nb * 16 + r) * 64];
            }
        }
    }
    if (!PLAIN) {
        SumCheck sums;
        sums.check(acc[0]);
        sums.check(acc[1]);
        if (__syncthreads_or(sums.refused())) return false;
    }

    // accumulator register r of lane (h, r32): channel 8*(r/4) + 4*h + r%4 of the wave's 32, pixels 2*r32 and 2*r32 + 1
    typedef float pair __attribute__((ext_vector_type(2), aligned(4)));
    if (g.ksplit > 1) {
        // partial tile: the workspace is padded to whole tiles
        if (NWG > 1 && wgrp > 0) return true;
        float* const ws = p.ws + ((int64_t)split * g.Kpad + tile_n * BC + wave * 32 + 4 * h) * g.Mpad + p0 + 2 * r32;
#pragma unroll
        for (int r = 0; r < 16; ++r) *reinterpret_cast<pair*>(ws + (int64_t)(8 * (r / 4) + r % 4) * g.Mpad) = pair{acc[0][r], acc[1][r]};
        return true;
    }
    // scale and shift of the tile's channels
    float* const bn = reinterpret_cast<float*>(lds);
    if (p.gamma) {
        __syncthreads();                                                   // the staging buffers are free
        if (thread < BC) {
            const int row = cl0 + thread;
            gconv::bn_constants(p, cog + (row < g.Kg ? row : g.Kg - 1), &bn[thread], &bn[BC + thread]);
        }
        __syncthreads();
    }
    if (NWG > 1 && wgrp > 0) return true;

    int64_t at_px[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const int m = p0 + 2 * r32 + nb;
        const int gr = g.d_ow.div(m), ow = m - gr * p.OW;
        const int n = g.d_oh.div(gr), oh = gr - n * p.OH;
        at_px[nb] = n * p.ys[0] + oh * p.ys[2] + ow;
    }
    const int m0 = p0 + 2 * r32;
    const bool pairs = __all(m0 + 1 < g.Mtot && at_px[1] == at_px[0] + 1);        // every lane's pixels are neighbours in y
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = wave * 32 + 8 * (r / 4) + 4 * h + r % 4;
        pair v = {acc[0][r], acc[1][r]};
        if (p.gamma) {
            const float scale = bn[row], shift = bn[BC + row];
            v[0] = fmaxf(fmaf(v[0], scale, shift), 0.f);
            v[1] = fmaxf(fmaf(v[1], scale, shift), 0.f);
        }
        if (cl0 + row >= g.Kg) continue;
        float* const y = p.y + (int64_t)(cog + cl0 + row) * p.ys[1];
        if (pairs) {
            __builtin_nontemporal_store(v, reinterpret_cast<pair*>(y + at_px[0]));
        } else {
            if (m0 < g.Mtot) y[at_px[0]] = v[0];
            if (m0 + 1 < g.Mtot) y[at_px[1]] = v[1];
        }
    }
    return true;
}

// One tile of a work-group: from the pieces, or PLAIN, with the fp32 instruction from x and w in the same order of k.
// False if a sum is refused: then nothing is stored.
template <int BC, int NWG, bool PLAIN>
__device__ __forceinline__ bool compute_tile(const ConvArgs& p, const Plan& g, const Pieces& z, const int thread)
{
    using S = Shape<BC, NWG>;
    constexpr int T = S::T, UB = S::UB;

    extern __shared__ __attribute__((aligned(16))) char slds[];
    const int wgrp = NWG > 1 ? __builtin_amdgcn_readfirstlane(thread / T) : 0;
    char* const region = slds + wgrp * 2 * S::BUF;
    uint32_t* const table = reinterpret_cast<uint32_t*>(slds + S::kRoom);
    const int tid = thread % T;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;

    // blockIdx.x = (split * tiles_n + tile_n) * tiles_m + tile_m
    const int tiles = g.tiles_m * g.tiles_n;
    const int split = g.d_tiles.div((int)blockIdx.x);
    const int trem = (int)blockIdx.x - split * tiles;
    const int tile_n = g.d_tiles_m.div(trem), tile_m = trem - tile_n * g.tiles_m;
    const int grp = g.d_tiles_ng.div(tile_n);                              // channel group of this tile
    const int p0 = tile_m * BP, cl0 = (tile_n - grp * g.tiles_ng) * BC;    // first pixel; first channel inside the group
    const int s_begin = __builtin_amdgcn_readfirstlane(split * g.chunks_per_split);
    const int s_end = __builtin_amdgcn_readfirstlane(min(s_begin + g.chunks_per_split, g.nchunks));

    // Offset of every tap of every pixel inside the units of its image's first eight channels (PLAIN: inside x).
    const int hw = p.H * p.W;
    for (int px = thread % BP; px < BP; px += T * NWG) {
        int m = p0 + px;
        m = m < g.Mtot ? m : g.Mtot - 1;      // columns past the end repeat the last pixel, never stored
        const int gr = g.d_ow.div(m), ow = m - gr * p.OW;
        const int n = g.d_oh.div(gr), oh = gr - n * p.OH;
        const int ihb = oh * p.stride_h - p.pad_h, iwb = ow * p.stride_w - p.pad_w;
        const int row = PLAIN ? (int)p.xs[2] : p.W;
        const int base = PLAIN ? (int)(n * p.xs[0] + (int64_t)grp * g.Cg * p.xs[1] + ihb * p.xs[2] + iwb) : n * (g.groups * z.cg8) * hw + ihb * p.W + iwb;
        for (int i = thread / BP; i < g.RS; i += T * NWG / BP) {
            const int r = g.d_s.div(i), s = i - r * p.S;
            const bool ok = ((unsigned)(ihb + r * p.dil_h) < (unsigned)p.H) & ((unsigned)(iwb + s * p.dil_w) < (unsigned)p.W);
            table[i * BP + px] = ok ? (PLAIN ? 4u : 16u) * (uint32_t)(base + r * p.dil_h * row + s * p.dil_w) : kOutOfRange;
        }
    }

    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(PLAIN ? (void*)p.x : z.at, 0, (int)(PLAIN ? g.x_bytes : z.x_bytes), 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc(PLAIN ? (void*)z.w : z.at + z.x_bytes, 0, (int)(PLAIN ? z.w_in_bytes : z.w_bytes), 0x00020000);
    // Staging of x: pixel tid % 64; unit tid / 64 of a step's two, or (one wave) both.
    const int bpx = tid % BP;
    auto unit_of = [&](int j) { return UB == 1 ? __builtin_amdgcn_readfirstlane(tid / BP) : j; };
    auto eights = [&](int u) { return (int)__umulhi(2u * (uint32_t)u, z.rs_mul); };        // u / RS, u < 2^25
    const int x_group = grp * z.cg8 * hw * 16;
    const int w_block = (tile_n * (BC / 32) + wave) * z.steps * 3072;
    // a lane's row of w in the second try: channels 4h .. 4h+3 of a unit are its
    const int w_co = grp * g.Kg + min(cl0 + wave * 32 + r32, g.Kg - 1);
    const uint32_t w_row = 4u * (uint32_t)(w_co / z.w_tile * z.w_tile_step + w_co % z.w_tile * z.w_row + 4 * h * g.RS);

    __syncthreads();

    // 16 bytes: a piece of a unit, or in the second try half a unit of floats.  Steps past the range load its last one again;
    // their weights are zero (and, in the second try, their pixels), and so are those of a unit past the last one.
    constexpr int PIECES = PLAIN ? 2 : 3;
    u32x4 ra[4][PIECES], rb[2][UB][PIECES];
    uint32_t off[2][UB];
    auto look_up = [&](int s, auto set_c) {                               // table entries of step s, a round ahead of its loads
        constexpr int set = decltype(set_c)::value % 2;
        s = min(s, s_end - 1);
#pragma unroll
        for (int j = 0; j < UB; ++j) {
            const int u = min(2 * s + unit_of(j), z.units - 1);
            off[set][j] = table[(u - eights(u) * g.RS) * BP + bpx];
        }
    };
    auto load_x = [&](int s, auto set_c) {
        constexpr int set = decltype(set_c)::value % 2;
        const bool live = s < s_end;
        s = min(s, s_end - 1);
#pragma unroll
        for (int j = 0; j < UB; ++j) {
            const int u = min(2 * s + unit_of(j), z.units - 1), c8 = eights(u);
            if constexpr (PLAIN) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const bool in = live && 2 * s + unit_of(j) < z.units && 8 * c8 + e < g.Cg;
                    rb[set][j][e / 4][e % 4] = __builtin_bit_cast(
                        uint32_t, __builtin_amdgcn_raw_buffer_load_b32(xrsrc, (int)(in ? off[set][j] : kOutOfRange), in ? 4 * (8 * c8 + e) * (int)p.xs[1] : 0, 0));
                }
            } else {
                const int at = x_group + c8 * hw * 16;
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    rb[set][j][q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, (int)off[set][j], at + q * (int)z.plane, 0));
            }
        }
    };
    auto load_w = [&](int s, auto set_c) {
        constexpr int set = decltype(set_c)::value;
        const uint32_t past = s < s_end ? 0u : kOutOfRange;
        s = min(s, s_end - 1);
#pragma unroll
        for (int q = 0; q < PIECES; ++q) {
            if constexpr (PLAIN) {
                const int u = 2 * s + q, c8 = eights(u);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool in = u < z.units && 8 * c8 + 4 * h + e < g.Cg;
                    const int at = u < z.units && 8 * c8 + e < g.Cg ? 4 * (c8 * z.w_unit + e * g.RS + u - c8 * g.RS) : 0;
                    ra[set][q][e] =
                        __builtin_bit_cast(uint32_t, __builtin_amdgcn_raw_buffer_load_b32(wrsrc, (int)((in ? w_row : kOutOfRange) | past), at, 0));
                }
            } else {
                ra[set][q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, (int)(16 * lane | past), w_block + s * 3072 + q * 1024, 0));
            }
        }
    };
    // (floats: plane 2 * unit + half of the unit)
    auto store_x = [&](int buf) {
#pragma unroll
        for (int j = 0; j < UB; ++j)
#pragma unroll
            for (int q = 0; q < PIECES; ++q)
                *reinterpret_cast<u32x4*>(region + buf * S::BUF + (PLAIN ? (2 * unit_of(j) + q) * S::UNIT : q * S::PLANE + unit_of(j) * S::UNIT) + S::slot(bpx)) = rb[buf][j][q];
    };
    // a wave's pixel operands of a step, read from its buffer a round ahead of their products
    u32x4 rv[2][2][PIECES];
    auto read_x = [&](auto buf_c) {
        constexpr int buf = decltype(buf_c)::value;
        const char* const b = region + buf * S::BUF + h * S::UNIT + r32 * 16;
#pragma unroll
        for (int q = 0; q < PIECES; ++q)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) rv[buf][nb][q] = *reinterpret_cast<const u32x4*>(b + (PLAIN ? 2 * q * S::UNIT : q * S::PLANE) + nb * S::BLOCK);
    };

    // the products of the first pieces (or of the floats themselves), and the other seven
    f32x16 acc[2], low[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[nb][r] = low[nb][r] = 0.f;
    auto multiply = [&](auto set_c) {
        constexpr int R = decltype(set_c)::value, P = R % 2;
        if constexpr (PLAIN) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) acc[nb] = mfma32(__builtin_bit_cast(f32x4, ra[R][q])[e], __builtin_bit_cast(f32x4, rv[P][nb][q])[e], acc[nb]);
        } else {
#pragma unroll
            for (int t = 0; t < kProducts; ++t)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) {
                    f32x16& sum = t < kProducts - 1 ? low[nb] : acc[nb];
                    sum = mfma_bf16(ra[R][kPieceA[t]], rv[P][nb][kPieceB[t]], sum);
                }
        }
    };

    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    using S2 = std::integral_constant<int, 2>;
    using S3 = std::integral_constant<int, 3>;
    int s = s_begin + wgrp;
    look_up(s, S0{});
    look_up(s + NWG, S1{});
    load_x(s, S0{});
    load_x(s + NWG, S1{});
    look_up(s + 2 * NWG, S0{});
    look_up(s + 3 * NWG, S1{});
    load_w(s, S0{});
    load_w(s + NWG, S1{});
    store_x(0);
    load_x(s + 2 * NWG, S0{});
    store_x(1);
    load_x(s + 3 * NWG, S1{});
    look_up(s + 4 * NWG, S0{});
    load_w(s + 2 * NWG, S2{});
    __syncthreads();
    read_x(S0{});
    // Round s: operands of step s are in registers and those of the group's next step in the other buffer; the step after
    // that goes from registers to the buffer that step s left, and later ones are requested.  The products stand between the
    // loads and the LDS traffic, so nothing keeps the matrix pipe waiting but the barrier (the same round with its loads,
    // stores and reads ahead of the products: 0.46 us a step against 0.33 with one wave on a SIMD).
    auto round = [&](int s, auto set_c) {
        constexpr int R = decltype(set_c)::value, P = R % 2;
        __syncthreads();
        look_up(s + 5 * NWG, std::integral_constant<int, P ^ 1>{});
        read_x(std::integral_constant<int, P ^ 1>{});
        store_x(P);
        load_x(s + 4 * NWG, std::integral_constant<int, P>{});
        load_w(s + 3 * NWG, std::integral_constant<int, (R + 3) % 4>{});
        multiply(set_c);
        if constexpr (!PLAIN) {
            constexpr int MATRIX = 0x008, LOAD = 0x020, LDS_READ = 0x100, LDS_WRITE = 0x200;
            __builtin_amdgcn_sched_group_barrier(LDS_READ, UB, 0);
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                __builtin_amdgcn_sched_group_barrier(MATRIX, 1, 0);
                __builtin_amdgcn_sched_group_barrier(LDS_READ, 1, 0);
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                __builtin_amdgcn_sched_group_barrier(MATRIX, 1, 0);
                __builtin_amdgcn_sched_group_barrier(LDS_WRITE, UB, 0);
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                __builtin_amdgcn_sched_group_barrier(MATRIX, 1, 0);
                __builtin_amdgcn_sched_group_barrier(LOAD, UB, 0);
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                __builtin_amdgcn_sched_group_barrier(MATRIX, 1, 0);
                __builtin_amdgcn_sched_group_barrier(LOAD, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(MATRIX, 1, 0);
        }
    };
    // every group runs the same number of rounds: the barriers are the work-group's
    int left = (s_end - s_begin + NWG - 1) / NWG;
#pragma unroll 1
    while (true) {
        round(s, S0{});
        if (left <= 1) break;
        round(s + NWG, S1{});
        if (left <= 2) break;
        round(s + 2 * NWG, S2{});
        if (left <= 3) break;
        round(s + 3 * NWG, S3{});
        if (left <= 4) break;
        s += 4 * NWG;
        left -= 4;
    }
    if (!PLAIN) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[nb][r] += low[nb][r];
    }
    return store_tile<BC, NWG, PLAIN>(p, g, acc, slds, thread, split, tile_n, p0, cl0, grp * g.Kg);
}

// Values the pieces cannot carry: the tile again with the fp32 instruction.
template <int BC, int NWG>
__global__ __launch_bounds__(2 * BC * NWG, 2) void conv_pieces_kernel(const ConvArgs p, const Plan g, const Pieces z)
{
    int thread = threadIdx.x;
    if (compute_tile<BC, NWG, false>(p, g, z, thread)) return;
    asm("" : "+v"(thread));                          // nothing of the second try is held through the first
    compute_tile<BC, NWG, true>(p, g, z, thread);
}

}  // namespace cpieces
}  // namespace anr
