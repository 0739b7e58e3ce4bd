// One 32 pixel x 32 channel block of a convolution with the fp32 matrix instruction and operands read
// element by element: what the bf16-split kernels fall back to for values the split cannot carry.
#pragma once
#include "conv_internal.h"
#include "split_bf16.h"

namespace anr {

constexpr uint32_t kPastExtent = 0x80000000u;       // byte offset beyond any descriptor extent

// Lane l is pixel (n, oh, ow) and output channel co (of group grp) number l % 32 of the block; its half
// supplies input channels c with c % 2 == l / 32 of [c_lo, c_hi), relative to the group.  Pixels and
// channels past the end may be repeats of valid ones.  Rows of the result are channels, columns pixels.
__device__ __forceinline__ f32x16 conv_block_fp32(const ConvArgs& p, __amdgpu_buffer_rsrc_t xrsrc,
                                                  __amdgpu_buffer_rsrc_t wrsrc, int n, int oh, int ow, int co, int grp,
                                                  int c_lo, int c_hi)
{
    const int h = (threadIdx.x & 63) >> 5;
    const int Cg = p.C / p.groups, RS = p.R * p.S;
    f32x16 v;
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = 0.f;
    for (int c0 = c_lo; c0 < c_hi; c0 += 2) {
        const int c = c0 + h;
        const uint32_t past = c < c_hi ? 0u : kPastExtent;
        const uint32_t xc = 4u * (uint32_t)(n * p.xs[0] + (int64_t)(grp * Cg + c) * p.xs[1]);
        const uint32_t wc = 4u * (uint32_t)((co * Cg + c) * RS);
        for (int r = 0; r < p.R; ++r)
            for (int s = 0; s < p.S; ++s) {
                const int ih = oh * p.stride_h - p.pad_h + r * p.dil_h, iw = ow * p.stride_w - p.pad_w + s * p.dil_w;
                const bool in = ((unsigned)ih < (unsigned)p.H) & ((unsigned)iw < (unsigned)p.W);
                const uint32_t xo = in ? (xc + 4u * (uint32_t)(ih * (int)p.xs[2] + iw)) | past : kPastExtent;
                const float x = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xrsrc, (int)xo, 0, 0));
                const float w = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wrsrc, (int)((wc + 4u * (uint32_t)(r * p.S + s)) | past), 0, 0));
                v = mfma32(w, x, v);
            }
    }
    return v;
}

}  // namespace anr
