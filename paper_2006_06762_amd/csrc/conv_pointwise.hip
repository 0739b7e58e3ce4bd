// Selection and launch of the streaming pointwise convolution (kernel in conv_pointwise_kernel.h).
#include "conv_pointwise_kernel.h"

namespace anr {
namespace {

// What the kernel takes: 1 x 1, stride 1, no padding (a dilation means nothing to one tap); C one
// of 32, 64, 96, 128, in groups of a multiple of 4 channels;
// images whose planes are dense and follow each other (x and y are then [C or K][H*W] matrices per
// image) with H*W a multiple of 4; 16-byte aligned pointers.  It is chosen where the layer is
// bound by traffic rather than by the matrix pipes: K <= 128 as well.
bool takes(const ConvArgs& a)
{
    if (a.route == 1) return false;
    const int64_t hw = (int64_t)a.H * a.W;
    const bool geom = a.R == 1 && a.S == 1 && a.stride_h == 1 && a.stride_w == 1 && a.pad_h == 0 && a.pad_w == 0 &&
                      a.groups >= 1 && (a.C % a.groups == 0) && (a.K % a.groups == 0) && ((a.C / a.groups) % 4 == 0);
    const bool chans = (a.C == 32 || a.C == 64 || a.C == 96 || a.C == 128) && a.K <= 128;
    const bool dense = a.xs[2] == a.W && a.xs[1] == hw && a.ys[2] == a.W && a.ys[1] == hw && (a.xs[0] % 4 == 0) &&
                       (a.ys[0] % 4 == 0) && (hw % 4 == 0) && is_aligned16(a.x) && is_aligned16(a.y) && is_aligned16(a.w);
    const int64_t tiles = (int64_t)a.N * ((hw + 63) / 64) * ((a.K + 63) / 64);
    return geom && chans && dense && hw < ((int64_t)1 << 30) && tiles < ((int64_t)1 << 31) && tiles >= 256;
}

template <int C_T>
hipError_t launch_as(const ConvArgs& a, hipStream_t stream)
{
    pw::Geom g{};
    g.hw = a.H * a.W;
    g.tiles_p = (g.hw + 63) / 64;
    g.tiles_k = (a.K + 63) / 64;
    const int64_t tiles = (int64_t)a.N * g.tiles_p * g.tiles_k;
    g.xcd_chunk = tiles % 8 == 0 ? (int)(tiles / 8) : 0;
    g.d_tiles_k = make_fastdiv(g.tiles_k);
    g.d_tiles_p = make_fastdiv(g.tiles_p);
    g.cg = a.C / a.groups;
    g.d_kg = make_fastdiv(a.K / a.groups);
    return launch_kernel(pw::conv1x1_stream_kernel<C_T>, dim3((unsigned)tiles), dim3(256), 0, stream, a, g);
}

}  // namespace

bool describe_conv2d_pointwise(const ConvArgs& a, ConvRoute* r)
{
    if (!takes(a)) return false;
    const int64_t hw = (int64_t)a.H * a.W;
    *r = ConvRoute{6, 64, 64, 1, 1, (int)((int64_t)a.N * ((hw + 63) / 64) * ((a.K + 63) / 64)), 0};
    return true;
}

hipError_t launch_conv2d_pointwise(const ConvArgs& a, hipStream_t stream, bool* taken)
{
    *taken = takes(a);
    if (!*taken) return hipSuccess;
    switch (a.C) {
        case 32: return launch_as<32>(a, stream);
        case 64: return launch_as<64>(a, stream);
        case 96: return launch_as<96>(a, stream);
        default: return launch_as<128>(a, stream);
    }
}

namespace {

// y[n] = w . x[n] on the bf16-split GEMM (M = K output channels, N = a plane, K = C; batch norm and ReLU per row where it
// stores), once there are tiles for most of the chip.  On planes that are no multiple of four pixels the convolution
// kernels store four bytes at a time: from 170 tiles of 64 x 64 on (batch 16, 48 -> 160 on 171 x 171 310 -> 161 us, batch 32, 64 ->
// 384 on 45 x 45 87 -> 46, batch 16, 64 -> 64 on 29 x 29 7.8 -> 7.5; 128 tiles 10.9 -> 11.1, 20 to 40 tiles 8.2 -> 9.4).  On others from
// 700 on and 96 channels (batch 16, 256 -> 256 on 84 x 84 150 -> 118, batch 32, 512 -> 256 on 20 x 20 41 -> 32; 288 tiles 13.7 ->
// 16.2, 504 tiles 15.5 -> 15.7); fewer channels were not tried there.
bool pointwise_gemm(const ConvArgs& a, GemmArgs* g)
{
    const int64_t plane = (int64_t)a.H * a.W;
    if (a.route != 0 || a.R != 1 || a.S != 1 || a.stride_h != 1 || a.stride_w != 1 || a.pad_h != 0 || a.pad_w != 0 || a.groups != 1 ||
        a.xs[2] != a.W || a.ys[2] != a.OW || plane < 256 || plane >= ((int64_t)1 << 29) || a.C < 32 || a.K < 48)
        return false;
    if ((int64_t)a.K * a.C >= ((int64_t)1 << 29) || (int64_t)(a.C - 1) * a.xs[1] + plane >= ((int64_t)1 << 29)) return false;
    const int64_t tiles = (int64_t)((a.K + 63) / 64) * ((plane + 63) / 64) * a.N;
    if (tiles < (plane % 4 ? 170 : 700) || (plane % 4 == 0 && (a.C < 96 || a.K < 96)) || tiles >= ((int64_t)1 << 22)) return false;
    *g = GemmArgs{};
    g->A = a.w;
    g->B = a.x;
    g->C = a.y;
    g->M = a.K;
    g->N = (int)plane;
    g->K = a.C;
    g->lda = a.C;
    g->ldb = a.xs[1];
    g->ldc = a.ys[1];
    g->batch = a.N;
    g->batch_inner = 1;
    g->sBo = a.xs[0];
    g->sCo = a.ys[0];
    g->gamma = a.gamma;
    g->beta = a.beta;
    g->mean = a.mean;
    g->var = a.var;
    g->scale_shift = a.scale_shift;
    g->eps = a.eps;
    return true;
}

}  // namespace

bool describe_conv2d_pointwise_gemm(const ConvArgs& a, ConvRoute* r)
{
    GemmArgs g;
    if (!pointwise_gemm(a, &g)) return false;
    int tile = 0, groups = 0;
    gemm_split_variant(g, &tile, &groups);
    *r = ConvRoute{6, tile, tile, 1, groups, (int)(((int64_t)(g.M + tile - 1) / tile) * ((g.N + tile - 1) / tile) * g.batch), 0};
    return true;
}

hipError_t launch_conv2d_pointwise_gemm(const ConvArgs& a, hipStream_t stream, bool* taken)
{
    GemmArgs g;
    *taken = pointwise_gemm(a, &g);
    return *taken ? launch_gemm_split(g, stream) : hipSuccess;
}

}  // namespace anr
