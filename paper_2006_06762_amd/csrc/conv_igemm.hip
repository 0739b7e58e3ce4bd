// Variant table and shape-driven selection for the implicit-GEMM convolution
// (kernel and its description in conv_igemm_kernel.h).
#include "conv_igemm_kernel.h"
#include "conv_patch_split_kernel.h"

namespace anr {
namespace {

using namespace igemm;

//                       WM WN  wM wN ks  R  S CPH   (tile = 32*WM*wM pixels x 32*WN*wN channels)
using V224x64 = Variant<7, 1, 1, 2, 2, 3, 3, 4>;   // 4 waves: two 7x1-block tiles, 2-way k split
using V224x32 = Variant<7, 1, 1, 1, 4, 3, 3, 4>;   // 4 waves share one 7x1-block tile along k
using V128x64 = Variant<2, 2, 2, 1, 2, 3, 3, 4>;   // 4 waves, 2x2 blocks each, 2-way k split
using V64x64 = Variant<2, 2, 1, 1, 4, 3, 3, 4>;    // 4 waves share one 2x2-block tile along k

template <class V>
void consider(const ConvArgs& a, double* best_cost, int* best, int id, Geom* g, size_t* lds)
{
    Geom gg;
    size_t l = 0;
    if (!V::plan(a, &gg, &l)) return;
    const double c = V::cost(a);
    if (*best < 0 || c < *best_cost) {
        *best_cost = c;
        *best = id;
        *g = gg;
        *lds = l;
    }
}

// Instantiations whose LDS geometry is a compile-time constant, one per (tile variant, LDS
// row stride, LDS plane stride): the shapes of the ResNet-style 3x3 layers this library is
// tuned on.  Anything else runs the same kernel with run-time strides.
template <class V, int XU, int RSL_T, int P_T, int NBUF>
bool try_fixed(const ConvArgs& a, const Geom& g, size_t lds, hipStream_t stream, hipError_t* err)
{
    if (g.RSL != RSL_T || g.P != P_T || V::units_per_thread(g) > XU) return false;
    *err = V::template launch_fixed<XU, RSL_T, P_T, NBUF>(a, g, lds, stream);
    return true;
}


// Picks the variant for `a`: its index, geometry and LDS size; -1 when no variant runs it.
int select_variant(const ConvArgs& a, Geom* g, size_t* lds)
{
    const int64_t x_extent = (int64_t)(a.N - 1) * a.xs[0] + (int64_t)(a.C - 1) * a.xs[1] +
                             (int64_t)(a.H - 1) * a.xs[2] + a.W;
    const int64_t w_extent = (int64_t)a.K * a.C * a.R * a.S;
    // 32-bit byte offsets inside x and w, 31-bit pixel and virtual-row indices
    // 3 x 3 only: pointwise layers were measured through this kernel as well (chunks of 32
    // channels) and ran level with or behind conv_taps_kernel on every ResNet-style shape
    const bool k3 = a.R == 3 && a.S == 3 && (a.C % 8 == 0);
    const bool ok = k3 && a.dil_h == 1 && a.dil_w == 1 && a.groups == 1 && (a.W % 4 == 0) && is_aligned16(a.x) &&
                    is_aligned16(a.w) && (a.xs[0] % 4 == 0) && (a.xs[1] % 4 == 0) &&
                    (a.xs[2] % 4 == 0) && x_extent < (int64_t)1 << 30 && w_extent < (int64_t)1 << 30 &&
                    (int64_t)a.N * a.OH * a.OW < (int64_t)1 << 30;
    if (!ok) return -1;

    double best_cost = 0.0;
    int best = -1;
    consider<V224x64>(a, &best_cost, &best, 0, g, lds);
    consider<V224x32>(a, &best_cost, &best, 1, g, lds);
    consider<V128x64>(a, &best_cost, &best, 2, g, lds);
    consider<V64x64>(a, &best_cost, &best, 3, g, lds);
    return best;
}

// The tuned kernel has no split of the reduction across work-groups: with few output tiles
// (batch 1) most CUs would idle, and the general kernel with split-K is faster.
constexpr int kMinTunedWorkGroups = 112;

struct IgemmPlan {
    int variant;     // 0 V224x64, 1 V224x32, 2 V128x64, 3 V64x64, 4 the bf16-split form at any width; -1: the kernel does not take the call
    Geom g;
    size_t lds;
    int cap;         // variant 4: patch pixels it needs room for (512 or 768)
    bool patch_order;      // variant 4: an fp32 form runs the layer too, so its pack has the order they share
};

// The bf16-split 224 x 64 tile without the fp32 forms' conditions (it loads single floats, so any width, alignment
// and row stride): stride 1, whole chunks of sixteen channels, a patch that fits whatever pixel a tile starts at.  An
// image's virtual rows are the zero rows above it and its own; the zero rows below it are the next image's.
static_assert(V224x64::BN == 64 && V128x64::BN == 64 && V64x64::BN == 64 && V224x64::CK == V128x64::CK && V224x64::CK == V64x64::CK &&
              V224x64::CK == 8, "one order of packed weights for all tiles of 64 channels");
bool plan_wide(const ConvArgs& a, IgemmPlan* p)
{
    constexpr int BM = psplit::BM, BN = 64;
    if (a.R != 3 || a.S != 3 || a.C % 16 != 0 || a.groups != 1 || a.stride_h != 1 || a.stride_w != 1 || a.dil_h != 1 || a.dil_w != 1 ||
        a.pad_h > 2 || a.OW < 24)
        return false;
    const int64_t x_extent = (int64_t)(a.N - 1) * a.xs[0] + (int64_t)(a.C - 1) * a.xs[1] + (int64_t)(a.H - 1) * a.xs[2] + a.W;
    const int64_t w_extent = (int64_t)a.K * a.C * 9, ohow = (int64_t)a.OH * a.OW, pack = V224x64::packed_floats(a);
    if (x_extent >= (int64_t)1 << 29 || w_extent >= (int64_t)1 << 29 || pack >= (int64_t)1 << 29 || a.N * ohow >= (int64_t)1 << 30) return false;
    Geom* g = &p->g;
    *g = Geom{};
    g->Mtot = (int)(a.N * ohow);
    g->ohow = (int)ohow;
    g->HV = a.H + a.pad_h;
    const int64_t rows = (BM - 1 + a.OW - 1) / a.OW + 1, crossings = (BM - 1 + ohow - 1) / ohow;
    const int64_t vr = rows + crossings * (g->HV > a.OH ? g->HV - a.OH : 0) + 2, px = vr * (a.OW + 2);
    if (px > 768 || (int64_t)(a.N + 1) * g->HV + vr >= (int64_t)1 << 31) return false;
    g->VR = (int)vr;
    p->cap = px <= 512 ? 512 : 768;
    g->vec_store = (ohow % 4 == 0) && a.ys[2] == a.OW && (a.ys[0] % 4 == 0) && (a.ys[1] % 4 == 0) && is_aligned16(a.y);
    g->d_ow = make_fastdiv(a.OW);
    g->d_oh = make_fastdiv(a.OH);
    g->d_hv = make_fastdiv(g->HV);
    g->x_bytes = (uint32_t)(4 * x_extent);
    g->w_bytes = (uint32_t)(4 * w_extent);
    g->wpack_bytes = (uint32_t)(4 * pack);
    g->tiles_m = (g->Mtot + BM - 1) / BM;
    g->tiles_n = (a.K + BN - 1) / BN;
    g->d_tiles_m = make_fastdiv(g->tiles_m);
    g->d_sub_n = make_fastdiv(1);
    return (int64_t)g->tiles_m * g->tiles_n < ((int64_t)1 << 31);
}

// Time estimates (us) of that form and of the fp32 tiles it competes with: rounds of one work-group per CU, each a
// fixed part and its channels.  Within 8 % of 90 layers of 16 to 512 channels on maps of 24 to 224 pixels.
double wide_us(const ConvArgs& a, const IgemmPlan& p)
{
    const double rounds = (double)(((int64_t)p.g.tiles_m * p.g.tiles_n + 255) / 256);
    return 2.0 + rounds * (4.5 + a.C / 16 * (p.cap == 512 ? 5.8 : 6.2));
}

double fp32_us(const ConvArgs& a, const Geom& g, int variant)
{
    const double rounds = (double)(((int64_t)g.tiles_m * g.tiles_n + 255) / 256);
    return 2.0 + rounds * (variant == 2 ? 4.0 + 0.274 * a.C : 2.5 + 0.145 * a.C);
}

// The one planning pass of a call: variant, geometry and LDS size, with the descriptor's route
// applied (1: whenever a variant runs the shape, the fp32 ones first; 2: never; 0: with enough output tiles).  Depends
// on the descriptor and on the alignment of x and w only (null pointers count as aligned), so a
// pack made for a descriptor fits every later call with it.
void plan_igemm(const ConvArgs& a, IgemmPlan* p)
{
    p->variant = -1;
    p->patch_order = false;
    if (a.route == 2) return;
    if (a.wpack && !is_aligned16(a.x)) {
        // a pack is for the plan of aligned pointers; of its kernels only the form for any width reads this x
        ConvArgs b = a;
        b.x = nullptr;
        plan_igemm(b, p);
        if (p->variant != 4) p->variant = -1;
        return;
    }
    const int best = select_variant(a, &p->g, &p->lds);
    const bool tuned = best >= 0 && (a.route == 1 || (int64_t)p->g.tiles_m * p->g.tiles_n >= kMinTunedWorkGroups);
    if (tuned && (best < 2 || a.route == 1)) {
        p->variant = best;
        return;
    }
    // The bf16-split tile at any width, where its estimate is the shorter one by the estimates' spread (81 x 81, 512 -> 96, batch
    // 4, 307 -> 215 us; 57 x 57, 64 -> 512, batch 4, 81 -> 65; 42 x 42, 128 -> 160, batch 32, 214 -> 184; 124 x 124, 32 -> 512, batch
    // 7, 452 -> 318, weights not packed; on average 0.82 of the time of the layers that take it).  Few or half-filled rounds, channels far from a
    // multiple of 64 and few input channels leave it behind (38 x 38, 128 -> 64, batch 16, 42 against 51).  Weights that are
    // not 16-byte aligned cost the general kernels more, so more layers take it (16 x 25 x 25, 256 -> 256, 156 -> 107; a
    // single 24 x 24, 512 -> 64, stays: 155 against 186).
    IgemmPlan wide;
    if (plan_wide(a, &wide) && (a.route == 1 || wide_us(a, wide) < 0.93 * (tuned ? fp32_us(a, p->g, best) : conv2d_gather_estimate_us(a)))) {
        *p = wide;
        p->variant = 4;
        p->patch_order = tuned;
        return;
    }
    if (tuned) p->variant = best;
}

// Patch pixels the bf16-split form of a 224-pixel tile needs room for (512 or 1024), 0 if it does not take
// the call: whole chunks of sixteen channels, a patch that fits its LDS, byte offsets below the out-of-range
// marker, and stride 1 (at stride 2 a patch pixel serves 2.25 taps, and splitting costs as much as the
// faster products save: 28x28, 256 -> 512, batch 16 67.3 against 71.6 us).
int split_patch(const ConvArgs& a, const Geom& g, int most, int* wp)
{
    *wp = (a.OW - 1) * a.stride_w + a.S;
    const int64_t px = (int64_t)g.VR * *wp;
    if (a.C % 16 != 0 || a.stride_h != 1 || a.stride_w != 1 || px > most || g.x_bytes >= psplit::kPastExtent || g.w_bytes >= psplit::kPastExtent ||
        g.wpack_bytes >= psplit::kPastExtent)
        return 0;
    return px <= 512 ? 512 : 1024;
}

template <int BN, int CAP>
hipError_t launch_patch_split(const ConvArgs& a, const Geom& g, int wp, hipStream_t stream)
{
    auto kern = a.wpack ? psplit::conv_patch_split_kernel<BN, CAP, true> : psplit::conv_patch_split_kernel<BN, CAP, false>;
    static LdsLimit granted[2];
    constexpr size_t lds_bytes = psplit::Lds<BN, CAP>::kBytes;
    const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), lds_bytes, granted[a.wpack ? 1 : 0]);
    if (e != hipSuccess) return e;
    return launch_kernel(kern, dim3((unsigned)(g.tiles_m * g.tiles_n)), dim3(psplit::T), lds_bytes, stream, a, g, wp);
}

hipError_t launch_igemm_plan(const ConvArgs& a, const IgemmPlan& p, hipStream_t stream)
{
    const Geom& g = p.g;
    const size_t lds = p.lds;
    hipError_t err = hipSuccess;
    int wp = 0;
    switch (p.variant) {
        case 0:
            // (left to the fp32 forms: channel counts of 8 mod 16, wider patches, offsets beyond 31 bits)
            if (split_patch(a, g, 512, &wp)) return launch_patch_split<64, 512>(a, g, wp, stream);
            if (try_fixed<V224x64, 3, 64, 384, 3>(a, g, lds, stream, &err)) return err;     // 56x56 maps, stride 1
            return V224x64::launch(a, g, lds, stream);
        case 1:
            if (const int cap = split_patch(a, g, 1024, &wp))
                return cap == 512 ? launch_patch_split<32, 512>(a, g, wp, stream) : launch_patch_split<32, 1024>(a, g, wp, stream);
            if (try_fixed<V224x32, 3, 36, 432, 3>(a, g, lds, stream, &err)) return err;     // 28x28 maps, stride 1
            if (try_fixed<V224x32, 8, 32, 1088, 3>(a, g, lds, stream, &err)) return err;    // 28x28 maps, stride 2
            return V224x32::launch(a, g, lds, stream);
        case 4: return p.cap == 512 ? launch_patch_split<64, 512>(a, g, a.OW + 2, stream) : launch_patch_split<64, 768>(a, g, a.OW + 2, stream);
        case 2: return V128x64::launch(a, g, lds, stream);
        default: return V64x64::launch(a, g, lds, stream);
    }
}

// Floats of the packed weights of plan p, and its channel tile and chunk (output channels x input channels); none for
// plans whose pack is a plain copy.  Plans 0, 2, 3 and 4 share one order.
int64_t packed_floats(const ConvArgs& a, const IgemmPlan& p, int* bn, int* ck)
{
    switch (p.variant == 4 && p.patch_order ? 0 : p.variant) {
        case 0: *bn = V224x64::BN; *ck = V224x64::CK; return V224x64::packed_floats(a);
        case 1: *bn = V224x32::BN; *ck = V224x32::CK; return V224x32::packed_floats(a);
        case 2: *bn = V128x64::BN; *ck = V128x64::CK; return V128x64::packed_floats(a);
        case 3: *bn = V64x64::BN; *ck = V64x64::CK; return V64x64::packed_floats(a);
        default: *bn = *ck = 0; return 0;
    }
}

// Writes the pack's weights part in the patch kernel's order: for channel tile t and chunk q the
// LDS image of the tile's BN channels, KC = CK * 9 weights each in OIHW order followed by the four
// floats of padding of an LDS row; channels past K are zero.  One thread per float.
__global__ __launch_bounds__(256) void conv_pack_patch_kernel(const float* __restrict__ w, float* __restrict__ out,
                                                              int K, int C, int bn, int ck, int64_t total)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int kc = ck * 9, ws = kc + 4, nchunks = C / ck;
    const int j = (int)(idx % ws);
    int64_t t = idx / ws;
    const int col = (int)(t % bn);
    t /= bn;
    const int chunk = (int)(t % nchunks);
    const int tile = (int)(t / nchunks);
    const int co = tile * bn + col;
    out[idx] = (j < kc && co < K) ? w[((int64_t)co * C + (int64_t)chunk * ck) * 9 + j] : 0.f;
}

// Plain copy (plans other than the patch kernel keep OIHW order).
__global__ __launch_bounds__(256) void conv_pack_copy_kernel(const float* __restrict__ w, float* __restrict__ out, int64_t total)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx < total) out[idx] = w[idx];
}

// Folded batch norm, the same fp32 arithmetic as the kernels' own epilogue: scale, then shift.
__global__ __launch_bounds__(256) void conv_pack_bn_kernel(const float* __restrict__ gamma, const float* __restrict__ beta,
                                                           const float* __restrict__ mean, const float* __restrict__ var,
                                                           float eps, float* __restrict__ out, int K)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= K) return;
    const float scale = gamma[k] / sqrtf(var[k] + eps);
    out[k] = scale;
    out[K + k] = beta[k] - mean[k] * scale;
}

}  // namespace

double conv2d_estimate_us(const ConvArgs& call, size_t* workspace, PackOrder* pack)
{
    *workspace = 0;
    ConvArgs a = call;
    a.x = a.w = a.wpack = nullptr;
    IgemmPlan p;
    plan_igemm(a, &p);
    packed_floats(a, p, &pack->tile, &pack->channels);
    ConvRoute r;
    if (p.variant < 0) return describe_conv2d_stem(a, &r) ? 0. : 1.05 * conv2d_gather_estimate_us(a, workspace);
    int wp;
    const double rounds = (double)(((int64_t)p.g.tiles_m * p.g.tiles_n + 255) / 256);
    switch (p.variant) {
        // (within 10 % of 60 layers of 16 to 512 channels)
        case 0: return split_patch(a, p.g, 512, &wp) ? 2.0 + rounds * (4.5 + a.C / 16 * 5.8) : 2.0 + rounds * (4.0 + 0.445 * a.C);
        case 1: return split_patch(a, p.g, 1024, &wp) ? 2.0 + rounds * (4.0 + a.C / 16 * 3.75) : 2.0 + rounds * (4.0 + 0.24 * a.C);
        case 4: return wide_us(a, p);
        default: return 1.1 * fp32_us(a, p.g, p.variant);
    }
}

bool conv2d_igemm_takes(const ConvArgs& a)
{
    IgemmPlan p;
    plan_igemm(a, &p);
    return p.variant >= 0;
}

bool describe_conv2d_igemm(const ConvArgs& a, ConvRoute* r)
{
    IgemmPlan p;
    plan_igemm(a, &p);
    if (p.variant < 0) return false;
    static const int kTileM[5] = {224, 224, 128, 64, 224}, kTileN[5] = {64, 32, 64, 64, 64};
    r->kernel = 1;
    r->tile_m = kTileM[p.variant];
    r->tile_n = kTileN[p.variant];
    r->ksplit = 1;
    r->wave_groups = 1;
    r->work_groups = p.g.tiles_m * p.g.tiles_n;
    r->workspace_bytes = 0;
    return true;
}

void describe_conv2d(const ConvArgs& a, ConvRoute* r)
{
    if (describe_conv2d_igemm(a, r) || describe_conv2d_pointwise(a, r) || describe_conv2d_pointwise_gemm(a, r) || describe_conv2d_stem(a, r) || describe_conv2d_gather(a, r))
        return;
    *r = ConvRoute{5, 0, 0, 1, 1, 0, 0};
}

hipError_t launch_conv2d_igemm(const ConvArgs& a, hipStream_t stream, bool* taken)
{
    IgemmPlan p;
    plan_igemm(a, &p);
    *taken = p.variant >= 0;
    return *taken ? launch_igemm_plan(a, p, stream) : hipSuccess;
}

size_t conv2d_fast_workspace_bytes(const ConvArgs& a)
{
    const size_t pieces = conv2d_pieces_workspace_bytes(a);
    return pieces ? pieces : conv2d_workspace_bytes(a);
}

size_t conv2d_workspace_bytes(const ConvArgs& a)
{
    if (conv2d_igemm_takes(a)) return 0;
    ConvRoute r;
    if (describe_conv2d_pointwise(a, &r) || describe_conv2d_pointwise_gemm(a, &r) || describe_conv2d_stem(a, &r)) return 0;
    return conv2d_gather_workspace_bytes(a);
}

ConvPackLayout conv2d_pack_layout(const ConvArgs& a)
{
    ConvPackLayout l{};
    l.ss_floats = ((size_t)2 * a.K + 63) / 64 * 64;
    // the plan for aligned pointers, whatever a.x and a.w hold at pack time
    ConvArgs b = a;
    b.x = nullptr;
    b.w = nullptr;
    b.wpack = nullptr;
    IgemmPlan p;
    plan_igemm(b, &p);
    int bn = 0, ck = 0;
    const int64_t pf = packed_floats(b, p, &bn, &ck);
    l.patch_layout = pf > 0 && pf < ((int64_t)1 << 30);
    l.w_floats = l.patch_layout ? (size_t)pf : (size_t)a.K * (a.C / a.groups) * a.R * a.S;
    return l;
}

hipError_t launch_conv2d_pack(const ConvArgs& a, float* pack, hipStream_t stream)
{
    const ConvPackLayout l = conv2d_pack_layout(a);
    if (a.gamma) {
        hipError_t e = launch_kernel(conv_pack_bn_kernel, dim3((unsigned)((a.K + 255) / 256)), dim3(256), 0, stream, a.gamma,
                                     a.beta, a.mean, a.var, a.eps, pack, a.K);
        if (e != hipSuccess) return e;
    }
    float* wout = pack + l.ss_floats;
    const int64_t total = (int64_t)l.w_floats;
    const dim3 grid((unsigned)((total + 255) / 256));
    if (!l.patch_layout) return launch_kernel(conv_pack_copy_kernel, grid, dim3(256), 0, stream, a.w, wout, total);
    ConvArgs b = a;
    b.x = nullptr;
    b.w = nullptr;
    IgemmPlan p;
    plan_igemm(b, &p);
    int bn = 0, ck = 0;
    packed_floats(b, p, &bn, &ck);
    return launch_kernel(conv_pack_patch_kernel, grid, dim3(256), 0, stream, a.w, wout, a.K, a.C, bn, ck, total);
}

hipError_t launch_conv2d(const ConvArgs& a, hipStream_t stream, int* ws_fault)
{
    *ws_fault = 0;
    bool taken = false;
    hipError_t err = launch_conv2d_pieces(a, stream, &taken);
    if (taken || err != hipSuccess) return err;
    err = launch_conv2d_igemm(a, stream, &taken);
    if (taken || err != hipSuccess) return err;
    err = launch_conv2d_pointwise(a, stream, &taken);
    if (taken || err != hipSuccess) return err;
    err = launch_conv2d_pointwise_gemm(a, stream, &taken);
    if (taken || err != hipSuccess) return err;
    err = launch_conv2d_stem(a, stream, &taken);
    if (taken || err != hipSuccess) return err;
    err = launch_conv2d_gather(a, stream, &taken, ws_fault);
    if (taken || err != hipSuccess) return err;
    return launch_conv2d_direct(a, stream);
}

}  // namespace anr
