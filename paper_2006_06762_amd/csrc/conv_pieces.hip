// Planning and launch of the general convolution on pieces made once per call (kernels and their description in
// conv_pieces_kernel.h).
#include "conv_pieces_kernel.h"

namespace anr {
namespace {

using cpieces::BP;
using cpieces::Pieces;
using gconv::Plan;

struct Variant {
    int channels, groups;     // tile, groups of waves
    int resident;             // work-groups per CU (two waves per SIMD)
    double round_us;          // a step of each group, waves alone on their SIMDs or in pairs
    double step_us;           // a CU's matrix time of a step of 4 waves once several work-groups fill it
};
// (four groups of 64 channels, eight waves at one barrier, were never the best by more than 4 %)
constexpr Variant kVariants[] = {{64, 1, 4, 0.281, 0.319}, {64, 2, 2, 0.333, 0.319}, {32, 1, 8, 0.33, 0.462}, {32, 4, 2, 0.617, 0.462}};
constexpr int kSplits[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32};
constexpr double kMostBytes = 256e6;         // of workspace

constexpr int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Estimated time of both kernels (and the third, where the reduction is split): the split pass by its bytes, the products by
// the longer of a work-group's chain of rounds and a CU's work, the stores, the partial tiles.  Fitted to 1900 times of
// 470 layers (3 x 3 to 7 x 7, batch 1 to 32), 8 % rms.
double estimate_us(const ConvArgs& a, const Plan& g, int cg8, int steps, const Variant& v, int ks)
{
    const int64_t per_split = ceil_div(steps, ks), splits = ceil_div(steps, per_split), rounds = ceil_div(per_split, v.groups);
    const int64_t column_tiles = g.groups * ceil_div(g.Kg, v.channels), tiles = ceil_div(g.Mtot, BP) * column_tiles;
    const double per_cu = (double)ceil_div(tiles * splits, 256);
    const double operands = (double)a.N * g.groups * cg8 * 8 * a.H * a.W + (double)column_tiles * v.channels * steps * 16;
    const double chain = ceil_div((int64_t)per_cu, v.resident) * (rounds * v.round_us + 1.22);
    const double work = per_cu * (v.channels / 32 * v.groups / 4. * rounds * v.step_us + 0.22);
    const double longer = chain > work ? chain : work, ratio = (chain > work ? work : chain) / longer, r2 = ratio * ratio;
    double us = 8.5 + operands * 10 / 4.6e6 + longer * (1. + r2 * r2 * r2 / 8) + 4. * g.Mtot * a.K / 3.6e6 * (g.ohow % 4 ? 1.4 : 1.);
    if (splits > 1) us += 0.75 + 2. * 4. * splits * tiles * BP * v.channels / 3.4e6;
    return us;
}

size_t partial_bytes(const Plan& g) { return g.ksplit > 1 ? sizeof(float) * (size_t)g.ksplit * g.Kpad * g.Mpad : 0; }

// The plan of a call and the bytes of workspace with which it is taken; false where the kernels do not take it or another one
// is faster.  Depends on the descriptor alone, not on pointers (but for the general route's choice between two kernels), so
// packed, unpacked and unaligned calls of a layer add the same products in the same order.
bool plan(const ConvArgs& a, Plan* g, Pieces* z, const Variant** variant, PackOrder* pack, size_t* bytes)
{
    const int RS = a.R * a.S;
    // (below 0.4 GFLOP two launches and the split pass are as long as the whole layer on any kernel)
    if (a.route == 1 || RS < 9 || RS > cpieces::kMaxTaps || 2. * a.N * a.OH * a.OW * a.K * (a.C / a.groups) * RS < 0.4e9) return false;
    if (a.route == 2) {       // where the library's choice is a patch kernel, the caller asks for the general kernel in its place
        ConvArgs b = a;
        b.route = 0;
        if (conv2d_igemm_takes(b)) return false;
    }
    if (!gconv::make_plan(a, g, false)) return false;
    const int cg8 = (g->Cg + 7) / 8, units = cg8 * RS, steps = (units + 1) / 2;
    const double x_units = (double)a.N * g->groups * cg8 * a.H * a.W;
    if (x_units * 48 > kMostBytes || units >= 1 << 24) return false;
    const Variant* best = nullptr;
    int best_ks = 1;
    double best_us = 0;
    for (const Variant& v : kVariants) {
        const int64_t column_tiles = g->groups * ceil_div(g->Kg, v.channels), tiles = ceil_div(g->Mtot, BP) * column_tiles;
        if (x_units * 48 + (double)column_tiles * v.channels * steps * 96 > kMostBytes || tiles >= 1 << 24) continue;
        for (const int ks : kSplits) {
            if (ks > 1 && (ks > steps || tiles * ks > 1600 || x_units * 48 + (double)column_tiles * v.channels * steps * 96 + 4. * ks * tiles * BP * v.channels > kMostBytes)) break;
            const double us = estimate_us(a, *g, cg8, steps, v, ks);
            if (!best || us < best_us) {
                best = &v;
                best_us = us;
                best_ks = ks;
            }
        }
    }
    size_t least;                // that other kernel's workspace
    // Four groups of waves and a split reduction leave a wave few rounds, and what is around those, the groups' meeting in LDS
    // above all, is 1 to 4 us longer than the estimate has it (318 layers; with this 5 % rms, without 9).  Only for the comparison
    // with the other kernel: among the variants it was still the best one where it was taken for that.
    if (best && best->groups == 4 && best_ks > 1) best_us = 0.9 * best_us + 4.0;
    // Both estimates are off by 5 to 10 %.  Of 3500 layers of 0.4 GFLOP and more (3 x 3 to 7 x 7, 16 to 512 channels) whose estimate
    // is below 0.88 of the other kernel's, 18 are slower by more than 3 %, half of them by 5 to 12 (without the line above 46, up to
    // 20: 4 x 256 x 8 x 123 -> 32 19.4 -> 23.3 us); 26 that gain 4 % are not taken for it.  All together run 1.31 times as fast.
    if (!best || best_us > 0.88 * conv2d_estimate_us(a, &least, pack)) return false;
    g->taps = 0;
    g->nchunks = steps;
    gconv::set_tile(a, g, BP, best->channels, best_ks);
    g->nwg = best->groups;
    *z = Pieces{};
    z->cg8 = cg8;
    z->units = units;
    z->steps = steps;
    z->x_units = (int)x_units;
    z->x_groups_of_256 = (z->x_units + 255) / 256;
    z->plane = ((uint32_t)z->x_units * 16 + 127) / 128 * 128;
    z->x_bytes = 3 * z->plane;
    z->w_bytes = (uint32_t)(g->tiles_n * (best->channels / 32)) * (uint32_t)steps * 3072;
    *bytes = partial_bytes(*g) + z->x_bytes + z->w_bytes;
    if (*bytes <= least) *bytes = least + 16;
    *variant = best;
    return true;
}

template <int BC, int NWG>
hipError_t launch_tile(const ConvArgs& a, const Plan& g, const Pieces& z, hipStream_t stream)
{
    using S = cpieces::Shape<BC, NWG>;
    const size_t lds_bytes = S::lds_bytes(g.RS);
    auto kern = cpieces::conv_pieces_kernel<BC, NWG>;
    if (lds_bytes > 48 * 1024) {
        static LdsLimit granted;
        const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), lds_bytes, granted);
        if (e != hipSuccess) return e;
    }
    return launch_kernel(kern, dim3((unsigned)(g.tiles_m * g.tiles_n * g.ksplit)), dim3(S::T * NWG), lds_bytes, stream, a, g, z);
}

}  // namespace

size_t conv2d_pieces_workspace_bytes(const ConvArgs& a)
{
    Plan g;
    Pieces z;
    const Variant* v;
    PackOrder pack;
    size_t bytes;
    return plan(a, &g, &z, &v, &pack, &bytes) ? bytes : 0;
}

hipError_t launch_conv2d_pieces(const ConvArgs& a, hipStream_t stream, bool* taken)
{
    *taken = false;
    Plan g;
    Pieces z;
    const Variant* v;
    PackOrder pack;
    size_t bytes;
    // (less room than the pieces of x alone: not planned; planning takes the host a microsecond or two)
    if (a.ws == nullptr || !is_aligned16(a.ws) || a.ws_bytes < 6. * a.N * a.C * a.H * a.W || !plan(a, &g, &z, &v, &pack, &bytes) || a.ws_bytes < bytes)
        return hipSuccess;
    z.at = reinterpret_cast<char*>(a.ws) + partial_bytes(g);
    z.d_hw = make_fastdiv(a.H * a.W);
    z.d_w = make_fastdiv(a.W);
    z.d_cg8g = make_fastdiv(z.cg8 * g.groups);
    z.d_cg8 = make_fastdiv(z.cg8);
    z.rs_mul = (uint32_t)((((uint64_t)1 << 31) + g.RS - 1) / g.RS);
    if (a.wpack) {
        if (pack.channels != 8) return hipSuccess;
        z.w = a.wpack;
        z.w_tile = pack.tile;
        z.w_row = 8 * g.RS + 4;
        z.w_unit = pack.tile * z.w_row;
        z.w_tile_step = z.cg8 * z.w_unit;
        z.w_in_bytes = 4u * (uint32_t)(ceil_div(a.K, pack.tile) * z.w_tile_step);
    } else {
        z.w = a.w;
        z.w_tile = 1;
        z.w_tile_step = g.Ktot;
        z.w_unit = 8 * g.RS;
        z.w_in_bytes = g.w_bytes;
    }
    *taken = true;
    const unsigned w_groups = 4u * (unsigned)(g.tiles_n * (g.bn / 32) * z.cg8);
    hipError_t e = launch_kernel(cpieces::split_operands_kernel, dim3(w_groups + (unsigned)z.x_groups_of_256), dim3(256), 0, stream, a, g, z);
    if (e != hipSuccess) return e;
    if (v->channels == 64) {
        e = v->groups == 1 ? launch_tile<64, 1>(a, g, z, stream) : launch_tile<64, 2>(a, g, z, stream);
    } else {
        e = v->groups == 1 ? launch_tile<32, 1>(a, g, z, stream) : launch_tile<32, 4>(a, g, z, stream);
    }
    return e != hipSuccess || g.ksplit == 1 ? e : gconv::launch_splitk_reduce(a, g, stream);
}

}  // namespace anr
