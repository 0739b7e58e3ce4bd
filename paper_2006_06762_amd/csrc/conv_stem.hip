// Convolutions of images with two or three channels and 7 x 7 kernels, stride 1 or 2 (the stem of an image
// network: 224x224x3, 7x7, stride 2), fp32 as three bf16 pieces (split_bf16.h).
//
// With three channels there is nothing to put side by side along k but the kernel row: a unit of eight k
// is one kernel row of one channel (its S <= 8 taps, zero weights beyond), and the operand of a pixel is
// eight consecutive columns of the input, so the input patch is staged once, as rows of bf16, and every
// kernel row reads it at another offset.  A work-group keeps all weights of its 64 output channels in LDS,
// split once, and walks pixel tiles of 16 x 16, two at a time: eight waves to a tile, each 2 rows of 16
// pixels x 64 channels.  The next tile's patch travels to registers while a tile is multiplied.  (One tile
// at a time with two patch buffers fits the LDS as well; with half the waves it took 44 us instead of 36
// for 224x224x3, 7x7, stride 2, batch 16.)  Rows of the result are channels and columns pixels: a store
// writes whole 64-byte runs.
//
// Kernel rows of a channel are padded to an even number (two units make one matrix instruction): 7 x 7
// does 8 x 8 / 49 = 1.3 times the products, at twice the fp32 rate.  Bound: half of a work-group's time is
// staging and stores, which its two barriers a round keep apart from the products.  Batch 16: 224x224x3 -> 64,
// stride 2, 48.2 -> 46.0 us, stride 1 160 -> 134; 128 channels 87 -> 80, 96 at batch 32 163 -> 133.
#include <type_traits>

#include "conv_internal.h"
#include "split_bf16.h"

namespace anr {
namespace stem {

constexpr uint32_t kPastExtent = 0x80000000u;       // byte offset beyond any descriptor extent
constexpr int TP = 16;                  // tile edge, pixels
constexpr int T = 512;                  // threads of a tile
constexpr int G = 2;                    // tiles a work-group has in hand
constexpr int kMaxC = 3;

template <int R_, int ST>
struct Shape {
    static constexpr int RP = (R_ + 1) / 2 * 2;                     // kernel rows, padded
    static constexpr int PR = (TP - 1) * ST + RP;                   // patch rows
    static constexpr int PW = ((TP - 1) * ST + 8 + 3) / 4 * 4;      // patch columns: whole quads
    static constexpr int PLANE = kMaxC * PR * PW * 2;               // bytes of a piece
    static constexpr int XBUF = 3 * PLANE;
    static constexpr int WUNITS = kMaxC * RP;
    static constexpr int WPLANE = WUNITS * 64 * 16;
    static constexpr int QUADS = PR * (PW / 4);                     // staging quads per channel
    static constexpr int SLOTS = (kMaxC * QUADS + T - 1) / T;       // per thread
    static constexpr size_t lds_bytes = 3 * WPLANE + G * XBUF + 2 * 64 * sizeof(float) + 4 * sizeof(int);
};

struct Geom {
    int tiles_x, tiles_y, tiles, per_n;        // pixel tiles; work-groups that share a channel tile's pixel tiles
    uint32_t x_bytes, w_bytes;
    FastDiv d_x, d_y;
};

template <int R_, int ST>
__global__ __launch_bounds__(T * G) void conv_stem_kernel(const ConvArgs p, const Geom g)
{
    using D = Shape<R_, ST>;
    extern __shared__ __attribute__((aligned(16))) char slds[];
    char* const lw = slds;                                                     // weights [piece][unit][64 channels]
    char* const lx = slds + 3 * D::WPLANE;                                     // patches [G][piece][channel][row][column]
    float* const lbn = reinterpret_cast<float*>(lx + G * D::XBUF);             // scale[64], shift[64]
    int* const flag = reinterpret_cast<int*>(lbn + 128);                       // tile whose patch lost bits [G]; weights did

    const int grp = __builtin_amdgcn_readfirstlane((int)threadIdx.x / T);
    const int tid = (int)threadIdx.x % T, lane = tid & 63, wave = tid >> 6;
    const int r32 = lane & 31, h = lane >> 5;
    const int tile_n = (int)blockIdx.x / g.per_n, first = (int)blockIdx.x - tile_n * g.per_n;
    const int co0 = tile_n * 64;
    const int C = p.C;

    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.x), 0, (int)g.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.w), 0, (int)g.w_bytes, 0x00020000);

    // staging slot j of this thread: quad of columns 4*sq .. of patch row sr of channel sc; slots of channels
    // past the last have a row that no image holds
    int sr[D::SLOTS], sq[D::SLOTS], soff[D::SLOTS], sdst[D::SLOTS];
#pragma unroll
    for (int j = 0; j < D::SLOTS; ++j) {
        const int i = tid + T * j;
        const int sc = i / D::QUADS, rem = i - sc * D::QUADS;
        sr[j] = rem / (D::PW / 4);
        sq[j] = 4 * (rem - sr[j] * (D::PW / 4));
        soff[j] = sc * (int)p.xs[1] + sr[j] * (int)p.xs[2] + sq[j];
        sdst[j] = sc < kMaxC ? ((sc * D::PR + sr[j]) * D::PW + sq[j]) * 2 : -1;
        if (sc >= C) sr[j] = 1 << 30;
    }
    float rx[D::SLOTS][4];
    auto origin = [&](int t, int& n, int& oh0, int& ow0) {
        const int row = g.d_x.div(t);
        n = g.d_y.div(row);
        oh0 = (row - n * g.tiles_y) * TP;
        ow0 = (t - row * g.tiles_x) * TP;
    };
    auto load_patch = [&](int t) {
        int n, oh0, ow0;
        origin(t, n, oh0, ow0);
        const int ih0 = oh0 * ST - p.pad_h, iw0 = ow0 * ST - p.pad_w;
        const int base0 = (int)(n * p.xs[0] + ih0 * p.xs[2]) + iw0;
#pragma unroll
        for (int j = 0; j < D::SLOTS; ++j) {
            // rows outside the image read zero
            const int iw = iw0 + sq[j];
            const bool row_ok = (unsigned)(ih0 + sr[j]) < (unsigned)p.H;
            const int base = base0 + soff[j];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool ok = row_ok & ((unsigned)(iw + e) < (unsigned)p.W);
                rx[j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xrsrc, (int)((uint32_t)(4 * (base + e)) | (ok ? 0u : kPastExtent)), 0, 0));
            }
        }
    };
    auto store_patch = [&](int t) {
        uint32_t lost = 0;
#pragma unroll
        for (int j = 0; j < D::SLOTS; ++j) {
            u32x2 s[3];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                uint32_t hh, mm, ll;
                split2(rx[j][2 * e], rx[j][2 * e + 1], hh, mm, ll, lost);
                s[0][e] = hh; s[1][e] = mm; s[2][e] = ll;
            }
            if (sdst[j] >= 0) {
                char* d = lx + grp * D::XBUF + sdst[j];
#pragma unroll
                for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x2*>(d + q * D::PLANE) = s[q];
            }
        }
        if (lost_bits(lost)) flag[grp] = t;
    };

    if (threadIdx.x < G + 1) flag[threadIdx.x] = -1;
    if (threadIdx.x < 64) {
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
        lbn[64 + tid] = shift;
    }
    // tile of round i: first + (G*i + grp) * per_n; past the end there is nothing to multiply
    auto tile_of = [&](int i) { return first + (G * i + grp) * g.per_n; };
    load_patch(min(tile_of(0), g.tiles - 1));
    __syncthreads();                                 // the flags are set
    auto load_weights = [&](int i, uint32_t (&w)[8]) {
        const int unit = i >> 6, co = co0 + (i & 63), c = unit / D::RP, r = unit - c * D::RP;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const bool ok = (s < R_) & (r < R_) & (c < C) & (co < p.K);
            w[s] = __builtin_amdgcn_raw_buffer_load_b32(wrsrc, (int)((uint32_t)(4 * ((co * C + c) * R_ * R_ + r * R_ + s)) | (ok ? 0u : kPastExtent)), 0, 0);
        }
    };
    {
        uint32_t lost = 0;
        bool huge = false;
        for (int i = threadIdx.x; i < D::WUNITS * 64; i += T * G) {
            uint32_t w[8];
            load_weights(i, w);
            u32x4 s[3];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t hh, mm, ll;
                split2(__builtin_bit_cast(float, w[2 * e]), __builtin_bit_cast(float, w[2 * e + 1]), hh, mm, ll, lost);
                s[0][e] = hh; s[1][e] = mm; s[2][e] = ll;
                huge |= (w[2 * e] << 1) > 0xfefe0000u || (w[2 * e + 1] << 1) > 0xfefe0000u;      // above the largest bf16
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(lw + q * D::WPLANE + i * 16) = s[q];
        }
        if (lost_bits(lost) || huge) flag[G] = 1;
    }
    // Weights the pieces cannot carry: as floats in their place, the halves of the word in the first two planes
    __syncthreads();
    const bool whole_weights = flag[G] == 1;
    if (whole_weights) {
        for (int i = threadIdx.x; i < D::WUNITS * 64; i += T * G) {
            uint32_t w[8];
            load_weights(i, w);
            *reinterpret_cast<u32x4*>(lw + i * 16) = u32x4{w[0] >> 16 | (w[1] & 0xffff0000u), w[2] >> 16 | (w[3] & 0xffff0000u),
                                                           w[4] >> 16 | (w[5] & 0xffff0000u), w[6] >> 16 | (w[7] & 0xffff0000u)};
            *reinterpret_cast<u32x4*>(lw + D::WPLANE + i * 16) = u32x4{(w[0] & 0xffffu) | w[1] << 16, (w[2] & 0xffffu) | w[3] << 16,
                                                                       (w[4] & 0xffffu) | w[5] << 16, (w[6] & 0xffffu) | w[7] << 16};
        }
    }

    const int py = 2 * wave + (r32 >> 4), px = r32 & 15;
    const char* const wl = lw + (h * 64 + r32) * 16;
    const int xoff = ((py * ST + h) * D::PW + (ST == 1 ? px & ~1 : 2 * px)) * 2;
    const uint32_t odd = ST == 1 ? 16u * (px & 1) : 0u;       // a pixel in an odd column starts in the middle of a word
    for (int i = 0; first + G * i * g.per_n < g.tiles; ++i) {
        const int t = tile_of(i);
        store_patch(t);
        __syncthreads();
        load_patch(min(tile_of(i + 1), g.tiles - 1));
        // keep the loads ahead of the matrix instructions
        __builtin_amdgcn_sched_barrier(0);
        if (t < g.tiles) {
            // the products of the first pieces, and the other seven
            f32x16 acc[2], low[2];
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[cb][r] = low[cb][r] = 0.f;
            for (int c = 0; c < C; ++c) {
                const char* wc = wl + c * D::RP * 1024;
                const char* xc = lx + grp * D::XBUF + xoff + c * D::PR * D::PW * 2;
#pragma unroll
                for (int j = 0; j < D::RP / 2; ++j) {
                    u32x4 xv[3];
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const uint32_t* s = reinterpret_cast<const uint32_t*>(xc + q * D::PLANE + 2 * j * D::PW * 2);
                        if (ST == 1) {
                            uint32_t d[5];
#pragma unroll
                            for (int e = 0; e < 5; ++e) d[e] = s[e];
#pragma unroll
                            for (int e = 0; e < 4; ++e) xv[q][e] = __builtin_amdgcn_alignbit(d[e + 1], d[e], odd);
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e) xv[q][e] = s[e];
                        }
                    }
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) {
                        u32x4 wv[3];
#pragma unroll
                        for (int q = 0; q < 3; ++q) wv[q] = *reinterpret_cast<const u32x4*>(wc + q * D::WPLANE + 2 * j * 1024 + cb * 512);
#pragma unroll
                        for (int i = 0; i < kProducts; ++i) {
                            f32x16& sum = i < kProducts - 1 ? low[cb] : acc[cb];
                            sum = mfma_bf16(wv[kPieceA[i]], xv[kPieceB[i]], sum);
                        }
                    }
                }
            }
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[cb][r] += low[cb][r];
            int n, oh0, ow0;
            origin(t, n, oh0, ow0);
            const int oh = oh0 + py, ow = ow0 + px;
            SumCheck sums;
            sums.check(acc[0]);
            sums.check(acc[1]);
            if (whole_weights || flag[grp] == t || __any(sums.refused())) {
                // Values the pieces cannot carry: the wave's block again with the fp32 instruction.  Its half h supplies
                // the input channels c with c % 2 == h; inputs come straight from memory, a kernel row's in flight at a
                // time, weights are the sums of their pieces (exact) or the floats themselves.  In every tile that is
                // 2.3 times an ordinary call (with weights from memory as well 3.8).
                int l = lane;
                asm("" : "+v"(l));               // nothing of this is held through the ordinary rounds
                const int hc = l >> 5;
                const char* const wbase = lw + (l & 31) * 16;
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[cb][r] = 0.f;
                const int iw = min(ow, p.OW - 1) * ST - p.pad_w, ih0 = min(oh, p.OH - 1) * ST - p.pad_h;
                for (int c0 = 0; c0 < C; c0 += 2) {
                    const int c = min(c0 + hc, C - 1);
                    const uint32_t past = c0 + hc < C ? 0u : kPastExtent;
                    const int xc = (int)(n * p.xs[0] + c * p.xs[1]) + iw;
#pragma unroll 1
                    for (int r = 0; r < R_; ++r) {
                        const uint32_t row = ((unsigned)(ih0 + r) < (unsigned)p.H ? 0u : kPastExtent) | past;
                        float x[R_];
#pragma unroll
                        for (int s = 0; s < R_; ++s) {
                            const uint32_t ok = (unsigned)(iw + s) < (unsigned)p.W ? row : kPastExtent;
                            x[s] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xrsrc, (int)((uint32_t)(4 * (xc + (ih0 + r) * (int)p.xs[2] + s)) | ok), 0, 0));
                        }
#pragma unroll
                        for (int cb = 0; cb < 2; ++cb) {
                            u32x4 w[3];
#pragma unroll
                            for (int q = 0; q < 3; ++q) w[q] = *reinterpret_cast<const u32x4*>(wbase + q * D::WPLANE + ((c * D::RP + r) * 64 + 32 * cb) * 16);
#pragma unroll
                            for (int s = 0; s < R_; ++s) {
                                uint32_t b[3];
#pragma unroll
                                for (int q = 0; q < 3; ++q) b[q] = s % 2 ? w[q][s / 2] & 0xffff0000u : w[q][s / 2] << 16;
                                const float sum = (__builtin_bit_cast(float, b[0]) + __builtin_bit_cast(float, b[1])) + __builtin_bit_cast(float, b[2]);
                                const float v = whole_weights ? __builtin_bit_cast(float, b[0] | b[1] >> 16) : sum;
                                acc[cb] = mfma32(v, x[s], acc[cb]);
                            }
                        }
                    }
                }
                // once more, so that their registers are free for this
                load_patch(min(tile_of(i + 1), g.tiles - 1));
            }
            // register r of lane (h, r32): channel 8*(r/4) + 4*h + r%4 of the block, pixel r32
            if (p.gamma) {
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int ch = 32 * cb + 8 * (r / 4) + (r % 4) + 4 * h;
                        acc[cb][r] = fmaxf(fmaf(acc[cb][r], lbn[ch], lbn[64 + ch]), 0.f);
                    }
            }
            if (oh < p.OH && ow < p.OW) {
                // uniform row of channels, the lane's part of the offset in 32 bits
                const uint32_t off = (uint32_t)(4 * h * (int)p.ys[1] + oh * (int)p.ys[2] + ow);
                float* const y = p.y + n * p.ys[0] + co0 * p.ys[1];
                auto store = [&](auto whole_c) {
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int ch = 32 * cb + 8 * (r / 4) + (r % 4);
                            if (decltype(whole_c)::value || co0 + ch + 4 * h < p.K) (y + ch * p.ys[1])[off] = acc[cb][r];
                        }
                };
                if (co0 + 64 <= p.K) store(std::true_type{});
                else store(std::false_type{});
            }
        }
        __syncthreads();
    }
}

}  // namespace stem

namespace {

using namespace stem;

// Where it is the faster one: 7 x 7 (5 x 5 pads 25 taps to 48: 11.8 against 12.9 us for 64x64x3 -> 64 at batch
// 16), two or three channels (with one there is too little to multiply per store: 16.2 against 18.7 us for
// 112x112x1 -> 64 at batch 32), a channel tile at least three quarters full, and of the 512 tiles that the chip
// has in hand at a time enough that are there: a round takes what the gather kernel does 370 tiles in (stride 2:
// 256 tiles 21.2 against 17.9 us, 392 27.9 against 27.8, 784 46.2 against 48.2, 1568 80 against 87; stride 1:
// 3136 132 against 160).
constexpr int kCUs = 256;
constexpr int kTilesWorthARound = 380;

bool plan_stem(const ConvArgs& a, Geom* g)
{
    if (a.groups != 1 || a.C < 2 || a.C > kMaxC || a.dil_h != 1 || a.dil_w != 1 || a.R != 7 || a.S != 7) return false;
    if (a.stride_h != a.stride_w || a.stride_h > 2 || a.route == 1) return false;
    const int64_t x_extent = (int64_t)(a.N - 1) * a.xs[0] + (int64_t)(a.C - 1) * a.xs[1] + (int64_t)(a.H - 1) * a.xs[2] + a.W;
    const int64_t w_extent = (int64_t)a.K * a.C * a.R * a.S;
    if (x_extent >= ((int64_t)1 << 29) || w_extent >= ((int64_t)1 << 29)) return false;
    g->tiles_x = (a.OW + TP - 1) / TP;
    g->tiles_y = (a.OH + TP - 1) / TP;
    const int64_t tiles = (int64_t)g->tiles_x * g->tiles_y * a.N;
    const int tiles_n = (a.K + 63) / 64;
    if (4 * a.K < 3 * 64 * tiles_n) return false;
    // (the lane's part of an output offset is 32 bits)
    if (a.ys[1] >= ((int64_t)1 << 27) || a.ys[2] >= ((int64_t)1 << 16) || a.ys[2] * a.OH >= ((int64_t)1 << 30)) return false;
    if (tiles >= ((int64_t)1 << 30)) return false;
    // half-empty tiles (14 x 14 and smaller maps leave a quarter and more of a tile unused)
    if ((double)a.OH * a.OW < 0.7 * g->tiles_x * g->tiles_y * TP * TP) return false;
    g->tiles = (int)tiles;
    // no more work-groups than CUs: each takes a CU's LDS, one too many would wait for a whole round
    g->per_n = tiles_n < kCUs ? kCUs / tiles_n : 1;
    if (g->per_n > g->tiles) g->per_n = g->tiles;
    const int64_t rounds = (tiles + G * g->per_n - 1) / (G * g->per_n);
    if (tiles * tiles_n < rounds * kTilesWorthARound) return false;
    g->x_bytes = (uint32_t)(4 * x_extent);
    g->w_bytes = (uint32_t)(4 * w_extent);
    g->d_x = make_fastdiv(g->tiles_x);
    g->d_y = make_fastdiv(g->tiles_y);
    return true;
}

template <int R_, int ST>
hipError_t launch_stem(const ConvArgs& a, const Geom& g, hipStream_t stream)
{
    auto kern = conv_stem_kernel<R_, ST>;
    static LdsLimit granted;
    const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), Shape<R_, ST>::lds_bytes, granted);
    if (e != hipSuccess) return e;
    return launch_kernel(kern, dim3((unsigned)(g.per_n * ((a.K + 63) / 64))), dim3(T * G), Shape<R_, ST>::lds_bytes, stream, a, g);
}

}  // namespace

bool describe_conv2d_stem(const ConvArgs& a, ConvRoute* r)
{
    Geom g;
    if (!plan_stem(a, &g)) return false;
    *r = ConvRoute{3, TP * TP, 64, 1, 1, g.per_n * ((a.K + 63) / 64), 0};
    return true;
}

hipError_t launch_conv2d_stem(const ConvArgs& a, hipStream_t stream, bool* taken)
{
    Geom g;
    *taken = plan_stem(a, &g);
    if (!*taken) return hipSuccess;
    return a.stride_h == 2 ? launch_stem<7, 2>(a, g, stream) : launch_stem<7, 1>(a, g, stream);
}

}  // namespace anr
