// Host-only arithmetic of the patch-staging convolution's plan (conv_igemm_kernel.h).
#pragma once
#include <stdint.h>

namespace anr {
namespace igemm {

// Largest number of virtual rows that any tile of `bm` consecutive pixels of the N x OH x OW output needs (R rows per
// output row, output rows stride_h apart, images hv rows apart).  What a whole tile needs depends only on where in an image
// it starts, m0 mod OH*OW, and that repeats after OH*OW / gcd(bm, OH*OW) tiles; the clipped last tile needs no more than
// a whole one at the same start.  So one period is scanned, not every tile of a large batch, and its first and last pixel
// are moved along without divisions: four variants are planned for each call, several hundred tiles each on large maps
// (7 x 132 x 132: 28 us of a call with divisions).
inline int max_virtual_rows(int N, int OH, int OW, int stride_h, int R, int bm, int hv)
{
    struct Pixel {
        int64_t n;
        int oh, ow;
    };
    const int64_t ohow = (int64_t)OH * OW, total = N * ohow;
    auto at = [&](int64_t m) { return Pixel{m / ohow, (int)(m % ohow / OW), (int)(m % OW)}; };
    int64_t x = bm, y = ohow;
    while (y) { const int64_t t = x % y; x = y; y = t; }
    const int64_t period = ohow / x;                      // tiles until the start offset repeats
    const int64_t tiles = (total + bm - 1) / bm;
    const int64_t scan = tiles < period ? tiles : period;
    const Pixel step = at(bm);
    Pixel first = at(0), last = at(bm - 1);
    auto move = [&](Pixel& p) {
        p.n += step.n;
        p.oh += step.oh;
        p.ow += step.ow;
        if (p.ow >= OW) {
            p.ow -= OW;
            ++p.oh;
        }
        if (p.oh >= OH) {
            p.oh -= OH;
            ++p.n;
        }
    };
    int64_t most = 0;
    for (int64_t t = 0; t < scan; ++t) {
        if (t == tiles - 1) last = at(total - 1);
        const int64_t rows = (last.n - first.n) * hv + (int64_t)(last.oh - first.oh) * stride_h;
        if (rows > most) most = rows;
        move(first);
        move(last);
    }
    return (int)most + R;
}

}  // namespace igemm
}  // namespace anr
