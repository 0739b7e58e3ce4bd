// Launch logic of the TBS batch matmul (kernel in tbg_kernel.h): the tile kernel when the
// operands allow 16-byte loads, the general batched GEMM otherwise.
#include "tbg_kernel.h"

namespace anr {
namespace {

template <int UT, int KB>
hipError_t launch_tbs_rows32(const tbg::Args& t0, int batch, int vec_store, hipStream_t stream)
{
    using T = tbg::TbsShape<KB>;
    tbg::Args t = t0;
    const int ld = (t.D < tbg::kChunk ? t.D : tbg::kChunk) + 4;     // the panel in LDS is one chunk wide
    t.tiles_i = (t.S + T::rows_q - 1) / T::rows_q;
    const int64_t items = (int64_t)batch * t.tiles_i;
    t.xcd_chunk = (items % 8 == 0) ? (int)(items / 8) : 0;
    // q rows, then the k panel, which the staged probabilities (rows_q x ldp) later overwrite
    const size_t kpanel = (size_t)T::rows_k * ld, probs = (size_t)T::rows_q * T::ldp;
    const size_t lds_bytes = sizeof(float) * ((size_t)T::rows_q * ld + (kpanel > probs ? kpanel : probs));
    t.d_tiles_i = make_fastdiv(t.tiles_i);
    t.d_h = make_fastdiv(t.H);
    // the whole form: S is exactly the keys of KB blocks and whole blocks of queries, D whole
    // chunks, 32-bit byte offsets inside one (b, h) view
    constexpr bool whole_ut = UT == (T::rows_q + T::rows_k) / 16;
    const bool whole = whole_ut && t.S == T::rows_k && (t.S % T::rows_q == 0) && (t.D % tbg::kChunk == 0) &&
                       (int64_t)(t.S - 1) * t.qs_s + t.D < ((int64_t)1 << 29) &&
                       (int64_t)(t.S - 1) * t.ks_s + t.D < ((int64_t)1 << 29) &&
                       (int64_t)(t.S - 1) * t.os_i + t.S < ((int64_t)1 << 29);
    constexpr int UTW = (T::rows_q + T::rows_k) / 16;
    auto kern = whole ? tbg::tbs_rows32_kernel<UTW, true, KB, true> : tbg::tbs_rows32_kernel<UT, true, KB, false>;
    if (lds_bytes > 48 * 1024) {
        static LdsLimit granted[2];    // one per kernel form
        hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), lds_bytes, granted[whole ? 1 : 0]);
        if (e != hipSuccess) return e;
    }
    return launch_kernel(kern, dim3((unsigned)items), dim3(256), lds_bytes, stream, t, ld, vec_store);
}

// UT for D <= 32 / more is (rows_q + rows_k) * (chunk/4) / 256 rounded up: 160 rows for KB = 4
// and 1, 128 rows for KB = 2; the chunk is at most 64 columns.
template <int KB>
hipError_t launch_tbs_by_d(const tbg::Args& t, int batch, int vec_store, hipStream_t stream)
{
    constexpr int rows = tbg::TbsShape<KB>::rows_q + tbg::TbsShape<KB>::rows_k;
    if (t.D <= 32) return launch_tbs_rows32<(rows * 8 + 255) / 256, KB>(t, batch, vec_store, stream);
    return launch_tbs_rows32<(rows * 16 + 255) / 256, KB>(t, batch, vec_store, stream);
}

template <int KW, int KBW>
hipError_t launch_tbs_long(const tbg::Args& t0, int batch, int vec_store, hipStream_t stream)
{
    tbg::Args t = t0;
    t.tiles_i = (t.S + 31) / 32;
    const int64_t items = (int64_t)batch * t.tiles_i;
    t.xcd_chunk = (items % 8 == 0) ? (int)(items / 8) : 0;
    t.d_tiles_i = make_fastdiv(t.tiles_i);
    t.d_h = make_fastdiv(t.H);
    const size_t lds_bytes = sizeof(float) * tbg::long_lds_floats<KW>(t.D);
    auto kern = tbg::tbs_long_kernel<KW, KBW>;
    if (lds_bytes > 48 * 1024) {
        static LdsLimit granted;
        hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), lds_bytes, granted);
        if (e != hipSuccess) return e;
    }
    return launch_kernel(kern, dim3((unsigned)items), dim3(64 * KW), lds_bytes, stream, t, vec_store);
}

}  // namespace

hipError_t launch_tbg(const GemmArgs& a, hipStream_t stream)
{
    // a describes out[z] = A[z] . B[z]^T with z = (b, h): see GemmArgs
    const bool fast = a.b_is_nk && a.M == a.N && (a.K % 4 == 0) && is_aligned16(a.A) && is_aligned16(a.B) &&
                      (a.lda % 4 == 0) && (a.ldb % 4 == 0) && (a.sAo % 4 == 0) && (a.sAi % 4 == 0) &&
                      (a.sBo % 4 == 0) && (a.sBi % 4 == 0);
    const int tiles = (a.M + tbg::kTile - 1) / tbg::kTile;
    const int64_t blocks = (int64_t)a.batch * tiles * tiles;
    const bool fused = a.softmax_rows && a.M <= tbg::kMaxKeys && a.K <= 1024 && (a.K % 8 == 0);
    const bool offsets32 = (int64_t)(a.M - 1) * a.lda + a.K < ((int64_t)1 << 29) && (int64_t)(a.N - 1) * a.ldb + a.K < ((int64_t)1 << 29);
    // whole tiles, whole chunks and 32-bit byte offsets inside one (b, h) view: the lean form
    const bool whole = (a.M % tbg::kTile == 0) && (a.K % tbg::kChunk == 0) && offsets32 &&
                       (int64_t)(a.M - 1) * a.ldc + a.N < ((int64_t)1 << 29);
    // Enough 128 x 128 tiles to fill the chip twice, mostly full: the bf16-split GEMM (32 x 12 heads of 512 x
    // 512 x 128 231 -> 200 us, 16 x 12 of 200 x 200 x 80 36 -> 26).  With fewer or half-empty tiles the kernels
    // below are the faster ones (8 x 8 of 312 x 312 x 64 15.0 against 16.5 us), and so they are with a single
    // chunk in the lean form (24 x 8 of 256 x 256 x 64 18.4 against 20.6, 48 x 8 of 512 x 512 x 64 129.7 against
    // 128.7).  The fused softmax keeps its sizes.
    const int64_t tiles128 = (a.M + 127) / 128;
    const bool split = a.M > tbg::kMaxKeys && !fused && offsets32 && tiles128 * tiles128 * a.batch >= 512 &&
                       (double)a.M * a.M >= 0.6 * tiles128 * tiles128 * 128 * 128 && (double)a.M * a.M * a.batch >= 384.0 * 128 * 128 &&
                       (a.K >= 48 || a.M % tbg::kTile == 0) && !(whole && a.K <= tbg::kChunk);
    // What is left with a softmax and up to 512 keys: one kernel that keeps the scores on the chip (16 x 16 heads, two
    // kernels / one: 160 x 160 x 64 52 / 28 us, 256 x 256 x 64 74 / 42, 481 x 481 x 32 193 / 131, 512 x 512 x 64 198 /
    // 158).  The split GEMM keeps its sizes: its scores are the closer ones, and those tbg gives for them.  A
    // work-group walks the keys in a row, so with few work-groups and a long walk the two kernels are faster (8 heads of
    // 300 x 300 x 128 11.1 / 16.1, x 64 9.8 / 10.4, x 32 9.7 / 8.5; 12 heads of 492 x 492 x 128 19.4 / 21.9, 16 of 400 x
    // 400 x 128 23.8 / 21.0), and so they are for wide heads with a third of the last keys missing (64 of 300 x 300 x 128
    // 39.0 / 41.7).
    const int64_t long_items = (int64_t)a.batch * ((a.M + 31) / 32);
    const int long_chunks = (a.M + 127) / 128;
    const bool long_pays = (long_items > (a.K > 96 ? 200 : 160) || long_chunks * a.K <= 128) && !(a.K > 96 && long_chunks == 3 && long_items < 1024);
    const bool rows_long = long_pays && !split && a.softmax_rows && a.M > tbg::kMaxKeys && a.M <= tbg::kLongKeys &&
                           a.K <= tbg::kLongD && (a.K % 8 == 0) && offsets32;
    if (!fast || split || blocks >= ((int64_t)1 << 31)) {
        GemmArgs g = a;
        return launch_gemm(g, stream);
    }
    tbg::Args t{};
    t.q = a.A; t.k = a.B; t.out = a.C;
    t.S = a.M; t.D = a.K; t.H = a.batch_inner;
    t.qs_b = a.sAo; t.qs_s = a.lda; t.qs_h = a.sAi;
    t.ks_b = a.sBo; t.ks_s = a.ldb; t.ks_h = a.sBi;
    t.os_b = a.sCo; t.os_h = a.sCi; t.os_i = a.ldc;
    t.tiles_i = tiles; t.tiles_j = tiles;
    t.xcd_chunk = (blocks % 8 == 0) ? (int)(blocks / 8) : 0;
    if (fused) {
        // fused TBS: a block of query rows x all keys per work-group
        const int vec_store = is_aligned16(a.C) && (a.ldc % 4 == 0) && (a.sCo % 4 == 0) && (a.sCi % 4 == 0);
        if (a.M <= 32) return launch_tbs_by_d<1>(t, a.batch, vec_store, stream);
        if (a.M <= 64) return launch_tbs_by_d<2>(t, a.batch, vec_store, stream);
        return launch_tbs_by_d<4>(t, a.batch, vec_store, stream);
    }
    if (rows_long) {
        // 1: rows of 16-byte units, 2: and every store a whole line (see stg4_nt)
        const bool units = is_aligned16(a.C) && (a.ldc % 4 == 0) && (a.sCo % 4 == 0) && (a.sCi % 4 == 0);
        const bool lines = units && (reinterpret_cast<uintptr_t>(a.C) & 127) == 0 && (a.ldc % 32 == 0) && (a.sCo % 32 == 0) && (a.sCi % 32 == 0);
        const int vec_store = lines ? 2 : units ? 1 : 0;
        if (t.S <= 256) return launch_tbs_long<4, 2>(t, a.batch, vec_store, stream);
        if (t.S <= 384) return launch_tbs_long<4, 3>(t, a.batch, vec_store, stream);
        return launch_tbs_long<4, 4>(t, a.batch, vec_store, stream);
    }
    t.d_tiles_j = make_fastdiv(t.tiles_j);
    t.d_tiles_i = make_fastdiv(t.tiles_i);
    t.d_h = make_fastdiv(t.H);
    hipError_t err = whole ? launch_kernel(tbg::tbg_tile64_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, t)
                           : launch_kernel(tbg::tbg_tile_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, t);
    if (err != hipSuccess || !a.softmax_rows) return err;
    return launch_softmax_rows(a, stream);
}

}  // namespace anr
