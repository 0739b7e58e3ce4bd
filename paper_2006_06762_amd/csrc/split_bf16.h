// fp32 products on the bf16 matrix pipes without giving up fp32 accuracy.
//
// gfx950 multiplies fp32 matrices at 157 TFLOP/s and bf16 ones at 2.5 PFLOP/s.  A float is the exact
// sum of three bf16 numbers, x = h + m + l (24 significant bits in three pieces of eight, each rounded to
// nearest, so m is at most 2^-8 and l at most 2^-17 of the leading bit of x), and a product of two floats
// is then the sum of the nine products of their pieces, each exact in fp32.  Eight of them are formed; ll,
// the ninth, is at most 2^-34 of the product.  (Six, without ml and lm, would leave out up to 2^-24 of the
// product: as much again as rounding it to fp32.)
//
// v_mfma_f32_32x32x16_bf16 adds the sixteen products of an instruction to the accumulator with one rounding.
// The seven small products, 2^-8 of hh and less, go to an accumulator of their own, so that the large sum is
// rounded once per sixteen k where the fp32 instruction rounds once per two: a single non-zero term comes out
// as one fp32 rounding of the product (measured 1.004 units of 2^-24 at most, the fp32 instruction 1.000; one
// accumulator for all products and six of them 4.99), sums of 1024 terms of one sign 2.6 units rms against
// 7.2, of random sign 0.12 against 0.40.  Denormal inputs and results are kept by the instruction (measured).
//
// Three kinds of value do not survive the split, and all are detected:
//   - magnitudes below 2^-110, whose last piece needs bits under the smallest bf16 denormal: l is the
//     difference of floats, so it is exact, and it is representable if and only if its low 16 bits
//     are zero; `lost` collects them;
//   - infinities, NaN and magnitudes that round to infinity in bf16: a piece of theirs is infinite or
//     NaN, so every accumulator they reach is not finite;
//   - sums below 2^-118 other than zero: there the roundings of the small products, at 2^-150, are no longer
//     small beside that of the result.
// A work-group that meets one recomputes its tile with the fp32 instruction.
#pragma once
#include "anr_device.h"

namespace anr {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// v_mfma_f32_32x32x16_bf16: D(32x32) += A(32x16) * B(16x32).  Lane l supplies A[i = l%32][k = 8*(l/32) + 0..7]
// and B[the same k][j = l%32]; the accumulator layout is that of mfma32.
__device__ __forceinline__ f32x16 mfma_bf16(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Two floats rounded to bf16 (nearest, ties to even), the first in the low half.
__device__ __forceinline__ uint32_t pack_bf16(float x, float y)
{
    const f32x2 v = {x, y};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// The pieces of two floats, packed; `lost` as described above.
__device__ __forceinline__ void split2(float x0, float x1, uint32_t& h, uint32_t& m, uint32_t& l, uint32_t& lost)
{
    h = pack_bf16(x0, x1);
    const float r0 = x0 - __builtin_bit_cast(float, h << 16);
    const float r1 = x1 - __builtin_bit_cast(float, h & 0xffff0000u);
    m = pack_bf16(r0, r1);
    const uint32_t l0 = __builtin_bit_cast(uint32_t, r0 - __builtin_bit_cast(float, m << 16));
    const uint32_t l1 = __builtin_bit_cast(uint32_t, r1 - __builtin_bit_cast(float, m & 0xffff0000u));
    l = __builtin_amdgcn_perm(l1, l0, 0x07060302u);
    lost |= l0 | l1;
}

// The products, smallest first: pieces of the two operands (0 h, 1 m, 2 l).  The last one is the large one.
constexpr int kProducts = 8;
constexpr int kPieceA[kProducts] = {1, 2, 0, 2, 1, 0, 1, 0};
constexpr int kPieceB[kProducts] = {2, 1, 2, 0, 1, 1, 0, 0};

__device__ __forceinline__ bool lost_bits(uint32_t lost) { return (lost & 0xffffu) != 0; }

// The bits that tell whether accumulators can be kept: start from {}, check every one, ask once.
struct SumCheck {
    float not_finite = 0.f;                // NaN once a register is infinite or NaN
    uint32_t smallest = 0xffffffffu;       // smallest magnitude other than zero, as 2 * bits - 1

    __device__ __forceinline__ void check(const f32x16& a)
    {
        bool small = false;                // or zero: most tiles have neither, and a comparison is half of what the exact answer costs
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float sum = a[r];        // (a copy: the compiler's bit cast of a vector's element takes the first one whatever its index)
            not_finite = fmaf(sum, 0.f, not_finite);
            small = small || fabsf(sum) < 0x1p-118f;
        }
        if (__any(small)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float sum = a[r];
                smallest = min(smallest, (__builtin_bit_cast(uint32_t, sum) << 1) - 1u);
            }
        }
    }
    __device__ __forceinline__ bool refused() const
    {
        constexpr uint32_t kSmall = (uint32_t)(127 - 118) << 23;      // 2^-118
        return not_finite != 0.f || smallest < (kSmall << 1) - 1u;
    }
};

}  // namespace anr
