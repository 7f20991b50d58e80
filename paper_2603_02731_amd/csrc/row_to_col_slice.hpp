// Shared by the two MXFP4 row -> column kernels: a 32-row slice of 8 columns, through the hardware conversions or in integers.
#pragma once

#include "mxfp4_device.hpp"

namespace mxfp4 {

// One lane's 32x8 slice through the hardware conversions, in two steps with the column scales between them
// (the workgroup sends the scale bytes off before it re-quantizes).  Exact while every value
// e2m1 * 2^(b-127) is an FP32 number, i.e. for row-scale bytes up to 252
// (6 * 2^125 < 2^128; the smallest, 0.5 * 2^-127, is an FP32 subnormal).
// Step 1: the UE8M0 bytes of the slice's 8 columns.
__device__ __forceinline__ void column_scales_hw(const uint32_t (&w)[32], const uint32_t (&sb)[8], uint32_t (&cb)[8])
{
    // column maxima of |value| (no NaN can occur: NaN row scales never get here)
    float amax[8];
#pragma unroll
    for (int c = 0; c < 8; ++c)
        amax[c] = 0.0f;
    static_for<16>([&](auto ip) {
        constexpr int i = 2 * decltype(ip)::value;
        const float sa = row_scale_operand<i>(sb), sbb = row_scale_operand<i + 1>(sb);
        static_for<4>([&](auto jp) {
            constexpr int j = decltype(jp)::value;
            const f32x2 fa = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i], sa, j);
            const f32x2 fb = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i + 1], sbb, j);
            amax[2 * j] = max3_abs_nan(fa.x, fb.x, amax[2 * j]);
            amax[2 * j + 1] = max3_abs_nan(fa.y, fb.y, amax[2 * j + 1]);
        });
    });
    // the sec. 3.1 rule on the exponent field.  A maximum with at most two significant bits (1.0 or 1.5
    // times a power of two) never exceeds 1.5 * 2^e, so the byte is its exponent field minus 2, clamped
    // at 0; zero and FP32 subnormals give 0.
#pragma unroll
    for (int c = 0; c < 8; ++c)
        cb[c] = max(f2u(amax[c]) >> 23, 2u) - 2u;
}

// Step 2 for the columns of the NJ nibble bytes from J0 on: decode again (cheaper than keeping 256 floats live) and re-quantize
// pairs of rows into output bytes: v_cvt_scalef32_pk_fp4_f32 takes rows (m, m+1) of one column.
template <int J0, int NJ>
__device__ __forceinline__ void requant_columns_hw(const uint32_t (&w)[32], const uint32_t (&sb)[8], const uint32_t (&cb)[8],
                                                   uint32_t (&o)[2 * NJ][4])
{
    float cs[2 * NJ];
#pragma unroll
    for (int c = 0; c < 2 * NJ; ++c)
        cs[c] = u2f(cb[2 * J0 + c] << 23);
#pragma unroll
    for (int c = 0; c < 2 * NJ; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            asm volatile("" : "=v"(o[c][g])); // no initial value needed: all four bytes are written
    static_for<16>([&](auto ip) {
        constexpr int i = 2 * decltype(ip)::value;
        constexpr int g = i >> 3, sel = (i >> 1) & 3; // output dword and byte of rows (i, i+1)
        const float sa = row_scale_operand<i>(sb), sbb = row_scale_operand<i + 1>(sb);
        static_for<NJ>([&](auto jp) {
            constexpr int jl = decltype(jp)::value, j = J0 + jl;
            const f32x2 fa = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i], sa, j);
            const f32x2 fb = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i + 1], sbb, j);
            o[2 * jl][g] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(o[2 * jl][g], fa.x, fb.x, cs[2 * jl], sel);
            o[2 * jl + 1][g] =
                __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(o[2 * jl + 1][g], fa.y, fb.y, cs[2 * jl + 1], sel);
        });
    });
}

// One column (c of the dwords at src) of the same slice in integers, for row-scale bytes 253 and 254, whose largest values
// (4 and 6 times 2^126 or 2^127) exceed FP32, and for NaN.  Never taken by real activations, so it is
// written for size, not speed: rolled loops that re-read the nibbles (they are still in
// cache) and the staged row scales.  Only the first n_valid rows of the slice exist (fewer than 32 at the ragged end of a split).
// Every non-zero E2M1 value is (1 + M/2) * 2^(E-1) with the pair (E, M) = (field, mantissa),
// except the subnormal 0.5 = 1.0 * 2^-1, i.e. (0, 0).  With at most two significant bits,
// ceil(log2(x/6)) = floor(log2 x) - 2, so the column byte is max(0, max(b_row + E) - 3); 255 where a row scale is NaN.
__device__ __forceinline__ uint32_t column_byte_int(const uint8_t *src, size_t src_pitch, const uint8_t *row_sf, int c, int n_valid)
{
    int emax = -1024;
    bool nan = false;
#pragma nounroll
    for (int i = 0; i < n_valid; ++i) {
        const uint32_t wi = *reinterpret_cast<const uint32_t *>(src + (size_t)i * src_pitch);
        const int mag = (int)(wi >> (4 * c)) & 7;
        nan |= row_sf[i] == 255u;
        if (mag)
            emax = max(emax, (int)row_sf[i] + (mag >> 1));
    }
    return nan ? 255u : (uint32_t)max(0, emax - 3);
}

// Its 32 codes relative to that byte: t = 2*(b_row + E - b_col) + M orders the values; t >= 2 are E2M1 normals
// and stay exact (code t), and below that RTNE gives t = 1 -> 1.0 (tie .75, even code 2),
// t = 0 and -1 -> 0.5 (code 1), t = -2 -> 0 (tie .25), lower -> 0.
__device__ __forceinline__ void column_codes_int(const uint8_t *src, size_t src_pitch, const uint8_t *row_sf, int c, int n_valid,
                                                 uint32_t bc, uint32_t *out)
{
#pragma nounroll
    for (int g = 0; g < 4; ++g) {
        uint32_t acc = 0;
#pragma nounroll
        for (int i8 = 0; i8 < 8; ++i8) {
            const int i = g * 8 + i8;
            if (i >= n_valid || bc == 255u)
                break; // the nibbles of rows that do not exist, and of a column with a NaN, stay 0
            const uint32_t wi = *reinterpret_cast<const uint32_t *>(src + (size_t)i * src_pitch);
            const uint32_t nib = (wi >> (4 * c)) & 0xFu;
            const int mag = (int)(nib & 7u);
            const int em = mag == 1 ? 0 : mag; // 2*E + M of the normalised value
            const int t2 = max(em + 2 * ((int)row_sf[i] - (int)bc) + 2, 0);
            int code = min(7, max(t2 - 2, (t2 + 1) >> 1));
            code = mag ? code : 0;
            acc |= ((nib & 8u) | (uint32_t)code) << (4 * i8);
        }
        out[g] = acc;
    }
}

} // namespace mxfp4
