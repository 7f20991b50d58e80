// Pieces shared by the row-blocked MXFP4 -> column-wise FP8 kernels (scale alignment and re-quantization): the
// write-out of a finished 256-column tile from LDS to the [K, rows] byte matrix of one expert, ragged ends and
// unaligned rows included; the staging of row scales; the arithmetic of either reading.
#pragma once

#include "mxfp4_device.hpp"

namespace mxfp4 {
namespace fp8col {

typedef short s16x2 __attribute__((ext_vector_type(2)));

// Write the finished tile out of LDS: 16 lanes per k-row, 256 contiguous bytes, 256 lanes.  LDS row
// c*32 + cg is column 8*cg + c of the tile, as 16 slots of 16 bytes, the slot of rows 16*l.. being
// (l + cg) % 16.  Chunk u*256 + tid of the tile is row c*32 + cgx, physical slot tid%16, with
// cgx = tid/16 in the even passes and tid/16 + 16 in the odd ones.
// krow0 = address of k-row 0, byte m0 of the expert's matrix; uniform k-row pointers plus
// one 32-bit lane offset (M <= 2^24).  n_rows = rows of the tile that exist (1..256).
// store_streaming instead of the non-temporal hint: 128 -> 139 us at [65536,7168].  The 256-byte pieces of
// neighbouring tiles are better merged in the caches than written through one by one.
__device__ __forceinline__ void write_tile_out(const u32x4 *s_out, uint8_t *krow0, const uint8_t *out_x, size_t pitch_x,
                                               uint32_t cols, uint32_t n_rows, uint32_t tid)
{
    constexpr int CP = 8, T = 256, HALVES = 2; // columns per lane, lanes, passes per column
    const uint32_t pslot = tid & 15u;
    const uint32_t lslot = (pslot - (tid >> 4)) & 15u; // 16 bytes = rows 16*lslot.. of the tile
    const uint32_t lane_off = (tid >> 4) * 8u * (uint32_t)pitch_x + lslot * 16u;
    // Rows on 64-byte boundaries (always, unless the splits are ragged) leave with non-temporal
    // stores.  The others leave with plain, possibly unaligned vector stores and the L2 merges
    // the pieces of neighbouring tiles: measured with 32 un-padded experts at [61440,7168]
    // 204 us, against 258 us with non-temporal stores and 286 us with the rows realigned in
    // registers (funnel shift of neighbouring 16-byte pieces, every store naturally aligned).
    // A tile's 256-byte piece of a k-row must consist of whole 64-byte segments for the
    // streaming form to pay: 32 experts of 1824 rows (32-byte boundaries) take 184 us with it
    // and about 162 us without, 1856 rows (64-byte boundaries) 142 us with it.
    const bool streaming = ((reinterpret_cast<uintptr_t>(out_x) | pitch_x) & 63u) == 0u;
    // bytes of this lane's 16-byte piece that exist: 16, or fewer at the ragged end of a split
    const uint32_t have = lslot * 16u < n_rows ? min(16u, n_rows - lslot * 16u) : 0u;
    static_for<HALVES>([&](auto oddp) {
        constexpr int odd = decltype(oddp)::value;
        if ((odd * 16u + (tid >> 4)) * 8u < cols && have != 0u) {
            if (have == 16u && streaming) {
#pragma unroll
                for (int c = 0; c < CP; ++c) {
                    uint8_t *dst = krow0 + (size_t)(odd * 128u + c) * pitch_x + lane_off;
                    __builtin_nontemporal_store(s_out[(HALVES * c + odd) * T + tid], reinterpret_cast<u32x4 *>(dst));
                }
            } else if (have == 16u) {
                // any alignment: global memory takes unaligned vector stores
#pragma unroll
                for (int c = 0; c < CP; ++c) {
                    uint8_t *dst = krow0 + (size_t)(odd * 128u + c) * pitch_x + lane_off;
                    *reinterpret_cast<u32x4_unaligned *>(dst) = s_out[(HALVES * c + odd) * T + tid];
                }
            } else {
#pragma nounroll
                for (int c = 0; c < CP; ++c) {
                    uint8_t *dst = krow0 + (size_t)(odd * 128u + c) * pitch_x + lane_off;
                    store_head_bytes(dst, s_out[(HALVES * c + odd) * T + tid], have);
                }
            }
        }
    });
}

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// Row scales of a wave's 64 rows (lane t: the 8 bytes v of row `row`) into LDS, with what the conversions need of them: whether a
// NaN byte (REQUANT: a byte of 253 or more) occurs per (64 rows, k-block), and for scale alignment the maximum of the non-NaN
// bytes over each 16 rows.  ROWS = rows that s_row_sf and s_max16 hold.
template <bool REQUANT, uint32_t STRIDE, uint32_t ROWS>
__device__ __forceinline__ void stage_row_scales(const u32x2 v, uint32_t row, uint32_t lane, uint8_t *s_row_sf, uint8_t *s_flag,
                                                 uint8_t *s_max16)
{
    store_row_scales<STRIDE>(s_row_sf, v, row, lane);
    u32x2 r = v;
    uint32_t flags = 0;
    constexpr uint32_t FROM = REQUANT ? 253u : 255u;
    // one test for the 8 bytes of a row and one ballot for the wave; the rest of it only runs when that fires
    if (__ballot((bytes_from<256u - FROM>(v.x) | bytes_from<256u - FROM>(v.y)) != 0u) != 0ull) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool f = ((v[j >> 2] >> (8 * (j & 3))) & 0xFFu) >= FROM;
            flags |= (__ballot(f) != 0ull ? 1u : 0u) << j;
            if (f)
                r[j >> 2] &= ~(0xFFu << (8 * (j & 3))); // NaN bytes take no part in the maximum
        }
    }
    if (lane < 8u)
        s_flag[(row >> 6) * 8u + lane] = (uint8_t)((flags >> lane) & 1u);
    if (!REQUANT) { // two k-blocks at a time
        uint32_t m[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u16x2 e = __builtin_bit_cast(u16x2, r[h] & 0x00FF00FFu), o = __builtin_bit_cast(u16x2, (r[h] >> 8) & 0x00FF00FFu);
            auto step = [&](auto ctrl) {
                constexpr int c = decltype(ctrl)::value;
                e = __builtin_elementwise_max(e, __builtin_bit_cast(u16x2, dpp_read<c>(__builtin_bit_cast(uint32_t, e))));
                o = __builtin_elementwise_max(o, __builtin_bit_cast(u16x2, dpp_read<c>(__builtin_bit_cast(uint32_t, o))));
            };
            step(std::integral_constant<int, DPP_QUAD_XOR1>{});
            step(std::integral_constant<int, DPP_QUAD_XOR2>{});
            step(std::integral_constant<int, DPP_ROW_HALF_MIRROR>{});
            step(std::integral_constant<int, DPP_ROW_MIRROR>{});
            m[h] = __builtin_bit_cast(uint32_t, e) | __builtin_bit_cast(uint32_t, o) << 8;
        }
        const uint32_t j = lane & 15u; // lane j of a row of 16 stores k-block j
        if (j < 8u)
            s_max16[j * (ROWS / 16u) + (row >> 4)] = (uint8_t)((j < 4u ? m[0] : m[1]) >> (8u * (j & 3u)));
    }
}

// ---- scale alignment

// Decode-scale operand of row I of a slice: exponent field max(127 - (bmax - b_I), 0) in bits
// 30:23, computed as a signed value so that one max() does the clamp.
template <int I>
__device__ __forceinline__ float row_shift_operand(const uint32_t (&sb)[8], int bias_minus_bmax)
{
    const int b = (int)((sb[I >> 2] >> (8 * (I & 3))) & 0xFFu);
    return u2f((uint32_t)max((int)((uint32_t)(b + bias_minus_bmax) << 23), 0));
}

// Maximum of the 8 bytes at p (8-byte aligned, LDS).
__device__ __forceinline__ uint32_t max_of_8_bytes(const uint8_t *p)
{
    const u32x2 v = *reinterpret_cast<const u32x2 *>(p);
    const uint32_t t = max(max(v.x & 0xFFu, (v.x >> 8) & 0xFFu), max((v.x >> 16) & 0xFFu, v.x >> 24));
    const uint32_t u = max(max(v.y & 0xFFu, (v.y >> 8) & 0xFFu), max((v.y >> 16) & 0xFFu, v.y >> 24));
    return max(t, u);
}

// ---- re-quantization

// Emax = biased exponent of a non-zero column maximum, plus one (FP32 subnormals: 2^-127 and
// 1.5 * 2^-127 give 1, 2^-128 gives 0).
__device__ __forceinline__ int emax_of_amax_bits(uint32_t bits)
{
    const int ef = (int)(bits >> 23);
    return ef >= 1 ? ef + 1 : (bits >= 0x00400000u ? 1 : 0);
}

// FP32 bit pattern of the group scale 2^(Emax - 136) (an FP32 subnormal for Emax <= 9); 1.0 for
// a group without a non-zero element.
__device__ __forceinline__ uint32_t scale_bits_of_emax(int emax, bool any_nonzero)
{
    if (!any_nonzero)
        return 0x3F800000u;
    const int field = emax - 9;
    return field >= 1 ? (uint32_t)field << 23 : 0x00400000u >> (uint32_t)(-field);
}

// The integer path.  Column kc of the tile over the rows [r0, r0 + n) of the tile (one scale
// group): Emax over the non-zero codes of the rows whose scale byte is not NaN, or -1 without
// any, plus GROUP_HAS_NAN when a NaN byte occurs.  Nibbles come from global memory, scale bytes
// from the staged copy.
constexpr int GROUP_HAS_NAN = 1 << 16;
[[maybe_unused]] static __device__ __noinline__ int group_emax_int(const uint8_t *tile_src, size_t pitch, const uint8_t *row_sf_kb,
                                           uint32_t kc, uint32_t r0, uint32_t n)
{
    int emax = -1;
    bool any_nan = false;
#pragma nounroll
    for (uint32_t r = r0; r < r0 + n; ++r) {
        const uint32_t b = row_sf_kb[r];
        const uint32_t byte = tile_src[(size_t)r * pitch + (kc >> 1)];
        const uint32_t mag = ((kc & 1u) ? byte >> 4 : byte) & 7u;
        if (b == 255u)
            any_nan = true;
        else if (mag)
            emax = max(emax, (int)b + (int)(mag >> 1));
    }
    return emax + (any_nan ? GROUP_HAS_NAN : 0);
}

// E4M3 byte of +-e2m1(nib) * 2^(b - 127) / 2^(emax - 136) in integers.  With h = 2 * |e2m1| the
// quotient is h * 2^(b - emax + 17) quanta of 2^-9 (the E4M3 subnormal step): an exact integer n
// when the shift is not negative, else rounded to nearest-even; n < 16 is its own code
// (subnormals and the first binade), above that the binade is the position of the leading bit.
__device__ __forceinline__ uint32_t e4m3_requant_int(uint32_t nib, uint32_t b, int emax)
{
    const uint32_t mag = nib & 7u, sign = (nib & 8u) << 4;
    const uint32_t h = mag < 4u ? mag : mag == 4u ? 4u : mag == 5u ? 6u : mag == 6u ? 8u : 12u;
    if (mag == 0u)
        return sign;
    const int sh = (int)b - emax + 17;
    uint32_t n;
    if (sh >= 0) {
        n = h << sh;
    } else if (sh < -5) {
        n = 0;
    } else {
        const uint32_t t = (uint32_t)(-sh), q = h >> t, rem = h & ((1u << t) - 1u), half = 1u << (t - 1u);
        n = q + ((rem > half || (rem == half && (q & 1u))) ? 1u : 0u);
    }
    if (n < 16u)
        return sign | n;
    const uint32_t p = 31u - (uint32_t)__builtin_clz(n);
    return sign | ((p - 2u) << 3) | ((n >> (p - 3u)) & 7u);
}

} // namespace fp8col
} // namespace mxfp4
