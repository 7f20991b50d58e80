// Row-blocked MXFP4 -> column-blocked MXFP4 or column-wise FP8 of one small matrix, gfx950.
//
// The conversions of row_to_col.hip, row_to_fp8_col.hip and row_to_fp8_col_requant.hip for launches that do not fill the chip, which
// last as long as one workgroup does: load, convert, turn round in LDS, store.  Here a lane takes 8 rows x 8 columns, a quarter of the
// 32 x 8 slice of those kernels (the quarters of a slice in a quad of lanes, which exchange column maxima by DPP), a workgroup 128 x 128
// elements, and there are four times as many of them.  MXFP4 needs one barrier, scale alignment two, re-quantization three.
// Calls in a HIP graph, us (tiles of 256 x 256 / here): row->col [128,7168] 5.3 / 3.0, [2048,2048] 5.8 / 3.6; alignment 5.3 / 3.1 and
// 6.3 / 3.7, re-quantization 6.1 / 4.2 and 6.9 / 4.8; of either about 2 are the launch.  A byte load per row scale instead of a dword
// per row turned round in LDS 3.2 and 3.8, nibbles through LDS by 16-byte loads 3.2 and 3.8.
// What a tile costs beside its elements (addresses, half lines, scales four or one at a time) is four times as much too, so where
// workgroups queue up this is up to twice as slow ([4096,7168] 9.6 / 12.7): col_in_small_tiles.
#include "fp8_col_tile.hpp"
#include "mxfp4_device.hpp"
#include "mxfp4_kernels.hpp"

namespace mxfp4 {
namespace col_small {

using namespace fp8col;

constexpr uint32_t THREADS = 256, TILE = 128;

struct Args {
    const uint8_t *q_row;
    const uint8_t *sf_row;
    uint8_t *out;
    void *out_sf; // bytes (MXFP4) or floats
    uint32_t M, K;
    uint32_t tiles_m, tiles_k;
};

template <class T, class F>
__device__ __forceinline__ T quad_reduce(T v, F &&f)
{
    v = f(v, __builtin_bit_cast(T, dpp_read<DPP_QUAD_XOR1>(__builtin_bit_cast(uint32_t, v))));
    return f(v, __builtin_bit_cast(T, dpp_read<DPP_QUAD_XOR2>(__builtin_bit_cast(uint32_t, v))));
}

// Scale operand of a UE8M0 byte.
__device__ __forceinline__ float scale_operand(uint32_t b) { return u2f(b << 23); }

} // namespace col_small

using namespace col_small;

template <ColKind KIND>
__global__ void __launch_bounds__(THREADS) col_small_kernel(const col_small::Args a)
{
    // The tile's output: column 8 cg + c is LDS row c * 16 + cg, so that what the lanes of a wave write at once lies on different banks.
    constexpr uint32_t BYTES = KIND == COL_MXFP4 ? TILE / 2u : TILE, ROW = BYTES + 16u;
    __shared__ alignas(16) uint8_t s_out[TILE * ROW];
    __shared__ alignas(4) uint8_t s_sf[KIND == COL_MXFP4 ? TILE : 1][4]; // [LDS row][32 rows]: scales
    __shared__ alignas(8) uint8_t s_row_sf[4][4][32];                    // [32 rows][k-block][row]
    __shared__ uint16_t s_max[4][4]; // [32 rows][k-block]: largest scale byte that is not NaN; bit 8: one of FROM or more, 9: a NaN
    __shared__ alignas(16) uint32_t s_amax[KIND == COL_REQUANT ? 4 : 1][TILE]; // [32 rows][column]: bits of the largest |value|, or Emax + 1

    const uint32_t tile_k = blockIdx.x % a.tiles_k, tile_m = blockIdx.x / a.tiles_k;
    const uint32_t m0 = tile_m * TILE, k0 = tile_k * TILE;
    const uint32_t n_rg = min(4u, (a.M - m0) / 32u); // whole blocks of 32 rows; all four for FP8
    const uint32_t tid = threadIdx.x;
    const uint32_t sub = tid & 3u, cg = tid >> 2 & 15u, rg = tid >> 6; // rows 32 rg + 8 sub, columns 8 cg of the tile
    const uint32_t pitch = a.K / 2u, Kb = a.K / 32u, kb = cg >> 2;

    // ---- the lane's 8 x 8 elements and its 8 row-scale bytes
    uint32_t w[8], b[8];
    {
        const uint32_t row0 = rg < n_rg ? rg * 32u : 0u; // past the end: any rows, not stored
        const uint8_t *src = a.q_row + (size_t)m0 * pitch + k0 / 2u;
        const uint32_t lane = tid & 63u;
        uint32_t sf = 0;
        if (lane < 32u)
            sf = *reinterpret_cast<const uint32_t *>(a.sf_row + (size_t)m0 * Kb + k0 / 32u + (row0 + lane) * Kb);
        // uniform row pointers plus a 32-bit lane offset (K is at most 2^24)
        const uint32_t at = (row0 + sub * 8u) * pitch + cg * 4u;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            w[i] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(src + (size_t)i * pitch + at));
        // four rows' bytes of four k-blocks, turned round in the quad
        uint32_t t = perm(dpp_read<DPP_QUAD_XOR1>(sf), sf, (lane & 1u) ? 0x03070105u : 0x06020400u);
        t = perm(dpp_read<DPP_QUAD_XOR2>(t), t, (lane & 2u) ? 0x03020706u : 0x05040100u);
        if (lane < 32u)
            *reinterpret_cast<uint32_t *>(&s_row_sf[rg][lane & 3u][lane & ~3u]) = t;
        wave_fence();
        const u32x2 bytes = *reinterpret_cast<const u32x2 *>(&s_row_sf[rg][kb][sub * 8u]);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            b[i] = bytes[i >> 2] >> (8 * (i & 3)) & 0xFFu;
    }
    uint32_t largest = 0; // of the scale bytes
#pragma unroll
    for (int i = 0; i < 8; ++i)
        largest = max(largest, b[i]);

    if (KIND == COL_MXFP4) {
        largest = quad_reduce(largest, [](uint32_t x, uint32_t y) { return max(x, y); });
        uint32_t cb[8], o[8];
        if (largest < 253u) {
            float amax[8];
#pragma unroll
            for (int c = 0; c < 8; ++c)
                amax[c] = 0.0f;
            static_for<4>([&](auto ip) {
                constexpr int i = 2 * decltype(ip)::value;
                static_for<4>([&](auto jp) {
                    constexpr int j = decltype(jp)::value;
                    const f32x2 fa = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i], scale_operand(b[i]), j);
                    const f32x2 fb = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i + 1], scale_operand(b[i + 1]), j);
                    amax[2 * j] = max3_abs_nan(fa.x, fb.x, amax[2 * j]);
                    amax[2 * j + 1] = max3_abs_nan(fa.y, fb.y, amax[2 * j + 1]);
                });
            });
#pragma unroll
            for (int c = 0; c < 8; ++c) { // one 32-row block: the quad.  The rule as in column_scales_hw
                const float m = quad_reduce(amax[c], [](float x, float y) { return __builtin_elementwise_maximum(x, y); });
                cb[c] = max(f2u(m) >> 23, 2u) - 2u;
                asm volatile("" : "=v"(o[c])); // no initial value needed: all four bytes are written
            }
            static_for<4>([&](auto ip) {
                constexpr int sel = decltype(ip)::value, i = 2 * sel;
                static_for<4>([&](auto jp) {
                    constexpr int j = decltype(jp)::value;
                    const f32x2 fa = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i], scale_operand(b[i]), j);
                    const f32x2 fb = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i + 1], scale_operand(b[i + 1]), j);
                    o[2 * j] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(o[2 * j], fa.x, fb.x, scale_operand(cb[2 * j]), sel);
                    o[2 * j + 1] =
                        __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(o[2 * j + 1], fa.y, fb.y, scale_operand(cb[2 * j + 1]), sel);
                });
            });
        } else {
            // values beyond FP32, or NaN: in integers, as column_byte_int and column_codes_int
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                int emax = -1024;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int mag = (int)(w[i] >> (4 * c)) & 7;
                    emax = mag ? max(emax, (int)b[i] + (mag >> 1)) : emax;
                }
                emax = quad_reduce(emax, [](int x, int y) { return max(x, y); });
                cb[c] = largest == 255u ? 255u : (uint32_t)max(0, emax - 3);
                o[c] = 0u;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint32_t nib = (w[i] >> (4 * c)) & 0xFu;
                    const int mag = (int)(nib & 7u), em = mag == 1 ? 0 : mag;
                    const int t2 = max(em + 2 * ((int)b[i] - (int)cb[c]) + 2, 0);
                    const int code = mag ? min(7, max(t2 - 2, (t2 + 1) >> 1)) : 0;
                    if (largest != 255u)
                        o[c] |= ((nib & 8u) | (uint32_t)code) << (4 * i);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < 8; ++c)
            *reinterpret_cast<uint32_t *>(s_out + (c * 16u + cg) * ROW + rg * 16u + sub * 4u) = o[c];
        if (sub == 0u) {
#pragma unroll
            for (int c = 0; c < 8; ++c)
                s_sf[c * 16u + cg][rg] = (uint8_t)cb[c];
        }
    } else {
        auto out_scale = [&](uint32_t column, uint32_t bits) {
            static_cast<uint32_t *>(a.out_sf)[(size_t)(k0 + column) * a.tiles_m + tile_m] = bits;
        };
        // ---- the scale group's largest scale byte, NaN apart, and whether a byte of FROM or more occurs
        constexpr uint32_t FROM = KIND == COL_ALIGN ? 255u : 253u;
        uint32_t finite = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            finite = max(finite, b[i] == 255u ? 0u : b[i]);
        finite = quad_reduce(finite, [](uint32_t x, uint32_t y) { return max(x, y); });
        const uint32_t any = quad_reduce((largest >= FROM ? 1u : 0u) | (largest == 255u ? 2u : 0u),
                                         [](uint32_t x, uint32_t y) { return x | y; });
        if (sub == 0u && (cg & 3u) == 0u)
            s_max[rg][kb] = (uint16_t)(finite | any << 8);
        __syncthreads();
                    uint32_t bmax = 0, flags = 0;
#pragma unroll
        for (uint32_t g = 0; g < 4u; ++g) {
            const uint32_t m = s_max[g][kb];
            bmax = max(bmax, m & 0xFFu);
            flags |= m >> 8;
        }
        const uint32_t scales = rg * 4u + sub; // lanes 0 to 7 that share 8 columns store a column's scale each
        uint32_t o[8][2];
        if (KIND == COL_ALIGN) {
            if (scales < 8u) {
                const int e = (int)bmax - 6; // biased exponent of 2^(max - 6 - 127); below 1: an FP32 subnormal
                const uint32_t bits = flags ? 0x7FC00000u : e >= 1 ? (uint32_t)e << 23 : 0x00400000u >> (uint32_t)(-e);
                out_scale(cg * 8u + scales, bits);
            }
            float dsc[8];
            const float enc = u2f(121u << 23); // the encoder divides by 2^-6: Algorithm 1's delta
            uint32_t nan[2] = {0u, 0u};
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                dsc[i] = u2f((uint32_t)max((int)((b[i] + 127u - bmax) << 23), 0));
                nan[i >> 2] |= b[i] == 255u ? 0xFFu << (8 * (i & 3)) : 0u;
            }
            static_for<4>([&](auto jp) {
                constexpr int j = decltype(jp)::value;
                static_for<2>([&](auto rp) {
                    constexpr int r = decltype(rp)::value;
                    const f32x2 f0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[4 * r], dsc[4 * r], j);
                    const f32x2 f1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[4 * r + 1], dsc[4 * r + 1], j);
                    const f32x2 f2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[4 * r + 2], dsc[4 * r + 2], j);
                    const f32x2 f3 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[4 * r + 3], dsc[4 * r + 3], j);
                    s16x2 e0, e1; // no initial value needed: both words are written
                    asm volatile("" : "=v"(e0), "=v"(e1));
                    e0 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(e0, f0.x, f1.x, enc, false);
                    e0 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(e0, f2.x, f3.x, enc, true);
                    e1 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(e1, f0.y, f1.y, enc, false);
                    e1 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(e1, f2.y, f3.y, enc, true);
                    // rows under a NaN scale byte are NaN
                    o[2 * j][r] = (__builtin_bit_cast(uint32_t, e0) & ~nan[r]) | (0x7F7F7F7Fu & nan[r]);
                    o[2 * j + 1][r] = (__builtin_bit_cast(uint32_t, e1) & ~nan[r]) | (0x7F7F7F7Fu & nan[r]);
                });
            });
        } else {
            // ---- the group's largest value of every column: its FP32 bits, or Emax where those do not do
            uint32_t m[8];
#pragma unroll
            for (int c = 0; c < 8; ++c)
                m[c] = 0u;
            if (flags == 0u) {
                float amax[8];
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    amax[c] = 0.0f;
                static_for<4>([&](auto ip) {
                    constexpr int i = 2 * decltype(ip)::value;
                    static_for<4>([&](auto jp) {
                        constexpr int j = decltype(jp)::value;
                        const f32x2 fa = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i], scale_operand(b[i]), j);
                        const f32x2 fb = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[i + 1], scale_operand(b[i + 1]), j);
                        amax[2 * j] = max3_abs_nan(fa.x, fb.x, amax[2 * j]);
                        amax[2 * j + 1] = max3_abs_nan(fa.y, fb.y, amax[2 * j + 1]);
                    });
                });
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    m[c] = f2u(quad_reduce(amax[c], [](float x, float y) { return __builtin_elementwise_maximum(x, y); }));
            } else {
                // Emax + 1 over the non-zero codes of rows whose scale byte is not NaN, 0 without any
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    uint32_t e = 0;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const uint32_t mag = (w[i] >> (4 * c)) & 7u;
                        e = mag && b[i] != 255u ? max(e, b[i] + (mag >> 1) + 1u) : e;
                    }
                    m[c] = quad_reduce(e, [](uint32_t x, uint32_t y) { return max(x, y); });
                }
            }
            if (sub == 0u) {
                u32x4 *dst = reinterpret_cast<u32x4 *>(s_amax[rg] + cg * 8u);
                dst[0] = u32x4{m[0], m[1], m[2], m[3]};
                dst[1] = u32x4{m[4], m[5], m[6], m[7]};
            }
            __syncthreads();
#pragma unroll
            for (uint32_t g = 0; g < 4u; ++g) {
                const u32x4 *p = reinterpret_cast<const u32x4 *>(s_amax[g] + cg * 8u);
                const u32x4 p0 = p[0], p1 = p[1];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    m[c] = max(m[c], p0[c]); // non-negative floats order like their bit patterns
                    m[4 + c] = max(m[4 + c], p1[c]);
                }
            }
            bool slow = flags != 0u;
            int emax[8];
            float enc[8];
            uint32_t mine = 0; // the scale that this lane stores
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const bool zero = m[c] == 0u;
                emax[c] = flags != 0u ? (int)m[c] - 1 : zero ? -1 : emax_of_amax_bits(m[c]);
                const uint32_t ef = m[c] >> 23;
                slow |= flags == 0u && !zero && ef < 8u; // a maximum below 2^-118: operand exponent negative
                enc[c] = u2f((zero ? 127u : ef - 8u) << 23);
                const uint32_t bits = (flags & 2u) ? 0x7FC00000u : scale_bits_of_emax(emax[c], !zero);
                mine = scales == (uint32_t)c ? bits : mine;
            }
            if (scales < 8u)
                out_scale(cg * 8u + scales, mine);
            if (!slow) {
                static_for<4>([&](auto jp) {
                    constexpr int j = decltype(jp)::value;
                    static_for<2>([&](auto rp) {
                        constexpr int r = decltype(rp)::value;
                        const f32x2 f0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[4 * r], scale_operand(b[4 * r]), j);
                        const f32x2 f1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[4 * r + 1], scale_operand(b[4 * r + 1]), j);
                        const f32x2 f2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[4 * r + 2], scale_operand(b[4 * r + 2]), j);
                        const f32x2 f3 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[4 * r + 3], scale_operand(b[4 * r + 3]), j);
                        s16x2 e0, e1; // no initial value needed: both words are written
                        asm volatile("" : "=v"(e0), "=v"(e1));
                        e0 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(e0, f0.x, f1.x, enc[2 * j], false);
                        e0 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(e0, f2.x, f3.x, enc[2 * j], true);
                        e1 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(e1, f0.y, f1.y, enc[2 * j + 1], false);
                        e1 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(e1, f2.y, f3.y, enc[2 * j + 1], true);
                        o[2 * j][r] = __builtin_bit_cast(uint32_t, e0);
                        o[2 * j + 1][r] = __builtin_bit_cast(uint32_t, e1);
                    });
                });
            } else {
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    o[c][0] = o[c][1] = 0u;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const uint32_t nib = (w[i] >> (4 * c)) & 0xFu;
                        const uint32_t v = b[i] == 255u ? 0x7Fu : e4m3_requant_int(nib, b[i], emax[c]);
                        o[c][i >> 2] |= v << (8 * (i & 3));
                    }
                }
            }
        }
#pragma unroll
        for (int c = 0; c < 8; ++c)
            *reinterpret_cast<u32x2 *>(s_out + (c * 16u + cg) * ROW + rg * 32u + sub * 8u) = u32x2{o[c][0], o[c][1]};
    }
    __syncthreads();

    // ---- out: 16-byte pieces
    constexpr uint32_t PIECES = BYTES / 16u;
    const uint32_t pitch_out = KIND == COL_MXFP4 ? a.M / 2u : a.M;
#pragma unroll
    for (uint32_t u = 0; u < TILE * PIECES / THREADS; ++u) {
        const uint32_t i = u * THREADS + tid, column = i / PIECES, p = i % PIECES;
        if (KIND != COL_MXFP4 || p < n_rg)
            *reinterpret_cast<u32x4 *>(a.out + (size_t)(k0 + column) * pitch_out + (KIND == COL_MXFP4 ? m0 / 2u : m0) + p * 16u) =
                *reinterpret_cast<const u32x4 *>(s_out + ((column & 7u) * 16u + (column >> 3)) * ROW + p * 16u);
    }
    if (KIND == COL_MXFP4 && tid < TILE) {
        const uint32_t pitch_sf = a.M / 32u;
        uint8_t *dst = static_cast<uint8_t *>(a.out_sf) + (size_t)(k0 + tid) * pitch_sf + m0 / 32u;
        const uint32_t v = *reinterpret_cast<const uint32_t *>(s_sf[(tid & 7u) * 16u + (tid >> 3)]);
        if (n_rg == 4u)
            *reinterpret_cast<u32_unaligned *>(dst) = v;
        else
            store_head_bytes(dst, u32x4{v, 0u, 0u, 0u}, n_rg);
    }
}

// Which matrices: two tiles per compute unit, a little more where a tile is shorter work.  On both sides of the lines, 256 compute units
// (us, tiles of 256 x 256 / small ones): row->col 640 tiles 6.40 / 5.59 [5120,2048] and 6.15 / 5.79 [20480,512], 704 tiles 6.42 / 5.77,
// 768 tiles 6.28 / 6.27 and 6.69 / 6.45, 896 tiles 7.19 / 7.50; alignment 576 tiles 6.89 / 6.44 and 6.75 / 6.52, 640 tiles 6.86 / 6.92
// and 7.21 / 6.76, 768 tiles 6.86 / 7.54; re-quantization 512 tiles 7.48 / 6.67 and 7.01 / 6.78, 576 tiles 7.67 / 7.72 and 7.48 / 8.04.
bool col_in_small_tiles(int64_t M, int64_t K, ColKind kind)
{
    const int64_t tiles = (M + TILE - 1) / TILE * (K / TILE), quarters = kind == COL_MXFP4 ? 11 : kind == COL_ALIGN ? 9 : 8;
    return 4 * tiles <= quarters * (int64_t)compute_units();
}

hipError_t launch_col_small(const uint8_t *q_row, const uint8_t *sf_row, int64_t M, int64_t K, uint8_t *out, void *out_sf, ColKind kind,
                            hipStream_t stream)
{
    col_small::Args a;
    a.q_row = q_row;
    a.sf_row = sf_row;
    a.out = out;
    a.out_sf = out_sf;
    a.M = (uint32_t)M;
    a.K = (uint32_t)K;
    a.tiles_m = (uint32_t)((M + TILE - 1) / TILE);
    a.tiles_k = (uint32_t)(K / TILE);
    const dim3 grid(a.tiles_m * a.tiles_k);
    if (kind == COL_MXFP4)
        hipLaunchKernelGGL(col_small_kernel<COL_MXFP4>, grid, dim3(THREADS), 0, stream, a);
    else if (kind == COL_ALIGN)
        hipLaunchKernelGGL(col_small_kernel<COL_ALIGN>, grid, dim3(THREADS), 0, stream, a);
    else
        hipLaunchKernelGGL(col_small_kernel<COL_REQUANT>, grid, dim3(THREADS), 0, stream, a);
    return hipGetLastError();
}

} // namespace mxfp4
