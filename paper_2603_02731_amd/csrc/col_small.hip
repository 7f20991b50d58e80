// Row-blocked MXFP4 -> column-blocked MXFP4 or column-wise FP8 of a small matrix or of ragged experts, gfx950.
//
// The conversions of row_to_col.hip, row_to_fp8_col.hip and row_to_fp8_col_requant.hip for launches that do not fill the chip, which
// last as long as one workgroup does: load, convert, turn round in LDS, store.  Here a lane takes 8 rows x 8 columns, a quarter of the
// 32 x 8 slice of those kernels (the quarters of a slice in a quad of lanes, which exchange column maxima by DPP), a workgroup 128 x 128
// elements, and there are four times as many of them.  MXFP4 needs one barrier, scale alignment two, re-quantization three.
// Calls in a HIP graph, us (tiles of 256 x 256 / here): row->col [128,7168] 5.0 / 2.6, [2048,2048] 5.3 / 3.2, [5120,2048] 6.1 / 4.6;
// alignment 5.0 / 2.8, 6.1 / 3.5 and 6.5 / 5.1, re-quantization 5.8 / 3.2, 6.8 / 4.0 and 7.2 / 5.9; of either about 2 are the launch.
// With every byte from and to HBM [2048,2048] 6.0 / 3.7, 6.3 / 4.0 and 7.0 / 4.6.  A byte load per row scale instead of a dword per row
// turned round in LDS 0.2 more, nibbles through LDS by 16-byte loads 0.2 more.  The XCDs take contiguous runs of tiles, row tile by row
// tile, so that neighbours along k, which share 128-byte lines of the nibbles, are in one L2 ([5120,2048] 5.6 -> 4.7; ids as they come
// deal them to eight).
// Ragged experts: the same tiles of every expert, rows that the last one does not have as zeros under scale byte 0.  They save half of
// what the larger tiles spend on last ones and the look-back rows of row_to_fp8_col_grouped.hip, and leave by 16-byte stores at any byte:
// [4436,1152] in 16 experts, not padded, 6.8 / 4.4, 8.7 / 5.0 and 10.0 / 5.8, [17315,1024] in 128 13.1 / 9.2, 14.1 / 10.6 and 16.4 / 11.3.
// What a tile costs beside its elements (addresses, half lines, scales four or one at a time) is four times as much too, so where
// workgroups queue up this is slower ([4096,7168], every byte from and to HBM, 10.2 / 14.6): col_small_rule.hpp.
// Not kept: plain loads, which leave the matrix in the memory-side cache for another pass over it ([8192,7168] of three in turn 25.4 ->
// 13.5, but 25.1 where every byte comes from HBM, where the larger tiles take 18.0; [2048,2048] 3.7 -> 4.5); 256 x 128, 128 x 256 and
// 256 x 256 elements with as many lanes as here per element ([2048,2048] 3.3 -> 3.7, 3.8 and 4.6, [4096,7168] no better).
#include "col_small_rule.hpp"
#include "fp8_col_tile.hpp"
#include "mxfp4_device.hpp"
#include "mxfp4_kernels.hpp"

namespace mxfp4 {
namespace col_small {

using namespace fp8col;

constexpr uint32_t MBM_MAX = 64;

struct Args {
    const uint8_t *q_row;
    const uint8_t *sf_row;
    uint8_t *out;
    void *out_sf; // bytes (MXFP4) or floats
    const int32_t *expert_offsets; // nullptr: one matrix of M rows
    int32_t num_experts;
    uint32_t M, K;
    uint32_t tiles_m, tiles_k; // tiles_m: of one matrix
    FastDiv by_tiles_k;
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

template <ColKind KIND, bool EXPERTS>
__global__ void __launch_bounds__(THREADS) col_small_kernel(const col_small::Args a)
{
    // The tile's output: column 8 cg + c is LDS row c * 16 + cg, so that what the lanes of a wave write at once lies on different banks.
    constexpr uint32_t BYTES = KIND == COL_MXFP4 ? TILE / 2u : TILE, ROW = BYTES + 16u;
    __shared__ alignas(16) uint8_t s_out[TILE * ROW];
    __shared__ alignas(4) uint8_t s_sf[KIND == COL_MXFP4 ? TILE : 1][4]; // [LDS row][32 rows]: scales
    __shared__ alignas(8) uint8_t s_row_sf[4][4][32];                    // [32 rows][k-block][row]
    __shared__ uint16_t s_max[4][4]; // [32 rows][k-block]: largest scale byte that is not NaN; bit 8: one of FROM or more, 9: a NaN
    __shared__ alignas(16) uint32_t s_amax[KIND == COL_REQUANT ? 4 : 1][TILE]; // [32 rows][column]: bits of the largest |value|, or Emax + 1

    // ---- the tile; of which rows, and where their outputs begin
    uint32_t tile_k, tile_m, rows = a.M, groups = a.tiles_m, row_base = 0;
    uint8_t *out = a.out;
    uint8_t *out_sf8 = static_cast<uint8_t *>(a.out_sf);
    uint32_t *out_sf32 = static_cast<uint32_t *>(a.out_sf);
    if (EXPERTS) {
        ExpertTile t;
        constexpr uint32_t UNIT_A = KIND == COL_MXFP4 ? 2 : 0, UNIT_B = KIND == COL_MXFP4 ? 32 : TILE;
        const uint32_t n = (uint32_t)a.num_experts;
        if (!(n <= 64u ? expert_tile<1, TILE, UNIT_A, UNIT_B, MBM_MAX>(a.expert_offsets, n, blockIdx.x, a.tiles_k, a.by_tiles_k, &t)
                       : expert_tile<EXPERTS_MAX / 64, TILE, UNIT_A, UNIT_B, MBM_MAX>(a.expert_offsets, n, blockIdx.x, a.tiles_k,
                                                                                      a.by_tiles_k, &t)))
            return;
        tile_m = t.tile_m;
        tile_k = t.tile_k;
        row_base = t.row_base;
        rows = t.rows;
        groups = (rows + TILE - 1u) / TILE;
        out += (size_t)a.K * (KIND == COL_MXFP4 ? t.a_before : row_base);
        out_sf8 += (size_t)a.K * t.b_before;
        out_sf32 += (size_t)a.K * t.b_before;
    } else {
        uint32_t entry;
        if (!order_entry_of_workgroup(blockIdx.x, a.tiles_m * a.tiles_k, &entry))
            return;
        tile_m = a.tiles_k == 1u ? entry : a.by_tiles_k(entry);
        tile_k = entry - tile_m * a.tiles_k;
    }
    const uint32_t m0 = tile_m * TILE, k0 = tile_k * TILE;
    const uint32_t n_rows = min(TILE, rows - m0); // 1..128; of one matrix whole blocks of 32, 128 for FP8
    const uint32_t n_rg = EXPERTS ? (n_rows + 31u) / 32u : n_rows / 32u;
    const uint32_t tid = threadIdx.x;
    const uint32_t sub = tid & 3u, cg = tid >> 2 & 15u, rg = tid >> 6; // rows 32 rg + 8 sub, columns 8 cg of the tile
    const uint32_t pitch = a.K / 2u, Kb = a.K / 32u, kb = cg >> 2;

    // Of this wave's 32 rows there are some: splits of 58 rows on the average take 17.1 us where waves without rows do nothing, else 18.4
    // ([7424,3712] in 128, MXFP4), of 32 rows 20.2 and 26.3 ([4096,7168] in 128).
    const bool present = !EXPERTS || (uint32_t)__builtin_amdgcn_readfirstlane((int)rg) < n_rg;

    // ---- the lane's 8 x 8 elements and its 8 row-scale bytes
    uint32_t w[8], b[8];
    {
        const uint8_t *src = a.q_row + (size_t)(row_base + m0) * pitch + k0 / 2u;
        const uint8_t *src_sf = a.sf_row + (size_t)(row_base + m0) * Kb + k0 / 32u;
        const uint32_t lane = tid & 63u;
        uint32_t sf = 0;
        // uniform row pointers plus a 32-bit lane offset (K is at most 2^24)
        if (!EXPERTS || n_rows == TILE) {
            const uint32_t row0 = rg < n_rg ? rg * 32u : 0u; // past the end: any rows, not stored
            if (lane < 32u)
                sf = *reinterpret_cast<const uint32_t *>(src_sf + (row0 + lane) * Kb);
            const uint32_t at = (row0 + sub * 8u) * pitch + cg * 4u;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                w[i] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(src + (size_t)i * pitch + at));
        } else if (present) { // rows that an expert does not have are zeros under scale byte 0 (read from its last row, then cleared)
            const uint32_t row0 = rg * 32u, first = row0 + sub * 8u;
            if (row0 + lane < min(row0 + 32u, n_rows))
                sf = *reinterpret_cast<const uint32_t *>(src_sf + (row0 + lane) * Kb);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                w[i] = __builtin_nontemporal_load(
                    reinterpret_cast<const uint32_t *>(src + min(first + i, n_rows - 1u) * pitch + cg * 4u));
#pragma unroll
            for (int i = 0; i < 8; ++i)
                w[i] = first + i < n_rows ? w[i] : 0u;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                w[i] = 0u;
        }
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
        if (!present) {
            // nothing to write
        } else if (largest < 253u) {
            uint32_t cb[8], o[8];
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
            if (EXPERTS) { // decode again rather than keep 64 values: 47 registers for 82, the waves of a compute unit are not bound by them
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    asm volatile("" : "+v"(w[i]));
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
#pragma unroll
            for (int c = 0; c < 8; ++c)
                *reinterpret_cast<uint32_t *>(s_out + (c * 16u + cg) * ROW + rg * 16u + sub * 4u) = o[c];
            if (sub == 0u) {
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    s_sf[c * 16u + cg][rg] = (uint8_t)cb[c];
            }
        } else {
            // values beyond FP32, or NaN: in integers, as column_byte_int and column_codes_int (rolled: written for size)
#pragma nounroll
            for (uint32_t c = 0; c < 8u; ++c) {
                int emax = -1024;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int mag = (int)(w[i] >> (4 * c)) & 7;
                    emax = mag ? max(emax, (int)b[i] + (mag >> 1)) : emax;
                }
                emax = quad_reduce(emax, [](int x, int y) { return max(x, y); });
                const uint32_t cb = largest == 255u ? 255u : (uint32_t)max(0, emax - 3);
                uint32_t o = 0u;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint32_t nib = (w[i] >> (4 * c)) & 0xFu;
                    const int mag = (int)(nib & 7u), em = mag == 1 ? 0 : mag;
                    const int t2 = max(em + 2 * ((int)b[i] - (int)cb) + 2, 0);
                    const int code = mag ? min(7, max(t2 - 2, (t2 + 1) >> 1)) : 0;
                    if (largest != 255u)
                        o |= ((nib & 8u) | (uint32_t)code) << (4 * i);
                }
                *reinterpret_cast<uint32_t *>(s_out + (c * 16u + cg) * ROW + rg * 16u + sub * 4u) = o;
                if (sub == 0u)
                    s_sf[c * 16u + cg][rg] = (uint8_t)cb;
            }
        }
    } else {
        auto out_scale = [&](uint32_t column, uint32_t bits) {
            out_sf32[(size_t)(k0 + column) * groups + tile_m] = bits;
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
        if (KIND == COL_ALIGN) {
            uint32_t o[8][2];
            if (scales < 8u) {
                const int e = (int)bmax - 6; // biased exponent of 2^(max - 6 - 127); below 1: an FP32 subnormal
                const uint32_t bits = flags ? 0x7FC00000u : e >= 1 ? (uint32_t)e << 23 : 0x00400000u >> (uint32_t)(-e);
                out_scale(cg * 8u + scales, bits);
            }
            if (present) {
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
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    *reinterpret_cast<u32x2 *>(s_out + (c * 16u + cg) * ROW + rg * 32u + sub * 8u) = u32x2{o[c][0], o[c][1]};
            }
        } else {
            // ---- the group's largest value of every column: its FP32 bits, or Emax where those do not do
            if (!present) {
                if (sub == 0u) {
                    u32x4 *dst = reinterpret_cast<u32x4 *>(s_amax[rg] + cg * 8u);
                    dst[0] = dst[1] = u32x4{0u, 0u, 0u, 0u};
                }
            } else if (flags == 0u) {
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
                uint32_t m[8];
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    m[c] = f2u(quad_reduce(amax[c], [](float x, float y) { return __builtin_elementwise_maximum(x, y); }));
                if (sub == 0u) {
                    u32x4 *dst = reinterpret_cast<u32x4 *>(s_amax[rg] + cg * 8u);
                    dst[0] = u32x4{m[0], m[1], m[2], m[3]};
                    dst[1] = u32x4{m[4], m[5], m[6], m[7]};
                }
            } else {
                // Emax + 1 over the non-zero codes of rows whose scale byte is not NaN, 0 without any (rolled: written for size)
#pragma nounroll
                for (uint32_t c = 0; c < 8u; ++c) {
                    uint32_t e = 0;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const uint32_t mag = (w[i] >> (4 * c)) & 7u;
                        e = mag && b[i] != 255u ? max(e, b[i] + (mag >> 1) + 1u) : e;
                    }
                    e = quad_reduce(e, [](uint32_t x, uint32_t y) { return max(x, y); });
                    if (sub == 0u)
                        s_amax[rg][cg * 8u + c] = e;
                }
            }
            __syncthreads();
            uint32_t m[8];
#pragma unroll
            for (int c = 0; c < 8; ++c)
                m[c] = 0u;
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
            float enc[8];
            uint32_t mine = 0; // the maximum of the column whose scale this lane stores
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const bool zero = m[c] == 0u;
                const uint32_t ef = m[c] >> 23;
                slow |= flags == 0u && !zero && ef < 8u; // a maximum below 2^-118: operand exponent negative
                enc[c] = u2f((zero ? 127u : ef - 8u) << 23);
                mine = scales == (uint32_t)c ? m[c] : mine;
            }
            auto emax_of = [&](uint32_t v) { return flags != 0u ? (int)v - 1 : v == 0u ? -1 : emax_of_amax_bits(v); };
            if (scales < 8u)
                out_scale(cg * 8u + scales, (flags & 2u) ? 0x7FC00000u : scale_bits_of_emax(emax_of(mine), mine != 0u));
            if (!present) {
                // nothing to write
            } else if (!slow) {
                uint32_t o[8][2];
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
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    *reinterpret_cast<u32x2 *>(s_out + (c * 16u + cg) * ROW + rg * 32u + sub * 8u) = u32x2{o[c][0], o[c][1]};
            } else {
#pragma nounroll
                for (uint32_t c = 0; c < 8u; ++c) {
                    uint32_t v = 0u;
#pragma unroll
                    for (uint32_t g = 0; g < 4u; ++g)
                        v = max(v, s_amax[g][cg * 8u + c]);
                    const int emax = emax_of(v);
                    u32x2 r = {0u, 0u};
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const uint32_t nib = (w[i] >> (4 * c)) & 0xFu;
                        r[i >> 2] |= (b[i] == 255u ? 0x7Fu : e4m3_requant_int(nib, b[i], emax)) << (8 * (i & 3));
                    }
                    *reinterpret_cast<u32x2 *>(s_out + (c * 16u + cg) * ROW + rg * 32u + sub * 8u) = r;
                }
            }
        }
    }
    __syncthreads();

    // ---- out: 16-byte pieces.  The k-rows of an expert begin at any byte and end in any piece
    constexpr uint32_t PIECES = BYTES / 16u;
    const uint32_t pitch_out = KIND == COL_MXFP4 ? (rows + 1u) / 2u : rows, nb = KIND == COL_MXFP4 ? (n_rows + 1u) / 2u : n_rows;
    // Stores are non-temporal where a tile's pieces are whole 64-byte segments ([2048,2048] with every byte from and to HBM, alignment
    // 5.1 -> 4.0 us), but for MXFP4 of experts, where that gains below 1024 tiles what it loses above (1152 tiles 7.3 -> 8.4).
    const bool segments = ((reinterpret_cast<uintptr_t>(out) | pitch_out) & 63u) == 0u;
#pragma unroll
    for (uint32_t u = 0; u < TILE * PIECES / THREADS; ++u) {
        const uint32_t i = u * THREADS + tid, column = i / PIECES, p = i % PIECES;
        uint8_t *dst = out + (size_t)(k0 + column) * pitch_out + (KIND == COL_MXFP4 ? m0 / 2u : m0) + p * 16u;
        const u32x4 v = *reinterpret_cast<const u32x4 *>(s_out + ((column & 7u) * 16u + (column >> 3)) * ROW + p * 16u);
        if (!EXPERTS) {
            if (KIND != COL_MXFP4 || p < n_rg)
                __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(dst));
        } else if (KIND != COL_MXFP4 && segments && p * 16u + 16u <= nb) {
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(dst));
        } else if (p * 16u + 16u <= nb) {
            *reinterpret_cast<u32x4_unaligned *>(dst) = v;
        } else if (p * 16u < nb) {
            store_head_bytes(dst, v, nb - p * 16u);
        }
    }
    if (KIND == COL_MXFP4 && tid < TILE) {
        uint8_t *dst = out_sf8 + (size_t)(k0 + tid) * ((rows + 31u) / 32u) + m0 / 32u;
        const uint32_t v = *reinterpret_cast<const uint32_t *>(s_sf[(tid & 7u) * 16u + (tid >> 3)]);
        if (n_rg == 4u)
            *reinterpret_cast<u32_unaligned *>(dst) = v;
        else
            store_head_bytes(dst, u32x4{v, 0u, 0u, 0u}, n_rg);
    }
}

bool col_in_small_tiles(int64_t M, int64_t K, int32_t num_experts, ColKind kind)
{
    return col_in_small_tiles(M, K, num_experts, kind, compute_units());
}

template <bool EXPERTS>
static void launch_kind(const col_small::Args &a, int64_t tiles, ColKind kind, hipStream_t stream)
{
    const dim3 grid((uint32_t)((tiles + NUM_XCD - 1) / NUM_XCD * NUM_XCD));
    if (kind == COL_MXFP4)
        hipLaunchKernelGGL((col_small_kernel<COL_MXFP4, EXPERTS>), grid, dim3(THREADS), 0, stream, a);
    else if (kind == COL_ALIGN)
        hipLaunchKernelGGL((col_small_kernel<COL_ALIGN, EXPERTS>), grid, dim3(THREADS), 0, stream, a);
    else
        hipLaunchKernelGGL((col_small_kernel<COL_REQUANT, EXPERTS>), grid, dim3(THREADS), 0, stream, a);
}

hipError_t launch_col_small(const uint8_t *q_row, const uint8_t *sf_row, const int32_t *expert_offsets, int32_t num_experts, int64_t M,
                            int64_t K, uint8_t *out, void *out_sf, ColKind kind, hipStream_t stream)
{
    col_small::Args a;
    a.q_row = q_row;
    a.sf_row = sf_row;
    a.out = out;
    a.out_sf = out_sf;
    a.expert_offsets = expert_offsets;
    a.num_experts = num_experts;
    a.M = (uint32_t)M;
    a.K = (uint32_t)K;
    a.tiles_m = (uint32_t)((M + TILE - 1) / TILE);
    a.tiles_k = (uint32_t)(K / TILE);
    a.by_tiles_k = FastDiv(a.tiles_k);
    const int64_t tiles = col_small_workgroups(M, K, expert_offsets ? num_experts : 0);
    if (expert_offsets)
        launch_kind<true>(a, tiles, kind, stream);
    else
        launch_kind<false>(a, tiles, kind, stream);
    return hipGetLastError();
}

} // namespace mxfp4
