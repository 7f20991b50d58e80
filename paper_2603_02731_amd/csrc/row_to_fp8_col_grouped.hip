// Row-blocked MXFP4 -> the transposed matrices of ragged experts as FP8 (E4M3 [K, T_e] + FP32 scale per 128 rows), gfx950.
// Both readings of the conversion; the arithmetic is that of row_to_fp8_col.hip (scale alignment) and of
// row_to_fp8_col_requant.hip (re-quantization).
//
// What is different for experts is where the output lies.  A k-row of an expert of T_e rows starts at any byte, so a tile that
// writes the bytes of its own 256 rows shares the first and the last 64-byte segment of every k-row with its neighbours.  The
// halves of a segment come from two workgroups and have to meet in an L2 that is too small for what is in flight between them;
// what leaves it half written costs the memory a read, modify and write.  Here a tile writes whole segments: the bytes from the
// segment that holds its first row on, and none after its last whole segment, which are the next tile's.  For that it converts
// up to 64 rows before its own once more (LOOK-BACK; for re-quantization it also takes the column maxima of the 64 rows before
// those, the rest of their scale group).  Experts whose k-rows are whole segments need none of it.
//
// Work split.  A workgroup of 256 lanes owns a tile of 256 rows x 256 columns; lane (rg, cg) the rows 32*rg.. and the columns
// 8*cg.., and of the look-back group the rows 8*rg.. of either half, so that all lanes have the same work (a fifth and a sixth
// wave for the look-back rows instead: 213 us, only two such workgroups were resident).  The tile leaves in two passes of
// four columns per lane: 46 and 50 KB of LDS, three workgroups per compute unit.  The pieces are put together from five dwords
// of LDS with byte alignments (unaligned 16-byte LDS reads: 55 us more).
//
// Measured at 65536 rows of K = 7168 in 32 experts (us, kernels that write their own rows only / this one; scale alignment and
// re-quantization): Zipf-sized 192 / 159 and 190 / 166, padded to 128 rows 149 / 142 and 152 / 141, equal 2041 rows 179 / 153
// and 187 / 160; K = 2048 58 / 46 and 60 / 50; 128 experts 214 / 179 and 221 / 187; 128 of 500 rows 200 / 170 and 188 / 176;
// 80 of 780 rows, where every fourth tile has 12 rows, 174 / 167 and 184 / 176; 100 of 268 104 / 102 and 111 / 102; 50 of 190, one
// tile along the rows each, 39 / 26 and 41 / 28.  A mover of the same bytes in the same tiles takes 155 (Zipf-sized) and 133
// (padded).  Bound by that pattern, and in a workgroup's 33 thousand cycles by the wait for its loads (8), the two conversions (4)
// and the two write-outs (6).
// Not kept: whole 128-byte lines (every lane converts twice the look-back rows, which re-quantization has loaded already and scale
// alignment has not; the mover gains 4 %); one pass (87 KB) 259;
// four passes and four workgroups per compute unit 172 against 168.
#include "fp8_col_tile.hpp"
#include "mxfp4_device.hpp"
#include "mxfp4_kernels.hpp"
#include "row_to_fp8_col_rule.hpp"

namespace mxfp4 {

namespace fp8col_grouped {

using namespace fp8col;

constexpr uint32_t TILE_M = 256, TILE_K = 256;
constexpr uint32_t GROUP = 128;            // rows of a scale group: the window begins one group before the tile
constexpr uint32_t WIN = GROUP + TILE_M;   // window row r is row m0 - GROUP + r of the expert
constexpr uint32_t THREADS = 256, WAVES = 4; // one lane per (32-row group of the tile, 8-column group)
constexpr uint32_t SEG = 64;               // the segments of the output that a tile writes whole
constexpr uint32_t FAR = GROUP - SEG;      // look-back rows that only enter the scales
constexpr int PASSES = 2, CPP = 8 / PASSES; // the tile leaves in passes; columns of a lane per pass
constexpr uint32_t ROW = SEG + TILE_M + 16; // bytes of an LDS k-row: an odd number of 16-byte slots
constexpr uint32_t SF = WIN + 16;          // row-scale bytes of one k-block in LDS

struct Args {
    const uint8_t *q_row;
    const uint8_t *sf_row;
    uint8_t *x_col;
    float *x_col_scale;
    const int32_t *expert_offsets;
    int32_t num_experts;
    uint32_t K;
    uint32_t tiles_k; // 256-column tiles
    FastDiv by_tiles_k;
    uint32_t stream; // the nibbles are not expected to be read again from the memory-side cache
};

} // namespace fp8col_grouped

using namespace fp8col_grouped;

// Four rows (4r.. of a slice) of two columns (nibble byte J) as E4M3: dword r of either column.
template <int J>
__device__ __forceinline__ void four_rows(const uint32_t *w, const float (&s)[4], float enc0, float enc1, uint32_t *o0,
                                          uint32_t *o1)
{
    const f32x2 f0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[0], s[0], J);
    const f32x2 f1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[1], s[1], J);
    const f32x2 f2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[2], s[2], J);
    const f32x2 f3 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[3], s[3], J);
    s16x2 e0, e1; // no initial value needed: both words are written
    asm volatile("" : "=v"(e0), "=v"(e1));
    e0 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(e0, f0.x, f1.x, enc0, false);
    e0 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(e0, f2.x, f3.x, enc0, true);
    e1 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(e1, f0.y, f1.y, enc1, false);
    e1 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(e1, f2.y, f3.y, enc1, true);
    *o0 = __builtin_bit_cast(uint32_t, e0);
    *o1 = __builtin_bit_cast(uint32_t, e1);
}

// The scale operands of four rows whose bytes are packed in a dword (the neighbouring bytes land in the sign and mantissa
// bits, which the conversions do not read).
__device__ __forceinline__ void operands_of(uint32_t sb, float (&s)[4])
{
    s[0] = u2f(sb << 23);
    s[1] = u2f(sb << 15);
    s[2] = u2f(sb << 7);
    s[3] = u2f(sb >> 1);
}

// Running maxima of |value| over N rows of 8 columns.
template <int N>
__device__ __forceinline__ void maxima(const uint32_t *w, const uint32_t *sb, float (&amax)[8])
{
    static_for<N / 4>([&](auto qp) {
        constexpr int q = decltype(qp)::value;
        float s[4];
        operands_of(sb[q], s);
        static_for<4>([&](auto jp) {
            constexpr int j = decltype(jp)::value;
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                const f32x2 fa = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[4 * q + i], s[i], j);
                const f32x2 fb = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[4 * q + i + 1], s[i + 1], j);
                amax[2 * j] = max3_abs_nan(fa.x, fb.x, amax[2 * j]);
                amax[2 * j + 1] = max3_abs_nan(fa.y, fb.y, amax[2 * j + 1]);
            }
        });
    });
}

typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

// Column maxima of two 32-lane halves of the wave as the upper halves of the FP32 values (the lower ones are zero: a maximum
// has at most two significant bits), combined: non-negative floats order like their bit patterns.
__device__ __forceinline__ u32x4 combined_halves(const float (&amax)[8])
{
    u32x4 r;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t v = perm(f2u(amax[2 * c + 1]), f2u(amax[2 * c]), 0x07060302u);
        const auto both = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        r[c] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, (uint32_t)both[0]),
                                                                      __builtin_bit_cast(u16x2, (uint32_t)both[1])));
    }
    return r;
}

template <bool REQUANT>
__global__ void __launch_bounds__(THREADS, 3) row_to_fp8_col_grouped_kernel(const fp8col_grouped::Args a)
{
    // [cl*32 + cg][window row - FAR]: the k-rows of a pass
    __shared__ alignas(16) uint8_t s_tile[32 * CPP * ROW > WAVES * 8192 ? 32 * CPP * ROW : WAVES * 8192];
    __shared__ alignas(16) uint8_t s_row_sf[8 * SF];       // [k-block of the tile][window row]
    __shared__ alignas(8) uint8_t s_max16[REQUANT ? 8 : 8 * (WIN / 16)]; // [k-block][16-row group]: max of the non-NaN bytes
    __shared__ uint8_t s_flag[WIN / 64 * 8]; // [64-row group][k-block]: a NaN scale byte (REQUANT: a byte >= 253) occurs
    // [wave][column]: maxima of pass 1 over the wave's rows of the tile, then over its rows of the look-back group
    __shared__ alignas(16) uint16_t s_amax[REQUANT ? 2 * WAVES * TILE_K : 8];

    ExpertTile et;
    if (!tile_of_expert_workgroup<TILE_M, 128, 0, 64>(a.expert_offsets, a.num_experts, blockIdx.x, a.tiles_k, a.by_tiles_k, &et))
        return;
    const uint32_t tile_m = et.tile_m, tile_k = et.tile_k, row_base = et.row_base, rows = et.rows, groups_before = et.a_before;
    const uint32_t m0 = tile_m * TILE_M; // first row of the tile inside its expert, below `rows`
    const uint32_t n_rows = min(TILE_M, rows - m0);
    const uint32_t n_g = (n_rows + 127u) / 128u;
    const uint32_t k0 = tile_k * TILE_K;
    const uint32_t cols = min(TILE_K, a.K - k0); // 128 or 256
    const uint32_t Kb = a.K / 32u, pitch = a.K / 2u;
    uint8_t *out_x = a.x_col + (size_t)a.K * row_base;
    float *out_s = a.x_col_scale + (size_t)a.K * groups_before;
    const size_t pitch_s = (rows + 127u) / 128u;

    const bool whole = ((reinterpret_cast<uintptr_t>(out_x) | rows) & (SEG - 1u)) == 0u; // every k-row is whole segments
    const bool look = tile_m != 0u && !whole;
    const uint32_t end = GROUP + n_rows; // window rows up to here exist

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t rg = tid >> 5, cg = tid & 31u, kb = cg >> 2;
    const bool in_cols = cg * 8u < cols;
    const bool active = rg * 32u < n_rows && in_cols;
    // window row 0, column k0 (before the expert where the look-back rows are not used)
    const uint8_t *win_src = a.q_row + ((int64_t)row_base + m0 - GROUP) * (int64_t)pitch + k0 / 2u;

    // ---- row scales: thread t takes row t of the tile and, for t < 128, row t of the look-back group
    auto row_scales = [&](uint32_t win_row) {
        const uint8_t *p = a.sf_row + (size_t)(row_base + m0 + win_row - GROUP) * Kb + k0 / 32u;
        if (cols > 128u) // one request at any 4-byte alignment
            return u32x2(*reinterpret_cast<const u32x2_unaligned *>(p));
        return u32x2{*reinterpret_cast<const uint32_t *>(p), 0u};
    };
    u32x2 sfv = {0u, 0u}, sfl = {0u, 0u};
    if (tid < n_rows)
        sfv = row_scales(GROUP + tid);
    if (look && wv < GROUP / 64u)
        sfl = row_scales(tid);
    // ---- nibbles.  A wave takes its own 64 rows of the tile by 8 rows x 128 bytes per instruction, then the 16 rows of the
    // near (and, for the scales of re-quantization, of the far) half of the look-back group that its lanes convert.
    auto piece_of = [&](uint32_t win_row) {
        return reinterpret_cast<const u32x4_unaligned *>(win_src + (size_t)(win_row * pitch + (lane & 7u) * 16u));
    };
    const bool piece_in = (lane & 7u) * 32u < cols;
    u32x4 stage_v[8], stage_l[4];
    if (wv * 64u < n_rows && piece_in) {
        auto row_of = [&](int j) { return min(GROUP + wv * 64u + j * 8u + (lane >> 3), end - 1u); };
        // Rows that the next tile reads again stay in the L2.  Nibbles of more than KEEP_BYTES leave the caches to the rest:
        // [65536, 7168] in 32 Zipf-sized experts 171 -> 164 us, padded 147.5 -> 142.4; smaller matrices are left in the
        // memory-side cache, as the de-quantizer does (read again and again: [65536, 2048] 51.6 -> 42.0, cold 52.3 -> 52.5).
        if (a.stream && (whole || wv < (REQUANT ? 2u : 3u))) {
            asm volatile("" : : "v"(tid)); // keeps the two forms of the loads apart
#pragma unroll
            for (int j = 0; j < 8; ++j)
                stage_v[j] = __builtin_nontemporal_load(piece_of(row_of(j)));
            asm volatile("" : : "v"(tid));
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                stage_v[j] = *piece_of(row_of(j));
        }
    }
    if (look && piece_in) {
#pragma unroll
        for (int j = 0; j < (REQUANT ? 4 : 2); ++j)
            stage_l[j] = *piece_of((j < 2 ? FAR : 0u) + wv * 16u + (j & 1) * 8u + (lane >> 3));
    }

    auto stage_scales = [&](const u32x2 v, uint32_t win_row) {
        stage_row_scales<REQUANT, SF, WIN>(v, win_row, lane, s_row_sf, s_flag, s_max16);
    };
    stage_scales(sfv, GROUP + tid);
    if (look && wv < GROUP / 64u)
        stage_scales(sfl, tid);

    // the lane's slices, a dword (8 columns) per row: 32 rows of the tile, 8 of the near and 8 of the far half
    uint32_t w[32], wl[REQUANT ? 16 : 8];
    {
        u32x4 *st = reinterpret_cast<u32x4 *>(s_tile) + wv * 512u;
        const uint32_t *s_in = reinterpret_cast<const uint32_t *>(st) + cg;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            st[j * 64u + lane] = stage_v[j];
        wave_fence();
#pragma unroll
        for (int i = 0; i < 32; ++i)
            w[i] = s_in[(rg & 1u) * 1024u + i * 32];
        if (look) {
            wave_fence();
#pragma unroll
            for (int j = 0; j < (REQUANT ? 4 : 2); ++j)
                st[j * 64u + lane] = stage_l[j];
            wave_fence();
#pragma unroll
            for (int i = 0; i < (REQUANT ? 16 : 8); ++i)
                wl[i] = s_in[(i & 8) * 64 + (rg & 1u) * 256u + (i & 7) * 32];
        }
        if (REQUANT && n_rows < TILE_M) { // rows that do not exist count as zeros
#pragma unroll
            for (int i = 0; i < 32; ++i)
                w[i] = rg * 32u + i < n_rows ? w[i] : 0u;
        }
    }
    __syncthreads();

    // ---- the lane's view: its k-block, its group of the tile (window group g + 1)
    const uint32_t g = rg >> 2;
    auto flagged = [&](uint32_t group, uint32_t k_block) {
        return (s_flag[2 * group * 8 + k_block] | s_flag[(2 * group + 1) * 8 + k_block]) != 0u;
    };
    const bool flag = flagged(g + 1u, kb), flag_l = look && flagged(0u, kb);
    const uint8_t *my_row_sf = &s_row_sf[kb * SF + GROUP + rg * 32u]; // of the slice's rows
    const uint8_t *my_row_sf_l = &s_row_sf[kb * SF + rg * 8u];        // far rows; near ones FAR bytes on
    uint32_t sb[8], sbl[4]; // row-scale bytes: byte i%4 of dword i/4 is row i (sbl: near, then far)
    {
        const u32x4 s0 = reinterpret_cast<const u32x4 *>(my_row_sf)[0];
        const u32x4 s1 = reinterpret_cast<const u32x4 *>(my_row_sf)[1];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            sb[q] = s0[q];
            sb[4 + q] = s1[q];
        }
        const u32x2 n = *reinterpret_cast<const u32x2 *>(my_row_sf_l + FAR), f = *reinterpret_cast<const u32x2 *>(my_row_sf_l);
        sbl[0] = n.x;
        sbl[1] = n.y;
        sbl[2] = f.x;
        sbl[3] = f.y;
    }

    float enc[8], enc_l[8];
    bool slow = false, slow_l = false;
    if (REQUANT) {
        float amax[8];
#pragma unroll
        for (int c = 0; c < 8; ++c)
            amax[c] = 0.0f;
        if (active && !flag)
            maxima<32>(w, sb, amax);
        const u32x4 m = combined_halves(amax);
        if (lane < 32u)
            *reinterpret_cast<u32x4 *>(&s_amax[wv * TILE_K + cg * 8u]) = m;
        if (look) {
#pragma unroll
            for (int c = 0; c < 8; ++c)
                amax[c] = 0.0f;
            if (in_cols && !flag_l)
                maxima<16>(wl, sbl, amax);
            const u32x4 ml = combined_halves(amax);
            if (lane < 32u)
                *reinterpret_cast<u32x4 *>(&s_amax[(WAVES + wv) * TILE_K + cg * 8u]) = ml;
        }
        __syncthreads();
        auto encoders = [&](uint32_t wave0, uint32_t n, float (&e)[8]) { // the encoder's operand exponent Emax - 9
            u16x8 mx = *reinterpret_cast<const u16x8 *>(&s_amax[wave0 * TILE_K + cg * 8u]);
            for (uint32_t i = 1; i < n; ++i)
                mx = __builtin_elementwise_max(mx, *reinterpret_cast<const u16x8 *>(&s_amax[(wave0 + i) * TILE_K + cg * 8u]));
            bool tiny = false;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const uint32_t mc = mx[c], ef = mc >> 7;
                tiny |= mc != 0u && ef < 8u; // a maximum below 2^-118: operand exponent negative
                e[c] = u2f((mc != 0u ? ef - 8u : 127u) << 23);
            }
            return tiny;
        };
        slow = encoders(2u * g, 2u, enc) || flag;
        if (look)
            slow_l = encoders(WAVES, WAVES, enc_l) || flag_l;
    } else {
#pragma unroll
        for (int c = 0; c < 8; ++c)
            enc[c] = enc_l[c] = u2f(121u << 23); // the encoder divides by 2^-6: Algorithm 1's delta
    }

    // ---- group scales: k-row t of the tile, one float per 128-row group
    if (tid < cols) {
        const uint32_t kbt = tid >> 5;
        uint32_t bits[2];
#pragma unroll
        for (int gg = 0; gg < 2; ++gg) {
            const bool f = flagged(gg + 1u, kbt);
            if (REQUANT) {
                if (!f) {
                    const uint32_t m = max((uint32_t)s_amax[2 * gg * TILE_K + tid], (uint32_t)s_amax[(2 * gg + 1) * TILE_K + tid]);
                    bits[gg] = scale_bits_of_emax(emax_of_amax_bits(m << 16), m != 0u);
                } else if ((uint32_t)gg < n_g) {
                    const int emax = group_emax_int(win_src, pitch, &s_row_sf[kbt * SF], tid, GROUP + gg * 128u,
                                                    min(128u, n_rows - gg * 128u));
                    bits[gg] = emax >= GROUP_HAS_NAN - 1 ? 0x7FC00000u : scale_bits_of_emax(emax, emax >= 0);
                } else {
                    bits[gg] = 0u;
                }
            } else {
                // biased exponent of 2^(max - 6 - 127); below 1: an FP32 subnormal
                const int e = (int)max_of_8_bytes(&s_max16[kbt * (WIN / 16) + (gg + 1) * 8]) - 6;
                bits[gg] = e >= 1 ? (uint32_t)e << 23 : 0x00400000u >> (uint32_t)(-e);
                if (f)
                    bits[gg] = 0x7FC00000u;
            }
        }
        float *dst = out_s + (size_t)(k0 + tid) * pitch_s + m0 / 128u;
        if (n_g == 2u) // one request per k-row, at any multiple of 4 bytes
            *reinterpret_cast<u64_unaligned *>(dst) = ((uint64_t)bits[1] << 32) | bits[0];
        else
            dst[0] = u2f(bits[0]);
    }

    if (!REQUANT) {
        // scale bytes -> exponent fields of the decode operands, max(127 - (bmax - b), 0), packed like the bytes
        auto shifts = [&](uint32_t group, uint32_t *s, int n) {
            const uint32_t bmax = max_of_8_bytes(&s_max16[kb * (WIN / 16) + group * 8]);
            const uint16_t add = (uint16_t)(bmax < 127u ? 127u - bmax : 0u), sub = (uint16_t)(bmax < 127u ? 0u : bmax - 127u);
            for (int q = 0; q < n; ++q) {
                u16x2 even = __builtin_bit_cast(u16x2, s[q] & 0x00FF00FFu),
                      odd = __builtin_bit_cast(u16x2, (s[q] >> 8) & 0x00FF00FFu);
                even = __builtin_elementwise_sub_sat(even + u16x2{add, add}, u16x2{sub, sub});
                odd = __builtin_elementwise_sub_sat(odd + u16x2{add, add}, u16x2{sub, sub});
                s[q] = perm(__builtin_bit_cast(uint32_t, odd), __builtin_bit_cast(uint32_t, even), 0x06020400u);
            }
        };
        shifts(g + 1u, sb, 8);
        if (look)
            shifts(0u, sbl, 2);
    }

    const bool last = m0 + TILE_M >= rows;
    static_for<PASSES>([&](auto pp) {
        constexpr int p = decltype(pp)::value;
        if (p != 0) { // the operands are cheaper made again than kept in registers while the first pass leaves
#pragma unroll
            for (int q = 0; q < 8; ++q)
                asm volatile("" : "+v"(sb[q]));
            asm volatile("" : "+v"(sbl[0]), "+v"(sbl[1]));
        }
        uint8_t *my = s_tile + cg * ROW + SEG + rg * 32u; // k-row cl*32 + cg of this pass, the lane's rows of the tile
        uint8_t *my_l = s_tile + cg * ROW + rg * 8u;      // and of the near half
        // the integer path (re-quantization): per column the group's Emax from all of its rows, then the lane's elements
        // (nibbles read again from global memory) byte by byte
        auto by_integers = [&](uint32_t win_row0, uint32_t n, uint32_t group_row0, uint32_t group_n, uint8_t *dst) {
#pragma nounroll
            for (uint32_t cl = 0; cl < (uint32_t)CPP; ++cl) {
                const uint32_t c = p * CPP + cl;
                int emax = group_emax_int(win_src, pitch, &s_row_sf[kb * SF], cg * 8u + c, group_row0, group_n);
                emax = emax >= GROUP_HAS_NAN - 1 ? emax - GROUP_HAS_NAN : emax;
#pragma nounroll
                for (uint32_t i = 0; i < n; ++i) {
                    const uint32_t b = s_row_sf[kb * SF + win_row0 + i];
                    const uint32_t byte = win_src[(size_t)(win_row0 + i) * pitch + cg * 4u + (c >> 1)];
                    const uint32_t nib = ((c & 1u) ? byte >> 4 : byte) & 0xFu;
                    dst[cl * 32u * ROW + i] = (uint8_t)(b == 255u ? 0x7Fu : e4m3_requant_int(nib, b, emax));
                }
            }
        };
        // rare: the rows under a NaN scale byte become E4M3 NaN
        auto patch_nan = [&](const uint8_t *row_sf, uint32_t n, uint8_t *dst) {
#pragma nounroll
            for (uint32_t i = 0; i < n; ++i) {
                if (row_sf[i] != 255u)
                    continue;
#pragma nounroll
                for (uint32_t c = 0; c < (uint32_t)CPP; ++c)
                    dst[c * 32u * ROW + i] = 0x7Fu;
            }
        };
        if (active && !(REQUANT && slow)) {
            static_for<CPP / 2>([&](auto jp) {
                constexpr int jl = decltype(jp)::value, j = p * (CPP / 2) + jl; // nibble byte: columns 2j, 2j+1
                uint32_t o[2][8];
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    float s[4];
                    operands_of(sb[r], s);
                    four_rows<j>(w + 4 * r, s, enc[2 * j], enc[2 * j + 1], &o[0][r], &o[1][r]);
                }
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) {
                    u32x4 *dst = reinterpret_cast<u32x4 *>(my + (2 * jl + cc) * 32u * ROW);
                    dst[0] = u32x4{o[cc][0], o[cc][1], o[cc][2], o[cc][3]};
                    dst[1] = u32x4{o[cc][4], o[cc][5], o[cc][6], o[cc][7]};
                }
            });
            if (!REQUANT && flag)
                patch_nan(my_row_sf, 32u, my);
        } else if (REQUANT && active) {
            by_integers(GROUP + rg * 32u, min(32u, n_rows - rg * 32u), GROUP + g * 128u, min(128u, n_rows - g * 128u), my);
        }
        if (look && in_cols && !(REQUANT && slow_l)) {
            static_for<CPP / 2>([&](auto jp) {
                constexpr int jl = decltype(jp)::value, j = p * (CPP / 2) + jl;
                uint32_t o[2][2];
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    float s[4];
                    operands_of(sbl[r], s);
                    four_rows<j>(wl + 4 * r, s, enc_l[2 * j], enc_l[2 * j + 1], &o[0][r], &o[1][r]);
                }
#pragma unroll
                for (int cc = 0; cc < 2; ++cc)
                    *reinterpret_cast<u32x2 *>(my_l + (2 * jl + cc) * 32u * ROW) = u32x2{o[cc][0], o[cc][1]};
            });
            if (!REQUANT && flag_l)
                patch_nan(my_row_sf_l + FAR, 8u, my_l);
        } else if (REQUANT && look && in_cols) {
            by_integers(FAR + rg * 8u, 8u, 0u, GROUP, my_l);
        }
        __syncthreads();

        // ---- out.  A wave instruction writes 4 k-rows of 16 lanes x 16 bytes, eight columns apart; step i of a wave has the
        // LDS k-rows 4 * (wv + WAVES * i).., i.e. the columns c = p * CPP + i / 2 of the column groups 4 * wv + 16 * (i % 2)..
        constexpr int STEPS = 32 * CPP / 4 / WAVES;
        constexpr uint32_t PPS = SEG / 16; // pieces of a segment
        const uint32_t part = lane & 15u;
        // k-row of the lane in step 0 and the tile's first row, SEG bytes late: what is subtracted from an offset stays below SEG
        uint8_t *const base = out_x + (size_t)(k0 + wv * 32u + p * CPP) * rows + m0 - SEG;
        const uint32_t lane_row = (lane >> 4) * 8u * rows;
        auto krow = [&](int i) { return lane_row + (uint32_t)((i & 1) * 128 + (i >> 1)) * rows; }; // of step i, from base
        const uint32_t lane_lds = (wv * 4u + (lane >> 4)) * ROW;
        constexpr uint32_t STEP_LDS = WAVES * 4 * ROW;
        auto read16 = [&](uint32_t at) { // 16 bytes of the tile buffer from any byte on
            const uint32_t *d = reinterpret_cast<const uint32_t *>(s_tile + (at & ~3u));
            const uint32_t d0 = d[0], d1 = d[1], d2 = d[2], d3 = d[3], d4 = d[4];
            return u32x4{__builtin_amdgcn_alignbyte(d1, d0, at), __builtin_amdgcn_alignbyte(d2, d1, at),
                         __builtin_amdgcn_alignbyte(d3, d2, at), __builtin_amdgcn_alignbyte(d4, d3, at)};
        };
        // Where every k-row begins on 16 bytes, so do the pieces.
        auto aligned16 = [&](uint32_t at) { return *reinterpret_cast<const u32x4 *>(s_tile + at); };
        const bool by16 = ((reinterpret_cast<uintptr_t>(out_x) | rows) & 15u) == 0u;
        // bytes by which a k-row is past the start of a segment
        const uint32_t base_low = (uint32_t)reinterpret_cast<uintptr_t>(base);
        auto past = [&](uint32_t row) { return (base_low + row) & (SEG - 1u); };
        // Every tile begins and ends on a segment of the k-row: it writes the bytes from the segment that holds its first row on,
        // and leaves what follows its last whole segment to the next tile.
        auto full = [&](auto read, auto first) { // all pieces are whole; first: without the first segment of the k-rows
            u32x4 v[STEPS];
            uint32_t off[STEPS];
#pragma unroll
            for (int i = 0; i < STEPS; ++i) {
                const uint32_t from = part * 16u + SEG - past(krow(i));
                off[i] = krow(i) + from;
                v[i] = read(lane_lds + i * STEP_LDS + from);
            }
#pragma unroll
            for (int i = 0; i < STEPS; ++i)
                if (!decltype(first)::value || part >= PPS)
                    __builtin_nontemporal_store(v[i], reinterpret_cast<u32x4 *>(base + off[i]));
        };
        // The only tile of an expert, or one of 128 columns: the ends of its k-rows take the 16 bytes at the end, some of them once
        // more.  The first and the last of several tiles do without its tests and double stores at every step (through it 80 of 780 rows
        // took 182 us, 128 of 270 142, now 167 and 129); the only tile of an expert has both ends, which are better written together
        // with the rest (50 of 190 rows 28 us, in the others' way 35).
        const int n = (int)n_rows;
        auto lo_of = [&](int sh) { return tile_m == 0u ? 0 : -sh; }; // the bytes that are this tile's, from its first row
        auto hi_of = [&](int sh) { return last ? n : (int)TILE_M - sh; };
        auto clamped = [&](int at, int sh, bool *take) {
            const int lo = lo_of(sh), hi = hi_of(sh);
            *take = at + 16 > lo && at < hi;
            return (uint32_t)(min(max(at, lo), hi - 16) + (int)SEG);
        };
        auto ends = [&](auto read) {
            u32x4 v[STEPS];
            uint32_t off[STEPS];
            bool take[STEPS];
#pragma unroll
            for (int i = 0; i < STEPS; ++i) {
                const int sh = (int)past(krow(i));
                const uint32_t from = clamped((int)part * 16 - sh, sh, &take[i]);
                off[i] = krow(i) + from;
                v[i] = read(lane_lds + i * STEP_LDS + from);
            }
            const bool half = cols != TILE_K; // 128 columns: the even steps
#pragma unroll
            for (int i = 0; i < STEPS; ++i)
                if (take[i] && !((i & 1) && half)) {
                    // segments that another tile or k-row completes wait for it in the L2
                    const int sh = (int)past(krow(i)), seg0 = (int)(part / (SEG / 16u) * SEG) - sh;
                    u32x4_unaligned *dst = reinterpret_cast<u32x4_unaligned *>(base + off[i]);
                    if (seg0 >= lo_of(sh) && seg0 + (int)SEG <= hi_of(sh)) {
                        asm volatile("" : : "v"(tid)); // keeps the two forms of the store apart
                        __builtin_nontemporal_store(v[i], dst);
                        asm volatile("" : : "v"(tid));
                    } else {
                        *dst = v[i];
                    }
                }
        };
        // The segments of a last tile that it writes whole.
        auto before_the_end = [&](auto read) {
            u32x4 v[STEPS];
            uint32_t off[STEPS];
            bool take[STEPS];
#pragma unroll
            for (int i = 0; i < STEPS; ++i) {
                const int sh = (int)past(krow(i));
                const uint32_t from = (uint32_t)((int)(part * 16u + SEG) - sh);
                take[i] = (int)((part / PPS + 1u) * SEG) - sh <= n && !((i & 1) && cols != TILE_K); // 128 columns: the even steps
                off[i] = krow(i) + from;
                v[i] = read(lane_lds + i * STEP_LDS + from);
            }
#pragma unroll
            for (int i = 0; i < STEPS; ++i)
                if (take[i])
                    __builtin_nontemporal_store(v[i], reinterpret_cast<u32x4 *>(base + off[i]));
        };
        // One segment of every k-row that another k-row or tile completes, 16 k-rows to a wave instruction: the one that begins
        // seg_at(bytes by which the k-row is past the start of a segment) from the tile's first row.
        auto shared_segment = [&](auto seg_at) {
            constexpr int N = 32 * CPP / 16 / WAVES;
            u32x4 v[N];
            uint8_t *dst[N];
            bool take[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const uint32_t kr = 16u * (wv + WAVES * i) + lane / PPS, kt = (kr & 31u) * 8u + p * CPP + (kr >> 5);
                dst[i] = out_x + (size_t)(k0 + kt) * rows + m0 - SEG;
                const int sh = (int)((uint32_t)reinterpret_cast<uintptr_t>(dst[i]) & (SEG - 1u));
                const uint32_t from = clamped(seg_at(sh) + (int)(lane % PPS * 16u), sh, &take[i]);
                take[i] = take[i] && kt < cols;
                dst[i] += from;
                v[i] = read16(kr * ROW + from);
            }
#pragma unroll
            for (int i = 0; i < N; ++i)
                if (take[i])
                    *reinterpret_cast<u32x4_unaligned *>(dst[i]) = v[i];
        };
        auto last_segment = [&](int sh) { return ((n + sh) & ~(int)(SEG - 1u)) - sh; };
        auto clamped_pieces = [&] {
            if (by16 && (n_rows & 15u) == 0u)
                ends(aligned16);
            else
                ends(read16);
            if (last && n > (int)(TILE_M - SEG)) { // past the 256 bytes that begin before the first row of the tile
                for (uint32_t kr = tid / PPS; kr < 32u * CPP; kr += THREADS / PPS) {
                    const uint32_t kt = (kr & 31u) * 8u + p * CPP + (kr >> 5);
                    uint8_t *dst = out_x + (size_t)(k0 + kt) * rows + m0;
                    const int sh = (int)((uint32_t)reinterpret_cast<uintptr_t>(dst) & (SEG - 1u));
                    bool take;
                    const uint32_t from = clamped((int)(TILE_M + tid % PPS * 16u) - sh, sh, &take);
                    if (take && kt < cols)
                        *reinterpret_cast<u32x4_unaligned *>(dst - SEG + from) = read16(kr * ROW + from);
                }
            }
        };
        if (tile_m == 0u && last && rows >= 16u && !(whole && n_rows == TILE_M && cols == TILE_K)) {
            clamped_pieces(); // a copy of its own, where both ends are the k-rows': 50 of 190 rows 27.5 -> 26.2 us
        } else if (cols == TILE_K && ((whole && n_rows == TILE_M) || (look && !last))) {
            if (by16)
                full(aligned16, std::false_type{});
            else
                full(read16, std::false_type{});
        } else if (cols == TILE_K && !last) { // the first of several
            full(read16, std::true_type{});
            shared_segment([](int sh) { return -sh; });
        } else if (tile_m != 0u && last) {
            // The two halves of the segment at the end of a k-row meet in the L2; the other one, of the next k-row, is written at the
            // end of a pass (above).  A long last tile is there later than the first tile and writes its half first (128 of 500 rows
            // 178 -> 171 us), a short one sooner and writes it last (128 of 300, K = 2048, 42 -> 33).  In launches that the memory-side
            // cache holds, where the halves meet all the same, it is written last (Zipf-sized [65536, 2048] 47.5 -> 44.7).
            const bool early = a.stream != 0u && n_rows > SEG;
            if (early)
                shared_segment(last_segment);
            if (by16)
                before_the_end(aligned16);
            else
                before_the_end(read16);
            if (!early)
                shared_segment(last_segment);
        } else if (rows >= 16u) {
            clamped_pieces();
        } else {
            for (uint32_t kr = tid; kr < 32u * CPP; kr += THREADS) {
                const uint32_t kt = (kr & 31u) * 8u + p * CPP + (kr >> 5);
                if (kt < cols)
                    for (uint32_t i = 0; i < n_rows; ++i)
                        out_x[(size_t)(k0 + kt) * rows + m0 + i] = s_tile[kr * ROW + SEG + i];
            }
        }
        if (p + 1 < PASSES)
            __syncthreads();
    });
}

// upper bound on the number of tiles: every expert may end in a partial one
static int64_t tiles_at_most(int64_t M, int64_t K, int32_t num_experts)
{
    return ((M + TILE_M - 1) / TILE_M + num_experts) * ((K + TILE_K - 1) / TILE_K);
}

bool fp8_col_in_segments(int64_t M, int64_t K, int32_t num_experts, bool requant)
{
    return fp8_col_in_segments(M, K, num_experts, requant, compute_units());
}

hipError_t launch_row_to_fp8_col_grouped(const uint8_t *q_row, const uint8_t *sf_row, const int32_t *expert_offsets,
                                         int32_t num_experts, int64_t M, int64_t K, uint8_t *x_col, float *x_col_scale,
                                         bool requant, hipStream_t stream)
{
    fp8col_grouped::Args a;
    a.q_row = q_row;
    a.sf_row = sf_row;
    a.x_col = x_col;
    a.x_col_scale = x_col_scale;
    a.expert_offsets = expert_offsets;
    a.num_experts = num_experts;
    a.K = (uint32_t)K;
    a.tiles_k = (uint32_t)((K + TILE_K - 1) / TILE_K);
    a.by_tiles_k = FastDiv(a.tiles_k);
    a.stream = M * (K / 2) > KEEP_BYTES;
    const dim3 grid((uint32_t)((tiles_at_most(M, K, num_experts) + NUM_XCD - 1) / NUM_XCD * NUM_XCD));
    if (requant)
        hipLaunchKernelGGL(row_to_fp8_col_grouped_kernel<true>, grid, dim3(THREADS), 0, stream, a);
    else
        hipLaunchKernelGGL(row_to_fp8_col_grouped_kernel<false>, grid, dim3(THREADS), 0, stream, a);
    return hipGetLastError();
}

} // namespace mxfp4
