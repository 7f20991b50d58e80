// Row-blocked MXFP4 -> column-blocked MXFP4 (stored transposed) in tiles that write whole 64-byte segments of the output, gfx950:
// large matrices whose k-rows are no whole segments (a multiple of 32 rows, not of 128).  The arithmetic is that of row_to_col.hip.
//
// A tile that writes the bytes of its own 256 rows shares the first and the last segment of every k-row with its neighbours, and
// what does not meet in the L2 in time costs the memory a read, modify and write.  Here a tile writes the bytes from the segment
// that holds its first row on, and leaves what follows its last whole segment to the next tile; for that it converts up to 128
// rows before its own once more.
//
// Work split.  A workgroup of 256 lanes owns a tile of 256 rows x 256 columns; lane (rg, cg) the rows 32*rg.. and the columns
// 8*cg.., and of the four 32-row blocks before the tile the one of its wave and four columns, two for either of the two passes
// in which the tile leaves (half a slice per lane: all lanes have the same work).  Rows and row scales of a wave's slices are
// fetched by the wave, so that a barrier is only needed where the tile buffer changes hands.  38 KB of LDS, four workgroups per
// compute unit (three: 118 -> 121 us at [65504, 7168]).
//
// Measured against row_to_col_kernel where one is chosen (launch_row_to_col): [65504, 7168] 146 -> 118 us, of which a mover of
// these pieces takes 103 to 110; [65536, 7168], whose k-rows are whole segments, takes row_to_col_kernel 90.  Bound by the
// pattern and by half as much arithmetic again.
#include "mxfp4_device.hpp"
#include "mxfp4_kernels.hpp"
#include "row_to_col_rule.hpp"
#include "row_to_col_slice.hpp"

namespace mxfp4 {

namespace row_to_col_seg {

constexpr uint32_t LOOK = 2 * SEG;           // the rows a tile's segments may hold before its own: one 32-row block per wave
constexpr uint32_t ROW = SEG + TILE_BYTES + 16; // bytes of an LDS k-row: an odd number of 16-byte slots
constexpr uint32_t SF = LOOK + TILE_M + 16;  // row-scale bytes of one k-block in LDS: the look-back rows, then the tile's

struct Args {
    const uint8_t *q_row;
    const uint8_t *sf_row;
    uint8_t *q_col;
    uint8_t *sf_col;
    uint32_t M;
    uint32_t K;
    uint32_t tiles_m; // 256-row tiles
    uint32_t tiles_k; // 256-column tiles
    uint32_t mbm;     // row tiles per macro block of the tile order
};

// Look-back slices: 32 rows of four columns, two rows to a dword (bytes: row i, row i, row i+1, row i+1; the first byte of
// either holds the columns of the first pass).
// Maxima of the four columns.
__device__ __forceinline__ void look_maxima(const uint32_t (&w)[16], const uint32_t (&sb)[8], float (&amax)[4])
{
#pragma unroll
    for (int c = 0; c < 4; ++c)
        amax[c] = 0.0f;
    static_for<16>([&](auto ip) {
        constexpr int r = decltype(ip)::value;
        const float sa = row_scale_operand<2 * r>(sb), sbb = row_scale_operand<2 * r + 1>(sb);
        static_for<2>([&](auto jp) {
            constexpr int j = decltype(jp)::value;
            const f32x2 fa = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[r], sa, j);
            const f32x2 fb = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[r], sbb, 2 + j);
            amax[2 * j] = max3_abs_nan(fa.x, fb.x, amax[2 * j]);
            amax[2 * j + 1] = max3_abs_nan(fa.y, fb.y, amax[2 * j + 1]);
        });
    });
}

// The 16 bytes of either column of pass P.
template <int P>
__device__ __forceinline__ void look_codes(const uint32_t (&w)[16], const uint32_t (&sb)[8], uint32_t cb0, uint32_t cb1,
                                           uint32_t (&o)[2][4])
{
    const float c0 = u2f(cb0 << 23), c1 = u2f(cb1 << 23);
#pragma unroll
    for (int g = 0; g < 4; ++g)
        asm volatile("" : "=v"(o[0][g]), "=v"(o[1][g])); // no initial value needed: all four bytes are written
    static_for<16>([&](auto ip) {
        constexpr int r = decltype(ip)::value, g = r >> 2, sel = r & 3;
        const f32x2 fa = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[r], row_scale_operand<2 * r>(sb), P);
        const f32x2 fb = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[r], row_scale_operand<2 * r + 1>(sb), 2 + P);
        o[0][g] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(o[0][g], fa.x, fb.x, c0, sel);
        o[1][g] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(o[1][g], fa.y, fb.y, c1, sel);
    });
}

// The integer path, by columns.
__device__ __noinline__ uint32_t slow_byte(const uint8_t *src, size_t src_pitch, const uint8_t *row_sf, int c)
{
    return column_byte_int(src, src_pitch, row_sf, c, 32);
}

__device__ __noinline__ void slow_codes(const uint8_t *src, size_t src_pitch, const uint8_t *row_sf, int c, uint32_t bc, uint32_t *out)
{
    column_codes_int(src, src_pitch, row_sf, c, 32, bc, out);
}

} // namespace row_to_col_seg

using namespace row_to_col_seg;

__global__ void __launch_bounds__(THREADS, 4) row_to_col_segments_kernel(const row_to_col_seg::Args a)
{
    constexpr uint32_t TILE_BUFFER = 32 * CPP * ROW > WAVES * 8192 ? 32 * CPP * ROW : WAVES * 8192;
    __shared__ alignas(16) uint8_t s_tile[TILE_BUFFER];   // [cl*32 + cg][SEG look-back bytes, then the tile's]: a pass
    __shared__ alignas(16) uint8_t s_row_sf[8 * SF];      // [k-block of the tile][row]
    __shared__ alignas(16) uint8_t s_col_sf[TILE_K * 8];  // [slot c*32 + cg of column cg*8 + c][row group]

    uint32_t tile_m, tile_k;
    if (!tile_of_workgroup<4>(blockIdx.x, a.tiles_m, a.tiles_k, a.mbm, &tile_m, &tile_k))
        return;
    const uint32_t rows = a.M;
    const uint32_t m0 = tile_m * TILE_M;
    const uint32_t n_rows = min(TILE_M, rows - m0); // 32 to 256, whole blocks of 32
    const uint32_t n_rg = n_rows / 32u;
    const uint32_t k0 = tile_k * TILE_K;
    const uint32_t cols = min(TILE_K, a.K - k0); // 128 or 256
    const uint32_t Kb = a.K / 32u, pitch = a.K / 2u;
    const uint32_t pitch_q = rows / 2u, pitch_sf = rows / 32u;

    const bool look = tile_m != 0u; // no k-row is whole segments: M is no multiple of 128

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t rg = tid >> 5, cg = tid & 31u;
    const bool active = rg * 32u < n_rows && cg * 8u < cols;
    // the look-back slice: row block wv, column group lane / 2, of its columns 2h, 2h + 1 (first pass) and 4 + 2h, 5 + 2h
    const uint32_t cgl = lane >> 1, h = lane & 1u;
    const bool active_l = look && cgl * 8u < cols;
    const uint8_t *tile_src = a.q_row + (size_t)m0 * pitch + k0 / 2u;

    // ---- row scales: thread t takes row t of the tile, the lower half of wave v the 32 look-back rows of block v
    auto row_scales = [&](size_t row) {
        const uint8_t *p = a.sf_row + row * Kb + k0 / 32u;
        if (cols > 128u) // one request at any 4-byte alignment
            return u32x2(*reinterpret_cast<const u32x2_unaligned *>(p));
        return u32x2{*reinterpret_cast<const uint32_t *>(p), 0u};
    };
    u32x2 sfv = {0u, 0u}, sfl = {0u, 0u};
    if (tid < n_rows)
        sfv = row_scales(m0 + tid);
    if (look && lane < 32u)
        sfl = row_scales(m0 - LOOK + wv * 32u + lane);
    // ---- nibbles, 8 rows x 128 bytes per wave instruction: the wave's 64 rows of the tile, its 32 look-back rows
    const bool piece_in = (lane & 7u) * 32u < cols;
    auto piece_of = [&](int32_t row) { // row of the tile, negative before it
        return reinterpret_cast<const u32x4_unaligned *>(tile_src + (int64_t)row * pitch + (lane & 7u) * 16u);
    };
    u32x4 stage_v[8], stage_l[4];
    if (wv * 64u < n_rows && piece_in) {
        auto row_of = [&](int j) { return (int32_t)min(wv * 64u + j * 8u + (lane >> 3), n_rows - 1u); };
        if (wv < 2u) { // read once; the last 128 rows are the next tile's look-back
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
        for (int j = 0; j < 4; ++j)
            stage_l[j] = *piece_of((int32_t)(wv * 32u + j * 8u + (lane >> 3)) - (int32_t)LOOK);
    }

    // Rows and row scales that a wave's slices need are the wave's own: what goes through LDS here is ordered by fences.
    auto wave_fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    store_row_scales<SF>(s_row_sf, sfv, LOOK + tid, lane); // rows that do not exist as byte 0
    if (look && lane < 32u)
        store_row_scales<SF>(s_row_sf, sfl, wv * 32u + lane, lane);
    // which (row group, k-block) pairs of the wave hold a byte of 253 or more (beyond FP32, or NaN)
    auto specials = [&](const u32x2 v, uint32_t *low, uint32_t *high) {
        *low = *high = 0u;
        if (__ballot((bytes_from<3>(v.x) | bytes_from<3>(v.y)) != 0u) == 0ull)
            return;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint64_t m = __ballot(((v[j >> 2] >> (8 * (j & 3))) & 0xFFu) >= 253u);
            *low |= ((uint32_t)m != 0u ? 1u : 0u) << j;
            *high |= ((uint32_t)(m >> 32) != 0u ? 1u : 0u) << j;
        }
    };
    uint32_t sp_low, sp_high, sp_look, sp_none;
    specials(sfv, &sp_low, &sp_high);
    specials(look && lane < 32u ? sfl : u32x2{0u, 0u}, &sp_look, &sp_none);

    uint32_t w[32], wl[16];
    {
        u32x4 *st = reinterpret_cast<u32x4 *>(s_tile) + wv * 512u;
        const uint32_t *s_in = reinterpret_cast<const uint32_t *>(st);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            st[j * 64u + lane] = stage_v[j];
        wave_fence();
#pragma unroll
        for (int i = 0; i < 32; ++i)
            w[i] = s_in[(rg & 1u) * 1024u + i * 32 + cg];
        if (look) {
            wave_fence();
#pragma unroll
            for (int j = 0; j < 4; ++j)
                st[j * 64u + lane] = stage_l[j];
            wave_fence();
            const uint32_t sel = h ? 0x07050301u : 0x06040200u;
#pragma unroll
            for (int i = 0; i < 16; ++i)
                wl[i] = perm(s_in[(2 * i + 1) * 32 + cgl], s_in[2 * i * 32 + cgl], sel);
        }
    }

    // ---- step 1: the column scales of every slice
    const uint8_t *my_row_sf = &s_row_sf[(cg >> 2) * SF + LOOK + rg * 32u], *my_row_sf_l = &s_row_sf[(cgl >> 2) * SF + wv * 32u];
    const bool special = (((rg & 1u) ? sp_high : sp_low) >> (cg >> 2)) & 1u, special_l = (sp_look >> (cgl >> 2)) & 1u;
    uint32_t sb[8], sbl[8], cb[8], cbl[4]; // cb: the UE8M0 bytes; 255 for the columns of a NaN row scale
    auto scales_of = [&](const uint8_t *p, uint32_t(&s)[8]) {
        const u32x4 s0 = reinterpret_cast<const u32x4 *>(p)[0], s1 = reinterpret_cast<const u32x4 *>(p)[1];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            s[g] = s0[g];
            s[4 + g] = s1[g];
        }
    };
    const uint8_t *src = tile_src + (size_t)(rg * 32u) * pitch + cg * 4u;                     // the slice's first row
    const uint8_t *src_l = tile_src + ((int64_t)(wv * 32u) - LOOK) * (int64_t)pitch + cgl * 4u;
    if (active) {
        scales_of(my_row_sf, sb);
        if (!special) {
            column_scales_hw(w, sb, cb);
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c)
                cb[c] = slow_byte(src, pitch, my_row_sf, c);
        }
#pragma unroll
        for (int c = 0; c < 8; ++c)
            s_col_sf[(c * 32 + cg) * 8u + rg] = (uint8_t)cb[c];
    }
    if (active_l) {
        scales_of(my_row_sf_l, sbl);
        if (!special_l) {
            float amax[4];
            look_maxima(wl, sbl, amax);
#pragma unroll
            for (int c = 0; c < 4; ++c)
                cbl[c] = max(f2u(amax[c]) >> 23, 2u) - 2u;
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                cbl[c] = slow_byte(src_l, pitch, my_row_sf_l, 2 * (int)h + (c & 1) + (c >> 1) * 4);
        }
    }
    __syncthreads();

    // ---- the column scales leave, one request per k-row
    const uint32_t sf_k = (tid & 31u) * 8u + (tid >> 5); // slot tid of the staged column scales is column sf_k
    if (sf_k < cols) {
        uint8_t *dst = a.sf_col + (size_t)(k0 + sf_k) * pitch_sf + m0 / 32u;
        const u32x2 v = *reinterpret_cast<const u32x2 *>(&s_col_sf[tid * 8u]);
        // at any alignment: 8 bytes for a full tile, the pieces of store_head_bytes for a tile that ends early
        if (n_rg == 8u)
            *reinterpret_cast<u64_unaligned *>(dst) = ((uint64_t)v.y << 32) | v.x;
        else
            store_head_bytes(dst, u32x4{v.x, v.y, 0u, 0u}, n_rg);
    }

    const bool last = m0 + TILE_M >= rows;
    const int n = (int)(n_rows / 2u); // bytes of the tile in a k-row
    static_for<PASSES>([&](auto pp) {
        constexpr int p = decltype(pp)::value;
        if (p != 0) { // the operands are cheaper made again than kept in registers while the first pass leaves
#pragma unroll
            for (int q = 0; q < 8; ++q)
                asm volatile("" : "+v"(sb[q]), "+v"(sbl[q]));
        }
        // ---- step 2: the columns of this pass
        if (active) {
            uint8_t *my = s_tile + cg * ROW + SEG + rg * 16u;
            if (!special) {
                uint32_t o[CPP][4];
                requant_columns_hw<p * CPP / 2, CPP / 2>(w, sb, cb, o);
#pragma unroll
                for (int c = 0; c < CPP; ++c)
                    *reinterpret_cast<u32x4 *>(my + c * 32u * ROW) = u32x4{o[c][0], o[c][1], o[c][2], o[c][3]};
            } else {
#pragma unroll
                for (int c = 0; c < CPP; ++c)
                    slow_codes(src, pitch, my_row_sf, p * CPP + c, cb[p * CPP + c],
                               reinterpret_cast<uint32_t *>(my + c * 32u * ROW));
            }
        }
        if (active_l) {
            uint8_t *my = s_tile + (2u * h * 32u + cgl) * ROW + wv * 16u;
            if (!special_l) {
                uint32_t o[2][4];
                look_codes<p>(wl, sbl, cbl[2 * p], cbl[2 * p + 1], o);
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    *reinterpret_cast<u32x4 *>(my + c * 32u * ROW) = u32x4{o[c][0], o[c][1], o[c][2], o[c][3]};
            } else {
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    slow_codes(src_l, pitch, my_row_sf_l, p * CPP + 2 * (int)h + c, cbl[2 * p + c],
                               reinterpret_cast<uint32_t *>(my + c * 32u * ROW));
            }
        }
        __syncthreads();

        // ---- out.  A wave instruction writes 8 k-rows of 8 lanes x 16 bytes, eight columns apart; step i of a wave has the LDS
        // k-rows 32 * i + 8 * wv.., i.e. the columns p * CPP + i of the column groups 8 * wv..
        constexpr int STEPS = CPP;
        const uint32_t part = lane & 7u;
        // k-row of the lane in step 0 and the tile's first byte, SEG bytes late: what is subtracted from an offset stays below SEG
        uint8_t *const base = a.q_col + (size_t)(k0 + wv * 64u + p * CPP) * pitch_q + m0 / 2u - SEG;
        // offsets of 32 bits: store_end, a condition of the launch
        const uint32_t lane_row = store_row<uint32_t>(lane, 0) * pitch_q;
        auto krow = [&](int i) { return lane_row + (uint32_t)i * pitch_q; }; // of step i, from base
        const uint32_t lane_lds = (wv * 8u + (lane >> 3)) * ROW;
        constexpr uint32_t STEP_LDS = 32 * ROW;
        // every k-row begins on 16 bytes, and so do the pieces
        auto piece16 = [&](uint32_t at) { return *reinterpret_cast<const u32x4 *>(s_tile + at); };
        // bytes by which a k-row is past the start of a segment
        const uint32_t base_low = (uint32_t)reinterpret_cast<uintptr_t>(base);
        auto past = [&](uint32_t row) { return (base_low + row) & (SEG - 1u); };
        // Every tile begins and ends on a segment of the k-row: it writes the bytes from the segment that holds its first row on,
        // and leaves what follows its last whole segment to the next tile.
        auto full = [&] { // all pieces are whole
            u32x4 v[STEPS];
            uint32_t off[STEPS];
#pragma unroll
            for (int i = 0; i < STEPS; ++i) {
                const uint32_t from = part * 16u + SEG - past(krow(i));
                off[i] = krow(i) + from;
                v[i] = piece16(lane_lds + i * STEP_LDS + from);
            }
#pragma unroll
            for (int i = 0; i < STEPS; ++i)
                __builtin_nontemporal_store(v[i], reinterpret_cast<u32x4 *>(base + off[i]));
        };
        // The first or last tile along m, or one of 128 columns: pieces before the first row and after the last are left out.
        auto lo_of = [&](int sh) { return tile_m == 0u ? 0 : -sh; }; // the bytes that are this tile's, from its first row
        auto hi_of = [&](int sh) { return last ? n : (int)TILE_BYTES - sh; };
        auto taken = [&](int at, int sh) { return at >= lo_of(sh) && at < hi_of(sh); }; // pieces are whole
        auto ends = [&] {
            u32x4 v[STEPS];
            uint32_t off[STEPS];
            bool take[STEPS];
#pragma unroll
            for (int i = 0; i < STEPS; ++i) {
                const int sh = (int)past(krow(i));
                const uint32_t from = (uint32_t)((int)(part * 16u + SEG) - sh);
                take[i] = taken((int)part * 16 - sh, sh);
                off[i] = krow(i) + from;
                v[i] = piece16(lane_lds + i * STEP_LDS + from);
            }
            if (wv * 64u >= cols) // a tile of 128 columns
                return;
#pragma unroll
            for (int i = 0; i < STEPS; ++i)
                if (take[i]) {
                    // segments that another tile or k-row completes wait for it in the L2
                    const int sh = (int)past(krow(i)), seg0 = (int)(part / (SEG / 16u) * SEG) - sh;
                    u32x4 *dst = reinterpret_cast<u32x4 *>(base + off[i]);
                    if (seg0 >= lo_of(sh) && seg0 + (int)SEG <= hi_of(sh)) {
                        asm volatile("" : : "v"(tid)); // keeps the two forms of the store apart
                        __builtin_nontemporal_store(v[i], dst);
                        asm volatile("" : : "v"(tid));
                    } else {
                        *dst = v[i];
                    }
                }
        };
        if (cols == TILE_K && look && !last) {
            full();
        } else {
            ends();
            if (last && n > (int)(TILE_BYTES - SEG)) { // past the 128 bytes that begin before the first row of the tile
                for (uint32_t kr = tid / (SEG / 16u); kr < 32u * CPP; kr += THREADS / (SEG / 16u)) {
                    const uint32_t kt = (kr & 31u) * 8u + p * CPP + (kr >> 5);
                    uint8_t *dst = a.q_col + (size_t)(k0 + kt) * pitch_q + m0 / 2u;
                    const int sh = (int)((uint32_t)reinterpret_cast<uintptr_t>(dst) & (SEG - 1u));
                    const int at = (int)(TILE_BYTES + tid % (SEG / 16u) * 16u) - sh;
                    const uint32_t from = (uint32_t)(at + (int)SEG);
                    if (taken(at, sh) && kt < cols)
                        *reinterpret_cast<u32x4 *>(dst - SEG + from) = piece16(kr * ROW + from);
                }
            }
        }
        if (p + 1 < PASSES)
            __syncthreads();
    });
}

hipError_t launch_row_to_col_segments(const uint8_t *q_row, const uint8_t *sf_row, int64_t M, int64_t K, uint8_t *q_col,
                                      uint8_t *sf_col, hipStream_t stream)
{
    row_to_col_seg::Args a;
    a.q_row = q_row;
    a.sf_row = sf_row;
    a.q_col = q_col;
    a.sf_col = sf_col;
    a.M = (uint32_t)M;
    a.K = (uint32_t)K;
    a.tiles_m = (uint32_t)((M + TILE_M - 1) / TILE_M);
    a.tiles_k = (uint32_t)((K + TILE_K - 1) / TILE_K);
    a.mbm = macro_block_rows(a.tiles_m);
    const uint32_t total = a.tiles_m * a.tiles_k;
    const dim3 grid((total + NUM_XCD - 1) / NUM_XCD * NUM_XCD);
    hipLaunchKernelGGL(row_to_col_segments_kernel, grid, dim3(THREADS), 0, stream, a);
    return hipGetLastError();
}

} // namespace mxfp4
