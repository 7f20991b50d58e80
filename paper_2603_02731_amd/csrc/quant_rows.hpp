// Shared by the FP8 -> MXFP4 quantizers: the arithmetic of 16 elements, and a source row that is quantized once and written
// to several output rows, by a wave or by a workgroup.
#pragma once

#include "mxfp4_device.hpp"

namespace mxfp4 {

// Quantize the lane's 16 elements given as four dwords of E4M3 bytes and the tile scale.
// Returns the 16 nibbles in out[0..1]; *scale_byte is the block's UE8M0 byte (identical
// in both lanes of the pair).
__device__ __forceinline__ void quant16(const u32x4 w, float s, uint32_t out[2], uint32_t *scale_byte)
{
    float v[16];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8(w[j], false);
        f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8(w[j], true);
        v[4 * j + 0] = lo.x * s;
        v[4 * j + 1] = lo.y * s;
        v[4 * j + 2] = hi.x * s;
        v[4 * j + 3] = hi.y * s;
    }
    float m = 0.0f;
#pragma unroll
    for (int j = 0; j < 16; j += 2)
        m = max3_abs_nan(v[j], v[j + 1], m);
    float other = u2f(dpp_read<DPP_QUAD_XOR1>(f2u(m)));
    m = __builtin_elementwise_maximum(m, other);

    uint32_t b = ue8m0_of_block_max(f2u(m));
    float sc = u2f(b << 23); // only the exponent field of the scale operand is used
    uint32_t r0 = 0, r1 = 0;
    r0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r0, v[0], v[1], sc, 0);
    r0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r0, v[2], v[3], sc, 1);
    r0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r0, v[4], v[5], sc, 2);
    r0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r0, v[6], v[7], sc, 3);
    r1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r1, v[8], v[9], sc, 0);
    r1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r1, v[10], v[11], sc, 1);
    r1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r1, v[12], v[13], sc, 2);
    r1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r1, v[14], v[15], sc, 3);
    const bool nan_block = b == 255u; // a NaN poisons the block: codes are zeroed
    out[0] = nan_block ? 0u : r0;
    out[1] = nan_block ? 0u : r1;
    *scale_byte = b;
}

// ---- one wave per row: the scatter of short rows and both gathers that quantize a row once
//
// A wave quantizes a segment of at most WAVE_SEG elements of one source row into its own 4 KiB of LDS (nibble bytes
// then scale bytes, as they sit in a per-token record), takes the finished bytes back as 16-byte pieces and writes
// them to every destination row.  No barrier: the waves of a workgroup are independent, which is what short rows need:
// with a workgroup of 512 lanes per 2048 elements three quarters of the lanes idle and every row waits for a barrier
// (65536 such rows, two copies each: 127 us; this form 49 us = 5.2 TB/s).  Bound by the writes; the pieces leave with
// non-temporal stores (65536 x 7168 gathered to eight records each: 603 us, plain stores 653; 16384 rows of 1536 the other
// way round, 46 against 43).
constexpr uint32_t WAVE_SEG = 7680; // 240 nibble pieces and 15 scale pieces: at most four 16-byte pieces per lane
constexpr int WAVE_CHUNKS = 8;      // 16-element chunks per lane
constexpr int WAVE_PIECES = 4;
constexpr int WAVE_LDS = 4096;

struct RowPieces {
    u32x4 v[WAVE_PIECES];
    uint32_t sf_dword;         // rows whose scale bytes are not whole 16-byte pieces: this lane's dword of them
};

// Elements [k0, k0 + n) of the source row at src / src_scale; n is a multiple of 128, of 512 with WIDE_SF.
// zero: the row of an index that names no source row.  Into the wave's LDS, and from there back as pieces.
// PARTS: what is loaded at once is the whole segment, or a half of it where registers are short.
template <int PARTS>
__device__ __forceinline__ void quant_segment_into(const uint8_t *src, const float *src_scale, uint32_t n, bool zero, uint8_t *rec,
                                                   uint32_t lane)
{
    const uint32_t n_chunks = n / 16u, nib_bytes = n / 2u;
    constexpr int AT_ONCE = WAVE_CHUNKS / PARTS;
#pragma unroll
    for (int part = 0; part < PARTS; ++part) {
        u32x4 w[AT_ONCE];
        float s[AT_ONCE];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {
            const uint32_t c = (part * AT_ONCE + u) * 64u + lane;
            w[u] = u32x4{0u, 0u, 0u, 0u};
            s[u] = 0.0f;
            if (c < n_chunks && !zero) { // the 8 lanes of a tile pass or fail together
                w[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + c * 16u));
                s[u] = src_scale[c >> 3];
            }
        }
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {
            const uint32_t c = (part * AT_ONCE + u) * 64u + lane;
            if (c < n_chunks) {
                uint32_t o[2], b;
                quant16(w[u], s[u], o, &b);
                uint32_t t = b | (dpp_read<DPP_QUAD_XOR2>(b) << 8); // lanes 0,1 of the tile: B0 | B1 << 8
                t |= row_shift_left4(t) << 16;                       // lane 0: ... | B2 << 16 | B3 << 24
                *reinterpret_cast<u32x2 *>(rec + c * 8u) = u32x2{o[0], o[1]};
                if ((lane & 7u) == 0u)
                    *reinterpret_cast<uint32_t *>(rec + nib_bytes + (c >> 3) * 4u) = t;
            }
        }
        if (PARTS > 1)
            __builtin_amdgcn_sched_barrier(0);
    }
    // the bytes of other lanes of this wave: ordered by the fence, no barrier of the workgroup needed
    wave_fence();
}

template <bool WIDE_SF>
__device__ __forceinline__ void quant_segment(const uint8_t *src, const float *src_scale, uint32_t n, bool zero,
                                              uint8_t *rec, uint32_t lane, RowPieces *out)
{
    quant_segment_into<1>(src, src_scale, n, zero, rec, lane);
    const uint32_t nib_bytes = n / 2u, nib_pieces = nib_bytes / 16u, pieces = nib_pieces + (WIDE_SF ? n / 512u : 0u);
#pragma unroll
    for (int i = 0; i < WAVE_PIECES; ++i) {
        const uint32_t p = i * 64u + lane;
        out->v[i] = u32x4{0u, 0u, 0u, 0u};
        if (p < pieces)
            out->v[i] = *reinterpret_cast<const u32x4 *>(rec + p * 16u);
    }
    out->sf_dword = 0u;
    if (!WIDE_SF && lane < n / 128u)
        out->sf_dword = *reinterpret_cast<const uint32_t *>(rec + nib_bytes + lane * 4u);
    // these reads of the LDS bytes come before the writes of the wave's next segment
    wave_fence();
}

// The finished segment to one destination: dq / dsf are where its nibbles and scale bytes start.
template <bool WIDE_SF>
__device__ __forceinline__ void store_segment(const RowPieces &r, uint32_t n, uint8_t *dq, uint8_t *dsf, uint32_t lane)
{
    const uint32_t nib_pieces = n / 32u, pieces = nib_pieces + (WIDE_SF ? n / 512u : 0u);
    // piece p of either kind sits 16 * p bytes after a base: the scale pieces follow the last nibble piece
    uint8_t *sf_base = dsf - n / 2u;
#pragma unroll
    for (int i = 0; i < WAVE_PIECES; ++i) {
        const uint32_t p = i * 64u + lane;
        if (p < pieces)
            __builtin_nontemporal_store(r.v[i], reinterpret_cast<u32x4 *>((p < nib_pieces ? dq : sf_base) + lane * 16u + i * 1024u));
    }
    if (!WIDE_SF && lane < n / 128u)
        *reinterpret_cast<uint32_t *>(dsf + lane * 4u) = r.sf_dword;
}

// The same from the wave's LDS, dealt to the lanes so that every wave instruction starts on a 128-byte line of the destination.
// A wave_fence has to follow before the LDS is written again.
template <bool WIDE_SF>
__device__ __forceinline__ void store_segment_on_lines(const uint8_t *rec, uint32_t n, uint8_t *dq, uint8_t *dsf, uint32_t lane)
{
    const uint32_t nib_pieces = n / 32u, pieces = nib_pieces + (WIDE_SF ? n / 512u : 0u);
    uint8_t *sf_base = dsf - n / 2u;
    const uint32_t shift = (uint32_t)(reinterpret_cast<uintptr_t>(dq) >> 4) & 7u;
    const uint32_t p0 = lane - shift; // wraps below zero for the lanes before the first piece
    u32x4 v[WAVE_PIECES];
#pragma unroll
    for (int i = 0; i < WAVE_PIECES; ++i) {
        const uint32_t p = p0 + i * 64u;
        v[i] = *reinterpret_cast<const u32x4 *>(rec + min(p, pieces - 1u) * 16u);
    }
#pragma unroll
    for (int i = 0; i < WAVE_PIECES; ++i) {
        const uint32_t p = p0 + i * 64u;
        if (p < pieces)
            __builtin_nontemporal_store(v[i], reinterpret_cast<u32x4 *>((p < nib_pieces ? dq : sf_base) + p * 16u));
    }
    if (pieces + shift > WAVE_PIECES * 64u) {
        const uint32_t p = p0 + WAVE_PIECES * 64u;
        if (p < pieces)
            __builtin_nontemporal_store(*reinterpret_cast<const u32x4 *>(rec + p * 16u),
                                        reinterpret_cast<u32x4 *>((p < nib_pieces ? dq : sf_base) + p * 16u));
    }
    if (!WIDE_SF && lane < n / 128u)
        *reinterpret_cast<uint32_t *>(dsf + lane * 4u) = *reinterpret_cast<const uint32_t *>(rec + n / 2u + lane * 4u);
}

// Elements per segment of a row that a wave takes at a time: equal parts of at most WAVE_SEG, in whole 512s.
inline uint32_t wave_segment(int64_t K, uint32_t *segs_per_row)
{
    const uint32_t n = (uint32_t)((K + WAVE_SEG - 1) / WAVE_SEG);
    const uint32_t seg = n == 1u ? (uint32_t)K : (uint32_t)((K / 128 + 4 * n - 1) / (4 * n)) * 512u;
    *segs_per_row = (uint32_t)((K + seg - 1) / seg);
    return seg;
}

// ---- one workgroup per row, for long rows: it quantizes the row into LDS (the K/2 nibble bytes followed by the
// K/32 scale bytes, as they sit in a per-token record) and writes it to each destination in 16-byte pieces, the
// whole row by one instruction per wave.  The pieces are dealt to the lanes so that every wave instruction starts
// on a 128-byte line of its destination (records of 3808 bytes start at any multiple of 32).
// Bound by the writes to many places: 65536 tokens of 7168, eight copies grouped by expert 508 -> 479 us = 5.2 TB/s with the
// pieces dealt that way (shuffled copies 553 -> 511; a kernel that only copies finished records: 477 and 500); 256 lanes and
// four workgroups per compute unit 484, 1024 lanes 584, one wave per row 520.
//
// Rows by runs of 32 to one XCD.  The copies of neighbouring source rows are often neighbours in the output, and records
// share lines and segments, which one L2 puts together but two do not.  Workgroup ids go round the eight XCDs, so in every
// 256 of them the rows are dealt in runs.  Us, row = id / runs of 4 / 16 / 32 / 64 / 256 / one eighth of the rows each:
// 65536 x 7168 to eight records grouped by expert 480 / 475 / 470 / 467 / 466 / 471 / 486, shuffled 508 / 508 / 503 / 501 / 501 /
// 503 / 504; two copies 171 -> 161, three of 30000 x 7680 103.5 -> 100.9.  Plain stores instead of non-temporal ones on top of
// that gain 2 % for copies grouped by expert and cost 15 % for shuffled ones; the waves of a workgroup dealt over the copies change
// nothing.  Few rows are all in flight at once: 512 rows of 7168, eight copies 7.5 -> 7.7, hence ROW_RUNS_FROM.
// The kernel of one wave per row gains nothing from runs (65536 x 2048, eight copies 139.7 -> 142.6).
constexpr int ROW_THREADS = 512;
constexpr uint32_t ROW_RUN = 32, ROW_RUNS_FROM = 2048;
static_assert((ROW_RUN & (ROW_RUN - 1u)) == 0u, "runs are taken apart by masks");

// The source row of workgroup `id`; the last rows, which do not fill a run for every XCD, in the order of the ids.
__device__ __forceinline__ uint32_t row_of_workgroup(uint32_t id, uint32_t rows)
{
    constexpr uint32_t ALL = NUM_XCD * ROW_RUN;
    if (rows < ROW_RUNS_FROM || id >= rows / ALL * ALL)
        return id;
    return id / ALL * ALL + id % NUM_XCD * ROW_RUN + id / NUM_XCD % ROW_RUN;
}

// The row of C 16-element chunks at src / src_scale into LDS: its nibble bytes, then its scale bytes.
__device__ __forceinline__ void quant_row_into(uint8_t *s_row, const uint8_t *src, const float *src_scale, uint32_t C, uint32_t tid)
{
    for (uint32_t c = tid; c < C; c += ROW_THREADS) { // the 8 lanes of a tile pass or fail together
        const u32x4 w = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + (size_t)c * 16u));
        const float s = src_scale[c >> 3];
        uint32_t out[2], b;
        quant16(w, s, out, &b);
        uint32_t t = b | (dpp_read<DPP_QUAD_XOR2>(b) << 8); // lanes 0,1 of the tile: B0 | B1 << 8
        t |= row_shift_left4(t) << 16;                       // lane 0: ... | B2 << 16 | B3 << 24
        *reinterpret_cast<u32x2 *>(s_row + c * 8u) = u32x2{out[0], out[1]};
        if ((tid & 7u) == 0u)
            *reinterpret_cast<uint32_t *>(s_row + C * 8u + (c >> 3) * 4u) = t;
    }
}

// The finished row to one destination: dq / dsf are where its nibbles and scale bytes start.  WIDE_SF: the K/32 scale bytes
// of a row are a whole number of 16-byte pieces (K % 512 == 0); records: they follow the nibbles.
template <bool WIDE_SF>
__device__ __forceinline__ void store_row(const uint8_t *s_row, uint8_t *dq, uint8_t *dsf, uint32_t C, bool records, uint32_t tid)
{
    const uint32_t nib_bytes = C * 8u, nib_pieces = nib_bytes / 16u, pieces = nib_pieces + (WIDE_SF ? C / 32u : 0u);
    const uint32_t shift = (uint32_t)(reinterpret_cast<uintptr_t>(dq) >> 4) & 7u;
    for (uint32_t i = tid; i < pieces + shift; i += ROW_THREADS) {
        const uint32_t p = i - shift;
        if (p < pieces) // wraps below zero for the lanes before the first piece
            __builtin_nontemporal_store(
                *reinterpret_cast<const u32x4 *>(s_row + p * 16u),
                reinterpret_cast<u32x4 *>(records || p < nib_pieces ? dq + p * 16u : dsf + (p - nib_pieces) * 16u));
    }
    if (!WIDE_SF)
        for (uint32_t i = tid; i < C / 8u; i += ROW_THREADS)
            *reinterpret_cast<uint32_t *>(dsf + i * 4u) = *reinterpret_cast<const uint32_t *>(s_row + nib_bytes + i * 4u);
}

} // namespace mxfp4
