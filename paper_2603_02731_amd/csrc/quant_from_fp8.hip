// FP8 (E4M3 + FP32 1x128 scales) -> MXFP4 (packed E2M1 + UE8M0 per 1x32), gfx950.
//
// Paper sec. 3.1: SF = 2^ceil(log2(group_max / 6)) per 1x32 block, then RTNE onto E2M1.
// The element values are the FP8 values themselves, fl32(e4m3 * tile scale): nothing
// passes through BF16 (the direct FP8 -> FP4 path of the paper's contributions).
//
// Work split: one lane owns 16 consecutive elements (one 16-byte load), so a block of 32
// is a pair of lanes and a 128-tile is 8 lanes.  Per lane:
//   16 B load -> 8 x v_cvt_pk_f32_fp8 -> 16 x v_mul_f32 (the one FP32 rounding)
//   -> NaN-propagating |max| (v_maximum3_f32) -> one DPP exchange with the pair lane
//   -> exponent-field arithmetic for the UE8M0 byte -> 8 x v_cvt_scalef32_pk_fp4_f32
//   -> one 8-byte store of 16 nibbles; the tile's four scale bytes are gathered by DPP
//      into lane 0 of its 8 lanes and leave as one dword.
// HBM-bound: 1.03125 B read + 0.53125 B written per element.
#include "mxfp4_device.hpp"
#include "mxfp4_kernels.hpp"
#include "quant_rows.hpp"

#include <algorithm>

namespace mxfp4 {

// Lanes per workgroup (each lane takes QUANT_UNROLL chunks).  Dense rows: 512 x 2 runs; at [65536,7168] over
// rotated buffers 256 x 2 and 256 x 4 are as fast, 1024 x 2 is 5 % slower.  Gathered, strided and scattered rows: 256.
constexpr int QUANT_THREADS = 512;        // dense rows
constexpr int QUANT_THREADS_ROUTED = 256; // gathered, strided, scattered rows
constexpr int QUANT_UNROLL = 2;
// Cache policy, measured at [65536,7168] over rotated buffer sets (every byte from and to HBM): non-temporal
// loads and stores 109 us; non-temporal loads with plain stores 118 us (that form is the faster one, 104 against
// 107 us, only when the 250 MB of output are rewritten in place and stay in the memory-side cache); plain
// loads 121 us.  Gathered rows are read several times: plain loads with non-temporal stores 1012 us for the
// top-8 payload of 65536 tokens, plain both ways 1090 us, non-temporal loads with plain stores 1130 us.

struct QuantArgs {
    const uint8_t *x;
    const float *x_scale;
    const int32_t *gather_idx;
    uint8_t *q;
    uint8_t *sf;
    int64_t ld_q;
    int64_t ld_sf;
    uint32_t n_chunks;       // M_out * K / 16
    uint32_t chunks_per_row; // K / 16
    FastDiv row_of;          // by chunks_per_row
    uint32_t K;
    uint32_t M_src;
};

// store_streaming instead of the non-temporal hint, measured at [65536,7168] on one buffer set: the 8-byte nibble stores of the
// dense kernel 112.0 -> 112.1 us (no difference), its scale dwords 112 -> 121 us, the scattered rows
// 463 -> 466 us, gathered per-token records 1065 -> 1400 us: not used here.
//
// One workgroup covers QUANT_UNROLL runs of THREADS consecutive chunks; a lane takes chunk
// `tid` of each run, so every load and store instruction of a wave stays contiguous
// (1 KiB in, 512 B out) while each lane keeps QUANT_UNROLL loads in flight.
// DENSE: no gather and dense outputs -- every address is a multiple of the flat chunk index.
// KEEP: a dense output of KEEP_FROM to KEEP_BYTES, left in the memory-side cache.
template <bool DENSE, bool GATHER, bool KEEP, int THREADS>
__global__ void __launch_bounds__(THREADS) quant_from_fp8_kernel(const QuantArgs a)
{
    const uint32_t c0 = blockIdx.x * (THREADS * QUANT_UNROLL) + threadIdx.x;

    u32x4 w[QUANT_UNROLL];
    float s[QUANT_UNROLL];
    uint8_t *dst_q[QUANT_UNROLL];
    uint8_t *dst_sf[QUANT_UNROLL]; // the tile's four scale bytes (one aligned dword)
#pragma unroll
    for (int u = 0; u < QUANT_UNROLL; ++u) {
        const uint32_t c = c0 + u * THREADS;
        if (c >= a.n_chunks)
            break; // n_chunks is a multiple of 8: the 8 lanes of a tile leave together
        const uint8_t *src;
        const float *src_scale;
        bool valid = true;
        if (DENSE) {
            src = a.x + (size_t)c * 16;
            src_scale = a.x_scale + (c >> 3);
            dst_q[u] = a.q + (size_t)c * 8;
            dst_sf[u] = a.sf + (size_t)(c >> 3) * 4;
        } else {
            const uint32_t row = a.row_of(c);
            const uint32_t cc = c - row * a.chunks_per_row;
            uint32_t src_row = row;
            if (GATHER) {
                src_row = (uint32_t)a.gather_idx[row];
                valid = src_row < a.M_src; // also rejects negative indices
                src_row = valid ? src_row : 0u;
            }
            src = a.x + (size_t)src_row * a.K + (size_t)cc * 16;
            src_scale = a.x_scale + (size_t)src_row * (a.K >> 7) + (cc >> 3);
            dst_q[u] = a.q + (size_t)row * a.ld_q + (size_t)cc * 8;
            dst_sf[u] = a.sf + (size_t)row * a.ld_sf + (size_t)(cc >> 3) * 4;
        }
        if (!GATHER)
            w[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src));
        else
            w[u] = *reinterpret_cast<const u32x4 *>(src); // gathered rows are read several times
        s[u] = *src_scale;
        if (!valid) { // an out-of-range gather index yields a zero row
            w[u] = u32x4{0u, 0u, 0u, 0u};
            s[u] = 0.0f;
        }
    }

#pragma unroll
    for (int u = 0; u < QUANT_UNROLL; ++u) {
        if (c0 + u * THREADS >= a.n_chunks)
            break;
        uint32_t out[2], b;
        quant16(w[u], s[u], out, &b);
        if (KEEP)
            store_through(dst_q[u], u32x2{out[0], out[1]});
        else
            __builtin_nontemporal_store(u32x2{out[0], out[1]}, reinterpret_cast<u32x2 *>(dst_q[u]));

        // lanes 2j, 2j+1 of the tile's 8 hold block j's byte: gather the four into lane 0
        uint32_t t = b | (dpp_read<DPP_QUAD_XOR2>(b) << 8); // lanes 0,1: B0 | B1 << 8
        t |= row_shift_left4(t) << 16;                       // lane 0: ... | B2 << 16 | B3 << 24
        if ((threadIdx.x & 7u) == 0u) {
            *reinterpret_cast<uint32_t *>(dst_sf[u]) = t;
        }
    }
}

// The routing turned around: every source row is read and quantized once and written to each of
// its `fanout` destination rows (a token and its top-k experts), instead of being read and
// quantized again for every destination.  Same lane layout; dense source, strided outputs.
struct QuantScatterArgs {
    const uint8_t *x;
    const float *x_scale;
    const int32_t *dst_idx; // [M_src, fanout]
    uint8_t *q;
    uint8_t *sf;
    int64_t ld_q;
    int64_t ld_sf;
    uint32_t n_chunks;       // M_src * K / 16
    uint32_t chunks_per_row; // K / 16
    FastDiv row_of;          // by chunks_per_row
    uint32_t fanout;
    uint32_t M_out;
};

// The first HELD destinations are requested with the elements: behind a store a load would wait for it (stores and loads are
// counted together).  HELD 1, 4 or 8, the least that holds the fan-out, 8 for more: no branches between the loads, few that are
// not wanted.  Us, calls in a HIP graph with every byte from and to HBM, loads behind the conversion / this way:
// 1035 x 1024 to one row 3.1 / 2.6, 40000 x 640 11.8 / 10.6, 2285 x 1152 to three 4.6 / 4.0 and four 5.0 / 4.4, 2174 x 896 to seven
// 4.8 / 4.1, 65536 x 512 to eight 61 / 58, 65536 x 1024 to three 37.0 / 37.3, to eight 85.8 / 85.2.
template <int HELD>
__global__ void __launch_bounds__(QUANT_THREADS_ROUTED) quant_from_fp8_scatter_kernel(const QuantScatterArgs a)
{
    const uint32_t c0 = blockIdx.x * (QUANT_THREADS_ROUTED * QUANT_UNROLL) + threadIdx.x;

    // Destinations from j0 on of a row; past the fan-out one that no output has.
    auto destinations = [&](uint32_t row, uint32_t j0, uint32_t(&d)[HELD]) {
        const int32_t *dst = a.dst_idx + (size_t)row * a.fanout;
#pragma unroll
        for (int j = 0; j < HELD; ++j)
            d[j] = (uint32_t)dst[HELD == 1 ? j0 : min(j0 + j, a.fanout - 1u)];
#pragma unroll
        for (int j = 1; j < HELD; ++j)
            d[j] = j0 + j < a.fanout ? d[j] : 0xFFFFFFFFu;
    };
    u32x4 w[QUANT_UNROLL];
    float s[QUANT_UNROLL];
    uint32_t row[QUANT_UNROLL], d[QUANT_UNROLL][HELD];
#pragma unroll
    for (int u = 0; u < QUANT_UNROLL; ++u) {
        const uint32_t c = c0 + u * QUANT_THREADS_ROUTED;
        if (c >= a.n_chunks)
            break; // n_chunks is a multiple of 8: the 8 lanes of a tile leave together
        w[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(a.x + (size_t)c * 16));
        s[u] = a.x_scale[c >> 3];
        row[u] = a.row_of(c);
        destinations(row[u], 0u, d[u]);
    }

#pragma unroll
    for (int u = 0; u < QUANT_UNROLL; ++u) {
        const uint32_t c = c0 + u * QUANT_THREADS_ROUTED;
        if (c >= a.n_chunks)
            break;
        uint32_t out[2], b;
        quant16(w[u], s[u], out, &b);
        // lanes 2j, 2j+1 of the tile's 8 hold block j's byte: gather the four into lane 0
        uint32_t t = b | (dpp_read<DPP_QUAD_XOR2>(b) << 8); // lanes 0,1: B0 | B1 << 8
        t |= row_shift_left4(t) << 16;                       // lane 0: ... | B2 << 16 | B3 << 24

        const uint32_t cc = c - row[u] * a.chunks_per_row;
        for (uint32_t j0 = 0;;) {
#pragma unroll
            for (int j = 0; j < HELD; ++j) {
                if (d[u][j] >= a.M_out) // also skips negative entries and the slots past the fan-out
                    continue;
                __builtin_nontemporal_store(u32x2{out[0], out[1]},
                                            reinterpret_cast<u32x2 *>(a.q + (size_t)d[u][j] * a.ld_q + (size_t)cc * 8));
                if ((threadIdx.x & 7u) == 0u)
                    *reinterpret_cast<uint32_t *>(a.sf + (size_t)d[u][j] * a.ld_sf + (size_t)(cc >> 3) * 4) = t;
            }
            j0 += HELD;
            if (j0 >= a.fanout)
                break;
            destinations(row[u], j0, d[u]);
        }
    }
}

constexpr int SCATTER_WAVES = 4; // rows (or row segments) per workgroup, one per wave

template <bool WIDE_SF>
__global__ void __launch_bounds__(64 * SCATTER_WAVES) quant_from_fp8_scatter_wave_kernel(const QuantScatterArgs a,
                                                                                        const uint32_t M_src,
                                                                                        const uint32_t seg,
                                                                                        const uint32_t segs_per_row)
{
    __shared__ __align__(16) uint8_t s_rec[SCATTER_WAVES][WAVE_LDS];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t unit = blockIdx.x * SCATTER_WAVES + wave;
    const uint32_t row = unit / segs_per_row;
    if (row >= M_src)
        return;
    const uint32_t K = a.chunks_per_row * 16u;
    const uint32_t k0 = (unit - row * segs_per_row) * seg;
    const uint32_t n = min(seg, K - k0);
    RowPieces r;
    quant_segment<WIDE_SF>(a.x + (size_t)row * K + k0, a.x_scale + (size_t)row * (K >> 7) + (k0 >> 7), n, false,
                           s_rec[wave], lane, &r);
    const int32_t *dst = a.dst_idx + (size_t)row * a.fanout;
    for (uint32_t j = 0; j < a.fanout; ++j) {
        const uint32_t d = (uint32_t)dst[j];
        if (d < a.M_out) // also skips negative entries
            store_segment<WIDE_SF>(r, n, a.q + (size_t)d * a.ld_q + k0 / 2u, a.sf + (size_t)d * a.ld_sf + k0 / 32u, lane);
    }
}

// The scatter form for long rows: quant_row_into and store_row by a workgroup of ROW_THREADS lanes.
template <bool WIDE_SF>
__global__ void __launch_bounds__(ROW_THREADS) quant_from_fp8_scatter_row_kernel(const QuantScatterArgs a, const bool records)
{
    extern __shared__ __align__(16) uint8_t s_row[];
    const uint32_t tid = threadIdx.x, row = row_of_workgroup(blockIdx.x, gridDim.x);
    const uint32_t C = a.chunks_per_row; // 16-element chunks per row
    const int32_t *dst = a.dst_idx + (size_t)row * a.fanout;

    // the first eight destinations, requested before anything else (uniform over the workgroup)
    uint32_t d[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        d[j] = (uint32_t)j < a.fanout ? (uint32_t)dst[j] : 0xFFFFFFFFu;

    quant_row_into(s_row, a.x + (size_t)row * C * 16u, a.x_scale + (size_t)row * (C / 8u), C, tid);
    __syncthreads();

    for (uint32_t j0 = 0;;) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (d[j] < a.M_out) // skips negative entries and the slots past the fan-out
                store_row<WIDE_SF>(s_row, a.q + (size_t)d[j] * a.ld_q, a.sf + (size_t)d[j] * a.ld_sf, C, records, tid);
        j0 += 8u;
        if (j0 >= a.fanout)
            break;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            d[j] = j0 + j < a.fanout ? (uint32_t)dst[j0 + j] : 0xFFFFFFFFu;
    }
}

hipError_t launch_quant_from_fp8_scatter(const uint8_t *x, const float *x_scale, int64_t M_src, int64_t K,
                                         const int32_t *dst_idx, int32_t fanout, int64_t M_out, uint8_t *q,
                                         int64_t ld_q, uint8_t *sf, int64_t ld_sf, hipStream_t stream)
{
    QuantScatterArgs a;
    a.x = x;
    a.x_scale = x_scale;
    a.dst_idx = dst_idx;
    a.q = q;
    a.sf = sf;
    a.ld_q = ld_q;
    a.ld_sf = ld_sf;
    a.n_chunks = (uint32_t)(M_src * (K / 16));
    a.chunks_per_row = (uint32_t)(K / 16);
    a.row_of = FastDiv(a.chunks_per_row);
    a.fanout = (uint32_t)fanout;
    a.M_out = (uint32_t)M_out;
    const bool rows16 = ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(sf) | (uintptr_t)ld_q |
                          (uintptr_t)ld_sf) & 15u) == 0u;
    const bool wide = K % 512 == 0; // the scale bytes of a row are whole 16-byte pieces
    // Which kernel.  Source rows of 256 M elements and their copies in about 150 MB of records or planes (us: one lane
    // per chunk / one wave per row / one workgroup per row), copies grouped by expert:
    //   K = 512, 8 copies 60 / 62 / 170, 2 copies 51 / 102 / 397; K = 1024 44 / 45 / 92, 51 / 59 / 211;
    //   K = 2048 36 / 36 / 56, 50 / 49 / 119, 1 copy 41 / 37 / 101; K = 3072 43 / 41 / 42, 50 / 52 / 86, 41 / 37 / 72;
    //   K = 4096 34 / 33 / 35, 50 / 49 / 67, 40 / 36 / 57; K = 5120 45 / 40 / 36, 50 / 51 / 58, 40 / 37 / 50;
    //   K = 7168 43 / 38 / 37, 51 / 51 / 49, 40 / 37 / 41; 65536 tokens of 7168, 8 copies (2 GB) 598 / 520 / 480.
    // A wave per row leaves lanes idle below 1024 elements and has its stores contiguous above; a workgroup per row
    // writes the longest runs, which pays for long rows with several copies.  Between 4608 and 6144 elements
    // the workgroup needs four copies, and more of them than the memory-side cache takes in (wave / workgroup, 140, 300 and 600
    // million elements of records): K = 5632 8 copies 22 / 20, 46 / 42, 91 / 81, 4 copies 24 / 22, 51 / 44, 98 / 86, 2 copies 31 / 31,
    // 59 / 62, 115 / 127; K = 4608 8 copies 22 / 21, 48 / 43, 93 / 82, 4 copies 24 / 24, 52 / 47, 99 / 91; K = 6016 8 copies 18 / 19,
    // 38 / 38, 77 / 72, 4 copies 19 / 22, 45 / 42, 88 / 82.  Scale planes that are not on 16-byte boundaries stay with the
    // lanes (1860 rows of 8064, 4 copies 8.7 against 11.0 us by workgroups).
    // A lane per chunk has its elements and destinations on the way at once and waits for nothing else: it takes what has one copy (us,
    // wave or workgroup per row / lanes, every byte from and to HBM, calls in a HIP graph: 500 x 2048 2.9 / 2.6, 65536 x 2048 39.2 / 37.4,
    // 16000 x 7168 34.0 / 33.0, 65536 x 7168 125 / 122, but 100 x 2048 2.36 / 2.44) and small launches: 2000 x 2048 two, four and eight
    // copies 4.1 / 3.7, 4.8 / 4.1 and 6.1 / 5.3, 1000 x 4096 3.7 / 3.6, 4.6 / 4.0 and 5.7 / 5.1, 2000 x 3072 5.3 / 4.8, 6.2 / 5.6 and 8.8 /
    // 8.1, 150 x 7168 3.2 / 3.2, 3.6 / 3.4 and 4.4 / 4.2; above the lines 3000 x 4096 6.6 / 7.0, 8.2 / 8.1 and 13.1 / 13.1, 12000 x 2048
    // 11.8 / 11.5, 15.7 / 17.1 and 25.9 / 26.2, 600 x 7168 4.2 / 4.2, 4.8 / 4.8 and 6.1 / 6.3, 3000 x 7168 11.2 / 10.9, 14.9 / 16.7, 23.6 / 28.6.
    const bool lanes = fanout == 1 || M_src * K <= (K < 6144 ? (int64_t)6 << 20 : (int64_t)3 << 19);
    uint32_t segs_per_row;
    const uint32_t seg = wave_segment(K, &segs_per_row);
    const uint32_t rec = (uint32_t)((K / 2 + K / 32 + 15) & ~(int64_t)15);
    const int64_t units = M_src * segs_per_row;
    const bool many = K >= 4608 && fanout >= 4 && M_src * K >= ((int64_t)1 << 28) / fanout;
    if (rows16 && !lanes && (K >= 6144 || many) && rec <= 48u * 1024u) {
        const bool records = sf == q + K / 2 && ld_sf == ld_q;
        if (wide)
            hipLaunchKernelGGL(quant_from_fp8_scatter_row_kernel<true>, dim3((uint32_t)M_src), dim3(ROW_THREADS), rec,
                               stream, a, records);
        else
            hipLaunchKernelGGL(quant_from_fp8_scatter_row_kernel<false>, dim3((uint32_t)M_src), dim3(ROW_THREADS), rec,
                               stream, a, records);
        return hipGetLastError();
    }
    if (rows16 && !lanes && K >= 2048) {
        const uint32_t blocks = (uint32_t)((units + SCATTER_WAVES - 1) / SCATTER_WAVES);
        if (wide)
            hipLaunchKernelGGL(quant_from_fp8_scatter_wave_kernel<true>, dim3(blocks), dim3(64 * SCATTER_WAVES), 0, stream,
                               a, (uint32_t)M_src, seg, segs_per_row);
        else
            hipLaunchKernelGGL(quant_from_fp8_scatter_wave_kernel<false>, dim3(blocks), dim3(64 * SCATTER_WAVES), 0,
                               stream, a, (uint32_t)M_src, seg, segs_per_row);
        return hipGetLastError();
    }
    constexpr uint32_t per_block = QUANT_THREADS_ROUTED * QUANT_UNROLL;
    const uint32_t blocks = (a.n_chunks + per_block - 1) / per_block;
    if (fanout == 1)
        hipLaunchKernelGGL(quant_from_fp8_scatter_kernel<1>, dim3(blocks), dim3(QUANT_THREADS_ROUTED), 0, stream, a);
    else if (fanout <= 4)
        hipLaunchKernelGGL(quant_from_fp8_scatter_kernel<4>, dim3(blocks), dim3(QUANT_THREADS_ROUTED), 0, stream, a);
    else
        hipLaunchKernelGGL(quant_from_fp8_scatter_kernel<8>, dim3(blocks), dim3(QUANT_THREADS_ROUTED), 0, stream, a);
    return hipGetLastError();
}

// Gather by owners.  Every source row that several output rows ask for is read and quantized once: a workgroup owns
// source rows, scans the whole index for the output rows that want one of them, sorts these by source row in LDS, and its
// waves quantize each row and write it to all of its destinations.  No communication between workgroups and no scratch
// memory: all of them read the same index (a few bytes per output row against K * 17/32 written).
//
// Balance.  Routing maps ask for every token about equally often, and the owner of a row is a hash of it, so that sources
// of which only a part is in use (the first quarter, every eighth row) spread over all workgroups.  Where a few rows are
// asked for by many (output rows padded with one and the same index, say), every workgroup counts the same sample of the
// index per owner while it scans; the rows of an owner with a quarter more than its share, and the zero rows of indices
// that name no source row, are dealt out by output row: every workgroup takes those of its own slice of the outputs.
// Bound by the writes: 8192 rows of 7168 to eight records each 78 us = 4.0 TB/s of what has to move (lane-wise 119, where
// half is reading every row eight times from the memory-side cache and a quarter quantizing it as often; the scatter form
// of the same routing 60 us, without the scan and with four workgroups per compute unit), 20 thousand of a workgroup's 160
// thousand cycles before its first write.  One workgroup of 16 waves per compute unit: two of them at 64 registers spill.
// Maps of 65536 slots, 7168 long rows (us, lane-wise / by owners): shuffled 118 / 82, a quarter of the slots naming one row 101 / 84,
// the last of every 16 slots 116 / 85, all naming one row 83 / 70, half unused 88 / 82, the first 512 rows only 86 / 76, every
// eighth row 96 / 75, 128 rows at random 84 / 88, a power law (exponents 1/4 and 1/8) 96 / 96 and 92 / 93.  With 32768 slots:
// routes 60 / 41, one row in a quarter 52 / 48, half unused 45 / 43, first 512 rows 45 / 40, but 128 rows at random 43 / 49 and
// the power laws 48 / 56 and 46 / 52, where some owners just below the line have more to write than one compute unit can.
constexpr int OWNER_WAVES = 16;
constexpr uint32_t OWNER_THREADS = 64 * OWNER_WAVES;
constexpr uint32_t OWNER_GROUPS = 512; // workgroups at most: counters of the sample
constexpr uint32_t OWNER_ROWS = 256;   // source rows of a workgroup at most
constexpr uint32_t OWNER_LIST = 8192;  // output rows a workgroup sorts at a time
// What the list is sorted by: own rows, the owners of dealt rows, rows of zeros.
constexpr uint32_t KEY_DEALT = OWNER_ROWS, KEY_ZERO = KEY_DEALT + OWNER_GROUPS, OWNER_KEYS = (KEY_ZERO + 64) / 64 * 64;
constexpr uint32_t OWNER_UNITS = OWNER_KEYS + OWNER_WAVES;
constexpr uint32_t SLICE_RUN = 32;     // output rows that are dealt out together
constexpr uint32_t OUT_BITS = 21;
constexpr int VMCNT_0 = 0x0F70; // operand of s_waitcnt: no vector memory operation outstanding, the other counters at any value
static_assert(OWNER_LIST / 2 * OWNER_GROUPS <= 1u << OUT_BITS && OWNER_KEYS <= 1u << (32 - OUT_BITS), "key and output row in a dword");

struct QuantOwnerArgs {
    const uint8_t *x;
    const float *x_scale;
    const int32_t *gather_idx;
    uint8_t *q;
    uint8_t *sf;
    int64_t ld_q;
    int64_t ld_sf;
    uint32_t M_src;
    uint32_t M_out;
    uint32_t K;
    uint32_t seg;     // elements of a row taken at a time
    uint32_t shift;   // 2^shift workgroups
    uint32_t samples; // runs of four that are sampled
    uint32_t eighths; // of the steps in which they are
    uint32_t heavy;   // sampled indices above which an owner's rows are dealt out
    // The owner of a row: of every 2^shift consecutive ones each has another, in an order that changes from run to run.
    __device__ __forceinline__ uint32_t turn(uint32_t run) const { return __umul24(run, 77u); }
    __device__ __forceinline__ uint32_t owner(uint32_t row) const { return (row + turn(row >> shift)) & ((1u << shift) - 1u); }
    __device__ __forceinline__ uint32_t row(uint32_t owner, uint32_t run) const
    {
        return (run << shift) + ((owner - turn(run)) & ((1u << shift) - 1u));
    }
};

template <bool WIDE_SF, bool LINES>
__global__ void __launch_bounds__(OWNER_THREADS) quant_from_fp8_owner_kernel(const QuantOwnerArgs a)
{
    __shared__ __align__(16) uint8_t s_rec[OWNER_WAVES][WAVE_LDS]; // first the unsorted list, then the waves' rows
    __shared__ uint32_t s_sorted[OWNER_LIST];
    __shared__ __align__(16) uint32_t s_sample[OWNER_GROUPS][4]; // sampled indices per owner; by lane, as crowds add to one
    __shared__ uint32_t s_fill[OWNER_KEYS];     // output rows per key; then where the next one goes
    __shared__ uint32_t s_units[OWNER_UNITS];   // parts of the sorted list for one wave: start << 16 | entries
    __shared__ uint32_t s_n;
    static_assert(sizeof(s_rec) >= OWNER_LIST * sizeof(uint32_t), "the unsorted list fits into the waves' rows");
    uint32_t *s_list = reinterpret_cast<uint32_t *>(s_rec);

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // consecutive source rows, whose output rows are often neighbours too, belong to workgroups of one XCD: output rows share
    // 128-byte lines, which the XCD's L2 puts together
    const uint32_t me = a.shift < 3u ? blockIdx.x : (blockIdx.x % NUM_XCD << (a.shift - 3u)) + blockIdx.x / NUM_XCD;

    auto clear_list = [&] {
        for (uint32_t i = tid; i < OWNER_KEYS; i += OWNER_THREADS)
            s_fill[i] = 0u;
        if (tid == 0u)
            s_n = 0u;
    };
    auto push = [&](uint32_t key, uint32_t out) {
        const uint32_t at = atomicAdd(&s_n, 1u);
        if (at < OWNER_LIST) {
            s_list[at] = (key << OUT_BITS) | out;
            atomicAdd(&s_fill[key], 1u);
        }
    };
    auto sampled = [&](uint32_t owner) {
        const u32x4 n = *reinterpret_cast<const u32x4 *>(s_sample[owner]);
        return n.x + n.y + n.z + n.w;
    };

    // ---- the output rows in quads [q0, q1) of the index (and, at its end, the last one to three) that want a row of ours
    constexpr int STEP = 4;
    const uint32_t quads = a.M_out / 4u;
    const u32x4_unaligned *idx4 = reinterpret_cast<const u32x4_unaligned *>(a.gather_idx);
    auto scan = [&](uint32_t q0, uint32_t q1, bool sample) {
        for (uint32_t base = q0; base < q1; base += OWNER_THREADS * STEP) {
            u32x4 v[STEP];
#pragma unroll
            for (int u = 0; u < STEP; ++u) {
                const uint32_t p = base + u * OWNER_THREADS + tid;
                v[u] = u32x4{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
                if (p < q1)
                    v[u] = idx4[p];
            }
            // A wave samples `samples` of its four runs of 256 indices, in `eighths` of its steps; which ones changes from wave
            // to wave and step to step without a pattern.
            const uint32_t hash = (base / OWNER_THREADS * OWNER_WAVES + wave) * 0x9E3779B1u;
            const uint32_t turn = hash >> 30, some = sample && (hash >> 27 & 7u) < a.eighths ? a.samples : 0u;
#pragma unroll
            for (int u = 0; u < STEP; ++u) {
                const uint32_t p = base + u * OWNER_THREADS + tid;
                const uint32_t o[4] = {a.owner(v[u].x), a.owner(v[u].y), a.owner(v[u].z), a.owner(v[u].w)};
                if ((o[0] == me) | (o[1] == me) | (o[2] == me) | (o[3] == me)) // one branch for four: the scan is bound by its
                                                                               // instructions
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (o[e] == me && v[u][e] < a.M_src) // also not the negative ones
                            push(v[u][e] >> a.shift, p * 4u + e);
                if ((((uint32_t)u - turn) & 3u) < some)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (v[u][e] < a.M_src)
                            atomicAdd(&s_sample[o[e]][lane & 3u], 1u);
            }
        }
        if (q1 >= quads && tid < (a.M_out & 3u)) {
            const uint32_t out = q1 * 4u + tid, src = (uint32_t)a.gather_idx[out];
            if (a.owner(src) == me && src < a.M_src)
                push(src >> a.shift, out);
        }
    };

    // ---- the output rows of our slice, every 2^shift-th run of SLICE_RUN, that are dealt out
    auto scan_dealt = [&] {
        uint32_t t = tid;
        asm volatile("" : "+v"(t)); // where the lane begins is worked out here: held over the loop around it, it would spill
        for (uint32_t out = ((t / SLICE_RUN << a.shift) + me) * SLICE_RUN + t % SLICE_RUN; out < a.M_out;
             out += OWNER_THREADS << a.shift) {
            const uint32_t src = (uint32_t)a.gather_idx[out];
            if (src >= a.M_src)
                push(KEY_ZERO, out);
            else if (sampled(a.owner(src)) > a.heavy)
                push(KEY_DEALT + a.owner(src), out);
        }
    };

    // ---- sorts the list, with the first `keys` of its keys in use, and writes its rows
    auto write_rows = [&](uint32_t listed, uint32_t keys) {
        // A unit is a source row and its destinations; rows with more of them than a wave's share are cut into several.
        uint32_t most_log2 = 4;
        while (OWNER_WAVES << most_log2 < listed)
            ++most_log2;
        if (wave == 0u) {
            uint32_t before = 0, units = 0;
            for (uint32_t b = 0; b < keys; b += 64u) {
                const uint32_t c = s_fill[b + lane];
                const uint32_t incl = wave_inclusive_sum(c);
                const uint32_t parts = (c + (1u << most_log2) - 1u) >> most_log2;
                const uint32_t units_incl = wave_inclusive_sum(parts);
                const uint32_t start = before + incl - c;
                s_fill[b + lane] = start;
                for (uint32_t i = 0; i < parts; ++i) {
                    const uint32_t at = i << most_log2;
                    s_units[units + units_incl - parts + i] = (start + at) << 16 | min(c - at, 1u << most_log2);
                }
                before += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                units += (uint32_t)__builtin_amdgcn_readlane((int)units_incl, 63);
            }
            if (lane == 0u)
                s_n = units;
        }
        __syncthreads();
        for (uint32_t i = tid; i < listed; i += OWNER_THREADS) {
            const uint32_t e = s_list[i];
            s_sorted[atomicAdd(&s_fill[e >> OUT_BITS], 1u)] = e;
        }
        const uint32_t units = s_n;
        __syncthreads();
        __builtin_amdgcn_s_waitcnt(VMCNT_0);
        auto write = [&](auto on_lines) {
            constexpr bool ON_LINES = decltype(on_lines)::value;
            uint32_t lane = tid & 63u;
            asm volatile("" : "+v"(lane)); // either copy works out its addresses itself (8192 x 7168 to eight records 78.6 -> 78.0 us)
            for (uint32_t k0 = 0; k0 < a.K; k0 += a.seg) {
                const uint32_t n = min(a.seg, a.K - k0);
                RowPieces r;
                uint32_t held = 0xFFFFFFFFu; // the source row in r; M_src: zeros
                for (uint32_t u = wave; u < units; u += OWNER_WAVES) {
                    const uint32_t unit = __builtin_amdgcn_readfirstlane(s_units[u]);
                    const uint32_t end = (unit >> 16) + (unit & 0xFFFFu);
                    for (uint32_t j = unit >> 16; j < end; j += 64u) {
                        const uint32_t e = j + lane < end ? s_sorted[j + lane] : 0u;
                        const uint32_t key = e >> OUT_BITS, out = e & ((1u << OUT_BITS) - 1u);
                        uint32_t src = key < KEY_DEALT ? a.row(me, key) : a.M_src;
                        if (key >= KEY_DEALT && key < KEY_ZERO) // used at once: the wait for it, and for every store before it,
                            src = min((uint32_t)a.gather_idx[out], a.M_src); // stays on this side of the branch
                        const int some = (int)min(64u, end - j);
                        for (int l = 0; l < some; ++l) {
                            const uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)src, l);
                            const uint32_t d = (uint32_t)__builtin_amdgcn_readlane((int)out, l);
                            if (row != held) {
                                const bool zero = row == a.M_src;
                                const uint32_t from = zero ? 0u : row;
                                if (ON_LINES)
                                    wave_fence(); // the copies of the row before were read from LDS
                                quant_segment<WIDE_SF>(a.x + (size_t)from * a.K + k0,
                                                       a.x_scale + (size_t)from * (a.K >> 7) + (k0 >> 7), n, zero, s_rec[wave],
                                                       lane, &r);
                                // The loads are in.  Said here, and before the loop, no store has to wait for them, and with them
                                // for the stores before it, where the paths join.
                                __builtin_amdgcn_s_waitcnt(VMCNT_0);
                                held = row;
                            }
                            uint8_t *dq = a.q + (size_t)d * a.ld_q + k0 / 2u, *dsf = a.sf + (size_t)d * a.ld_sf + k0 / 32u;
                            if (ON_LINES)
                                store_segment_on_lines<WIDE_SF>(s_rec[wave], n, dq, dsf, lane);
                            else
                                store_segment<WIDE_SF>(r, n, dq, dsf, lane);
                        }
                    }
                }
            }
        };
        // A workgroup with a quarter more than its share of the output rows is waited for by all others and bound by its own compute
        // unit, where reading every copy from LDS costs 5 %: it keeps the row in registers (power law of exponent 1/8 111 -> 105 us;
        // the line at an eighth: routes 0.4 us slower).
        if (LINES && listed <= (a.M_out >> a.shift) + (a.M_out >> (a.shift + 2u)))
            write(std::true_type{});
        else
            write(std::false_type{});
    };

    // All of it at once, or, where that is more output rows than the list holds, first those that are dealt to us, then ours
    // from as much of the index at a time as cannot overflow the list.
    constexpr uint32_t PART = OWNER_LIST / 4u - 1u; // quads; the last part has up to three indices more
    if (tid < OWNER_GROUPS)
        *reinterpret_cast<u32x4 *>(s_sample[tid]) = u32x4{0u, 0u, 0u, 0u};
    bool own = true, whole = true, dealt = true;
    for (uint32_t q0 = 0, q1 = quads;;) {
        clear_list();
        __syncthreads();
        scan(q0, q1, whole);
        __syncthreads();
        if (whole)
            own = sampled(me) <= a.heavy; // else our rows are dealt out too
        const uint32_t own_listed = s_n;
        __syncthreads();
        if (!own) {
            clear_list();
            __syncthreads();
        }
        if (dealt)
            scan_dealt();
        __syncthreads();
        const uint32_t listed = s_n;
        __syncthreads();
        if (listed > OWNER_LIST) {
            whole = false;
            q1 = 0u;
            continue;
        }
        write_rows(listed, own && listed == own_listed ? (((a.M_src - 1u) >> a.shift) + 64u) & ~63u : OWNER_KEYS);
        if (whole || !own || q1 >= quads)
            break;
        dealt = false;
        q0 = q1;
        q1 = min(q0 + PART, quads);
        __syncthreads();
    }
}

// One workgroup per compute unit, or the next lower power of two.
static uint32_t owner_shift()
{
    const uint32_t most = std::min(compute_units(), OWNER_GROUPS);
    uint32_t shift = 0;
    while (2u << shift <= most)
        ++shift;
    return shift;
}

// Gather by owners: where every source row is asked for at least twice on average, there are at least four of them per
// workgroup, rows are long and what quantizing them once saves is well above the kernel's phases before the first write.  Per
// million elements the lane-wise kernel takes 0.245 us of output, this one 0.106 us of output and 0.158 us of source and 0.124 us
// per thousand source rows (on 256 compute units; fewer of them save more).  The line lies where maps with crowds and unused
// slots still lose nothing, not where routing maps begin to gain.  Measured on both sides of it (us, lane-wise / by owners;
// the same with a quarter of the slots naming one row; with 40 % unused; naming 512 rows): saving 28 us, 58600 x 4096 from an
// eighth as many rows 58 / 44, 49 / 49, 46 / 44, 43 / 39; 33500 x 7168 59 / 43, 51 / 50, 47 / 45, 46 / 42; rows of two
// segments, 29800 x 8064 60 / 42, but 52 / 56, 47 / 44, 46 / 40; saving 54, 57000 x 8064 115 / 75, 101 / 91, 89 / 76, 87 / 68; saving
// 14, 16700 x 7168 30 / 24, but 26 / 32, 25 / 26, 25 / 25; 3584 long rows, saving 28, 61 / 51, but
// 53 / 55, 48 / 51, 45 / 50; 2048 long ones, saving 27, 59 / 51, but 52 / 58, 46 / 52, 42 / 48.
static bool gather_by_owners(int64_t M_src, int64_t K, int64_t M_out, const uint8_t *q, int64_t ld_q)
{
    const int64_t groups = (int64_t)1 << owner_shift();
    if (K < 4096 || M_src < 4 * groups || M_src > OWNER_ROWS * groups || M_out < 2 * M_src ||
        M_out > OWNER_LIST / 2 * groups || ((reinterpret_cast<uintptr_t>(q) | (uintptr_t)ld_q) & 15u) != 0u)
        return false;
    const int64_t saved_fs = (139 * M_out - 158 * M_src) * K - 124000 * M_src; // in 10^-15 s, from the rates above
    return saved_fs >= (K > (int64_t)WAVE_SEG ? (int64_t)40000000000 : (int64_t)25000000000); // rows of one segment or more
}

hipError_t launch_quant_from_fp8(const uint8_t *x, const float *x_scale, int64_t M_src, int64_t K,
                                 const int32_t *gather_idx, int64_t M_out, uint8_t *q, int64_t ld_q,
                                 uint8_t *sf, int64_t ld_sf, hipStream_t stream)
{
    if (gather_idx && gather_by_owners(M_src, K, M_out, q, ld_q)) {
        QuantOwnerArgs o;
        o.x = x;
        o.x_scale = x_scale;
        o.gather_idx = gather_idx;
        o.q = q;
        o.sf = sf;
        o.ld_q = ld_q;
        o.ld_sf = ld_sf;
        o.M_src = (uint32_t)M_src;
        o.M_out = (uint32_t)M_out;
        o.K = (uint32_t)K;
        uint32_t segs_per_row;
        o.seg = wave_segment(K, &segs_per_row);
        o.shift = owner_shift();
        const uint32_t groups = 1u << o.shift;
        // as much of the index as gives 64 sampled indices per owner, a thirty-second of it at least
        o.samples = o.M_out >= 256u * groups ? 1u : o.M_out >= 128u * groups ? 2u : 4u;
        o.eighths = std::min(8u, std::max(1u, 2048u * groups / o.M_out));
        o.heavy = 5u * (o.M_out / 32u * o.samples * o.eighths / groups) / 4u + 8u;
        const bool wide = K % 512 == 0 && ((reinterpret_cast<uintptr_t>(sf) | (uintptr_t)ld_sf) & 15u) == 0u;
        // Long rows of one segment that do not begin on 64-byte segments leave by whole lines, read from LDS for every copy, so that
        // no wave instruction ends inside a segment.  Maps of 65536 slots, records or planes 16 bytes off (us, from registers / by
        // lines: routes; 40 % unused; a quarter of the slots naming one row; a power law of exponent 1/4): K = 6272 71.5 / 69.3,
        // 73.2 / 68.9, 77.2 / 77.6, 93.5 / 94.5; 6400 73.3 / 70.4, 74.5 / 70.1, 78.4 / 78.7, 94.9 / 96.0; 6656 78.7 / 75.2,
        // 80.8 / 75.9, 82.3 / 81.1, 98.0 / 97.3; 7168 80.0 / 77.6, 82.3 / 78.6, 83.9 / 83.8, 100.6 / 100.0; 7552 83.6 / 80.1,
        // 85.0 / 80.1, 88.7 / 88.6, 108.9 / 108.9; 7680 89.7 / 85.3, 91.8 / 86.7, 93.1 / 91.1, 115.4 / 115.2; 65536 x 8 copies of
        // 7168 608 / 585.  Shorter rows gain less and lose more where rows are asked for unevenly: 6144 73.9 / 72.1, 76.2 / 73.0,
        // 77.2 / 77.5, 89.5 / 90.6; 4224 53.1 / 51.7, 52.8 / 52.0, 58.5 / 60.6, 71.0 / 73.9.  On whole segments nothing is gained
        // (planes of 6272 66.8 / 67.3, 7552 77.7 / 78.2; 8064, two segments, 83.2 / 82.8).
        const bool lines = ((reinterpret_cast<uintptr_t>(q) | (uintptr_t)ld_q) & 63u) != 0u && K > 6144 && K <= (int64_t)WAVE_SEG;
        auto launch = [&](auto w, auto l) {
            hipLaunchKernelGGL((quant_from_fp8_owner_kernel<decltype(w)::value, decltype(l)::value>), dim3(groups),
                               dim3(OWNER_THREADS), 0, stream, o);
        };
        if (lines)
            wide ? launch(std::true_type{}, std::true_type{}) : launch(std::false_type{}, std::true_type{});
        else
            wide ? launch(std::true_type{}, std::false_type{}) : launch(std::false_type{}, std::false_type{});
        return hipGetLastError();
    }
    QuantArgs a;
    a.x = x;
    a.x_scale = x_scale;
    a.gather_idx = gather_idx;
    a.q = q;
    a.sf = sf;
    a.ld_q = ld_q;
    a.ld_sf = ld_sf;
    a.n_chunks = (uint32_t)(M_out * (K / 16));
    a.chunks_per_row = (uint32_t)(K / 16);
    a.row_of = FastDiv(a.chunks_per_row);
    a.K = (uint32_t)K;
    a.M_src = (uint32_t)M_src;
    const bool dense = gather_idx == nullptr && ld_q == K / 2 && ld_sf == K / 32;
    const uint32_t per_block = (dense ? QUANT_THREADS : QUANT_THREADS_ROUTED) * QUANT_UNROLL;
    const uint32_t blocks = (a.n_chunks + per_block - 1) / per_block;
    if (dense && M_out * (K / 2) >= KEEP_FROM && M_out * (K / 2) <= KEEP_BYTES)
        hipLaunchKernelGGL((quant_from_fp8_kernel<true, false, true, QUANT_THREADS>), dim3(blocks), dim3(QUANT_THREADS), 0,
                           stream, a);
    else if (dense)
        hipLaunchKernelGGL((quant_from_fp8_kernel<true, false, false, QUANT_THREADS>), dim3(blocks), dim3(QUANT_THREADS), 0,
                           stream, a);
    else if (gather_idx)
        hipLaunchKernelGGL((quant_from_fp8_kernel<false, true, false, QUANT_THREADS_ROUTED>), dim3(blocks),
                           dim3(QUANT_THREADS_ROUTED), 0, stream, a);
    else
        hipLaunchKernelGGL((quant_from_fp8_kernel<false, false, false, QUANT_THREADS_ROUTED>), dim3(blocks),
                           dim3(QUANT_THREADS_ROUTED), 0, stream, a);
    return hipGetLastError();
}

} // namespace mxfp4
