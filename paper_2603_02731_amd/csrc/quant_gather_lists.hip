// FP8 -> MXFP4 through a gather index, every source row quantized once, gfx950.
//
// The gather form names a source row for every output row; a dispatch map names each of them several times.  Two kernels: one
// turns the index around, into a workspace of the caller's (source row -> a short list of the output rows that want it); the other
// quantizes every source row once and writes it to the rows of its list, as the scatter form does.  8192 rows of 7168 to eight
// records each: 4.9 us and 59.9 us, which is what the scatter form takes (without a workspace 78.6); 65536 rows 16 and 455 (584).
#include "mxfp4_device.hpp"
#include "mxfp4_kernels.hpp"
#include "quant_rows.hpp"

#include <algorithm>

namespace mxfp4 {

// The index is cut into WINDOWS parts, each to SHARES workgroups that own the source rows of one residue each.  A source row's
// list has EACH places for every window, so that an entry's place is known inside its workgroup, without additions in global memory
// (a counter per source row there would have to be cleared by a kernel of its own, and takes 11 ns for every addition to the same
// address: 65536 entries that name one row 740 us).  Source rows that a window names more often, and entries that name no source
// row, go to the rest of the workgroup, the entries of one row next to each other.
// Lists are not cleared either: whoever reads a place checks that what is there is an output row of the window and wants the
// source row.  A place that was not written may pass by chance, or because an earlier call left it: then that output row gets the
// right bytes twice.
constexpr uint32_t WINDOWS = 32, EACH = 2, PLACES = WINDOWS * EACH, SHARES = 4, GROUPS = WINDOWS * SHARES;
constexpr uint32_t COPIES_MOST = 24; // of a row on the average, rounded down: a share of the rest is no more
static_assert(COPIES_MOST <= 64u, "a share is what a wave reads at once");
static_assert(PLACES == 64u && EACH == 2u, "a list is what a wave reads at once; its two entries of a window are neighbours");
static_assert(GROUPS == 128u && (SHARES & (SHARES - 1u)) == 0u, "two groups to a lane; shares by masks");

struct GatherListsArgs {
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
    uint32_t window;       // entries
    uint32_t counters;     // of a workgroup, a power of two
    uint32_t *lists;       // [M_src + 1][PLACES]; row M_src: entries that name no source row
    uint32_t *n_rest;      // [GROUPS]
    uint32_t *rest;        // [GROUPS][window]
    __device__ __forceinline__ uint32_t source(uint32_t out) const { return min((uint32_t)gather_idx[out], M_src); }
};

constexpr uint32_t BUILD_THREADS = 1024;
constexpr uint32_t COUNTERS_MOST = 32768; // 16 bits each: 64 KB of LDS

// HELD entries per lane are kept in registers; 0: there may be up to 32, and the index is read again for every step.
template <uint32_t HELD>
__global__ void __launch_bounds__(BUILD_THREADS) gather_lists_build_kernel(const GatherListsArgs a)
{
    // Entries per source row of ours (modulo `counters`: more rows share one), two to a dword; then where the next entry of a row
    // goes in the rest.
    extern __shared__ uint32_t s_count[];
    __shared__ uint32_t s_n;
    const uint32_t tid = threadIdx.x;
    const uint32_t window = blockIdx.x / SHARES, share = blockIdx.x % SHARES;
    const uint32_t first = window * a.window, end = min(first + a.window, a.M_out);
    const uint32_t each = HELD ? HELD : (a.window + BUILD_THREADS - 1u) / BUILD_THREADS;
    uint32_t src[HELD ? HELD : 1];
    auto entry = [&](uint32_t j) { return first + j * BUILD_THREADS + tid; };
    auto source = [&](uint32_t j) { return HELD ? src[HELD ? j : 0] : a.source(entry(j)); };
    auto half = [&](uint32_t row) { return row / SHARES & (a.counters - 1u); };
    auto count = [&](uint32_t h) { // the counter before
        return atomicAdd(&s_count[h >> 1], (h & 1u) ? 0x10000u : 1u) >> ((h & 1u) * 16u) & 0xFFFFu;
    };
    uint16_t *s_half = reinterpret_cast<uint16_t *>(s_count);
#pragma unroll
    for (uint32_t j = 0; j < HELD; ++j)
        src[j] = entry(j) < end ? a.source(entry(j)) : share + 1u; // not ours
    for (uint32_t i = tid; i < a.counters / 2u; i += BUILD_THREADS)
        s_count[i] = 0u;
    if (tid == 0u)
        s_n = 0u;
    __syncthreads();
    uint32_t ours = 0, is_first = 0, is_second = 0, to_rest = 0; // bit j: of its row's entries in the window; goes to the rest
#pragma unroll 16
    for (uint32_t j = 0; j < each; ++j) {
        if (entry(j) < end) {
            const uint32_t row = source(j);
            if (row % SHARES == share) {
                const uint32_t o = count(half(row));
                ours |= 1u << j;
                is_first |= (o == 0u ? 1u : 0u) << j;
                is_second |= (o == 1u ? 1u : 0u) << j;
            }
        }
    }
    __syncthreads();
    uint32_t room = 0; // in the rest, for the rows of which this lane has the first entry
#pragma unroll 16
    for (uint32_t j = 0; j < each; ++j) {
        if (ours >> j & 1u) {
            const uint32_t row = source(j), n = s_half[half(row)];
            if (n <= EACH) {
                a.lists[(size_t)row * PLACES + window * EACH + (is_second >> j & 1u)] = entry(j);
            } else {
                to_rest |= 1u << j;
                room += (is_first >> j & 1u) ? n : 0u;
            }
        }
    }
    if (__syncthreads_or((int)to_rest)) {
        uint32_t at = room != 0u ? atomicAdd(&s_n, room) : 0u;
        for (uint32_t left = to_rest & is_first; left != 0u; left &= left - 1u) {
            uint16_t *c = &s_half[half(a.source(entry((uint32_t)__ffs((int)left) - 1u)))];
            const uint32_t n = *c;
            *c = (uint16_t)at;
            at += n;
        }
        __syncthreads();
        for (; to_rest != 0u; to_rest &= to_rest - 1u) {
            const uint32_t e = entry((uint32_t)__ffs((int)to_rest) - 1u);
            a.rest[(size_t)blockIdx.x * a.window + count(half(a.source(e)))] = e;
        }
    }
    if (tid == 0u)
        a.n_rest[blockIdx.x] = s_n;
}

// The list of a source row: in lane i the output row at place i, if it is one of the window; then the lanes that hold one which
// wants the row.
__device__ __forceinline__ uint32_t listed_at(const GatherListsArgs &a, uint32_t row, uint32_t lane)
{
    const uint32_t out = a.lists[(size_t)row * PLACES + lane], first = lane / EACH * a.window;
    return out >= first && out < min(first + a.window, a.M_out) ? out : 0xFFFFFFFFu;
}

__device__ __forceinline__ uint64_t listed(uint32_t out, uint32_t source, uint32_t row, uint32_t lane)
{
    const bool twice = dpp_read<DPP_QUAD_XOR1>(out) == out && (lane & 1u) != 0u;
    return __ballot(out != 0xFFFFFFFFu && source == row && !twice);
}

// An equal share of the rest: a lane finds one entry, its output row and its source row, all lanes together, so that a share waits for
// them once and not for two loads in a chain per entry (us, a chain per entry / this way: copies of a row next to each other 8192 x 8 of
// 7168 82 / 78, 65536 x 8 624 / 606, 16384 x 8 of 2048 56 / 51, 65536 x 4 of 2048 125 / 115; a quarter of the entries naming one row there
// 102 / 99, every one 129 / 119; maps that leave little to the rest unchanged).
struct Rest {
    uint32_t n, all;      // lane i: entries of groups 2 i and 2 i + 1, 16 bits each
    uint32_t incl;        // lane i: entries up to and with these groups
    uint32_t i, end;
    __device__ __forceinline__ Rest(const u32x2 counts)
    {
        n = counts.x | counts.y << 16; // a window has at most 32768 entries
        incl = wave_inclusive_sum(counts.x + counts.y);
        all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
    __device__ __forceinline__ void share(uint32_t worker, uint32_t workers)
    {
        const uint32_t each = max((all + workers - 1u) / workers, 4u); // four at least: neighbours often want the same source row
        i = min(worker * each, all);
        end = min(i + each, all);
    }
    __device__ __forceinline__ static uint32_t of_lane(uint32_t v, uint32_t lane)
    {
        return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(lane * 4u), (int)v);
    }
    // Entry i + lane (the last one for the lanes past the end): its output row.
    __device__ __forceinline__ uint32_t output(const GatherListsArgs &a, uint32_t lane) const
    {
        const uint32_t t = min(i + lane, end - 1u);
        uint32_t l = 0; // the first lane whose groups end behind the entry
#pragma unroll
        for (uint32_t step = 32; step != 0u; step /= 2u)
            l += of_lane(incl, l + step - 1u) <= t ? step : 0u;
        const uint32_t two = of_lane(n, l), even = two & 0xFFFFu;
        const uint32_t at = t - (of_lane(incl, l) - even - (two >> 16));
        return a.rest[(size_t)(2u * l + (at < even ? 0u : 1u)) * a.window + (at < even ? at : at - even)];
    }
};

// A wave's share of the rest, elements [k0, k0 + n) of the rows.
template <bool WIDE_SF>
__device__ __forceinline__ void write_rest(const GatherListsArgs &a, const Rest &rest, uint32_t k0, uint32_t n, uint8_t *rec, uint32_t lane)
{
    uint32_t held = 0xFFFFFFFFu; // the source row in LDS
    if (rest.i == rest.end)
        return;
    const uint32_t dsts = rest.output(a, lane), srcs = a.source(dsts);
    for (uint32_t l = 0; l < rest.end - rest.i; ++l) {
        asm volatile("" : "+v"(lane)); // addresses are worked out where they are used: held over the loop they would spill
        const uint32_t dst = (uint32_t)__builtin_amdgcn_readlane((int)dsts, l), src = (uint32_t)__builtin_amdgcn_readlane((int)srcs, l);
        if (src != held) {
            held = src;
            const uint32_t from = src < a.M_src ? src : 0u;
            wave_fence(); // the copies of the row before are read
            quant_segment_into<2>(a.x + (size_t)from * a.K + k0, a.x_scale + (size_t)from * (a.K >> 7) + (k0 >> 7), n,
                                  src == a.M_src, rec, lane);
        }
        store_segment_on_lines<WIDE_SF>(rec, n, a.q + (size_t)dst * a.ld_q + k0 / 2u, a.sf + (size_t)dst * a.ld_sf + k0 / 32u, lane);
    }
}

// Long rows: a workgroup per source row; then its waves take their shares of the rest, where there is any.  Workgroups of their own
// for it cost 1.5 us per 1024 where there is none.
constexpr uint32_t REST_WAVES = 4; // of a workgroup: LDS for all eight would hold up the next workgroups

template <bool WIDE_SF>
__global__ void __launch_bounds__(ROW_THREADS, 8) gather_lists_row_kernel(const GatherListsArgs a, const bool records, const uint32_t seg)
{
    extern __shared__ __align__(16) uint8_t s_row[]; // a row, or WAVE_LDS for each of REST_WAVES
    const uint32_t tid = threadIdx.x, lane = tid & 63u, C = a.K / 16u;
    const uint32_t row = row_of_workgroup(blockIdx.x, a.M_src + 1u);
    const uint32_t out = listed_at(a, row, lane);
    const u32x2 counts = reinterpret_cast<const u32x2 *>(a.n_rest)[lane];
    if (__ballot(out != 0xFFFFFFFFu) != 0ull) {
        // the sources of what is listed and the row are on their way together
        uint32_t source = a.M_src + 1u;
        if (out != 0xFFFFFFFFu)
            source = a.source(out);
        if (row < a.M_src)
            quant_row_into(s_row, a.x + (size_t)row * a.K, a.x_scale + (size_t)row * (a.K >> 7), C, tid);
        else
            for (uint32_t c = tid; c < (C * 8u + C / 2u) / 4u; c += ROW_THREADS)
                reinterpret_cast<uint32_t *>(s_row)[c] = 0u;
        __syncthreads();
        for (uint64_t left = listed(out, source, row, lane); left != 0ull; left &= left - 1ull) {
            const uint32_t dst = (uint32_t)__builtin_amdgcn_readlane((int)out, __ffsll((unsigned long long)left) - 1);
            store_row<WIDE_SF>(s_row, a.q + (size_t)dst * a.ld_q, a.sf + (size_t)dst * a.ld_sf, C, records, tid);
        }
    }
    Rest rest(counts);
    if (rest.all == 0u)
        return;
    __syncthreads();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave >= REST_WAVES)
        return;
    for (uint32_t k0 = 0; k0 < a.K; k0 += seg) {
        rest.share(blockIdx.x * REST_WAVES + wave, (a.M_src + 1u) * REST_WAVES);
        write_rest<WIDE_SF>(a, rest, k0, min(seg, a.K - k0), s_row + wave * WAVE_LDS, lane);
    }
}

// Shorter rows: a wave per segment of a source row.
constexpr uint32_t LIST_WAVES = 4;

template <bool WIDE_SF>
__global__ void __launch_bounds__(64 * LIST_WAVES, 7) gather_lists_wave_kernel(const GatherListsArgs a, const uint32_t seg,
                                                                              const uint32_t segs_per_row)
{
    __shared__ __align__(16) uint8_t s_rec[LIST_WAVES][WAVE_LDS];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t unit = blockIdx.x * LIST_WAVES + wave;
    const uint32_t row = unit / segs_per_row, k0 = (unit - row * segs_per_row) * seg, n = min(seg, a.K - k0);
    if (row > a.M_src)
        return;
    const uint32_t out = listed_at(a, row, lane);
    const u32x2 counts = reinterpret_cast<const u32x2 *>(a.n_rest)[lane];
    if (__ballot(out != 0xFFFFFFFFu) != 0ull) {
        uint32_t source = a.M_src + 1u;
        if (out != 0xFFFFFFFFu)
            source = a.source(out);
        RowPieces r;
        const uint32_t from = row < a.M_src ? row : 0u;
        quant_segment<WIDE_SF>(a.x + (size_t)from * a.K + k0, a.x_scale + (size_t)from * (a.K >> 7) + (k0 >> 7), n, row == a.M_src,
                               s_rec[wave], lane, &r);
        for (uint64_t left = listed(out, source, row, lane); left != 0ull; left &= left - 1ull) {
            const uint32_t dst = (uint32_t)__builtin_amdgcn_readlane((int)out, __ffsll((unsigned long long)left) - 1);
            store_segment<WIDE_SF>(r, n, a.q + (size_t)dst * a.ld_q + k0 / 2u, a.sf + (size_t)dst * a.ld_sf + k0 / 32u, lane);
        }
    }
    Rest rest(counts);
    if (rest.all == 0u)
        return;
    rest.share(row, a.M_src + 1u);
    write_rest<WIDE_SF>(a, rest, k0, n, s_rec[wave], lane);
}

constexpr int64_t ENTRIES_MOST = (int64_t)WINDOWS * BUILD_THREADS * 32; // of an index

// Which calls.  What the two kernels save is the reading and quantizing of a row for each of its output rows (lane-wise kernel), or
// the owners' search and their one workgroup per compute unit; what they cost is the first of them, 5 us with its launch, and 3 us of
// the host.  Us, without a workspace / this way, records; routing maps; the same with a quarter of the entries naming one row; with
// 40 % naming none:
//   8192 x 8 copies of 7168 (470 million elements of output) 78.6 / 64.8, 83.7 / 74.1, 78.7 / 72.3; 65536 x 8 584 / 472, 614 / 532,
//   610 / 559; 65536 x 4 329 / 293, 363 / 325, 351 / 314; 65536 x 2 207 / 180; 4096 x 16 71 / 70; 2048 x 32 70 / 70; 2048 x 64 134 / 155
//   at the line, 4 copies or more: 4096 x 8 of 7168 (235) 38.4 / 37.1, 49.4 / 41.2, 40.0 / 40.1; 4096 x 8 of 8192 (268) 62 / 40,
//   52 / 46, 49 / 42; 8192 x 5 of 5120 (210) 51 / 39, 44 / 41, 39 / 40; 16384 x 8 of 2048 (268) 64 / 45, 55 / 50, 49 / 46;
//   65536 x 4 of 1536 (403) 98 / 69, -, 78 / 83, of 1280 (336) 85 / 68, -, 65 / 82;
//   below it: 8192 x 8 of 3072 (201) 38.3 / 34.6, 35.5 / 37.0, 35.2 / 37.5; 8192 x 8 of 2048 (134) 24.6 / 24.5, 24.3 / 30.3;
//   fewer copies: 32768 x 2 of 4096 (268) 68 / 55, 65 / 59, 60 / 57; 65536 x 2 of 2048 (268) 71 / 59, 66 / 67, 60 / 64;
//   below it: 32768 x 2 of 3072 (201) 50 / 45, 43 / 49, 37 / 48.
// Maps in which many rows have more than two entries in a window lose: 512 of 8192 rows named 128 times each at random 73 / 92, 1024 64
// times 72 / 114, 2048 32 times 74 / 86 (but a power law of exponent 1/4 97 / 85), and those with a row's copies next to each other:
// 8192 x 8 of 7168 74 / 78, 65536 x 8 556 / 606, 16384 x 8 of 2048 48 / 51 (but 65536 x 4 129 / 115).  Not kept for the latter: runs of
// up to eight entries as one, with their length (73, but routing maps 65.0 -> 65.6, of 2048 43.4 -> 44.7).
int64_t gather_lists_workspace(int64_t M_src, int64_t K, int64_t M_out, const uint8_t *q, int64_t ld_q)
{
    const bool many = M_out / 4 >= M_src;
    if (M_src <= 0 || K <= 0 || K >= (int64_t)1 << 31 || M_out / 2 < M_src || M_out / COPIES_MOST > M_src || M_out > ENTRIES_MOST ||
        K < (many ? 1536 : 2048) || M_out * K < (many ? (int64_t)220 << 20 : (int64_t)256 << 20) ||
        ((reinterpret_cast<uintptr_t>(q) | (uintptr_t)ld_q) & 15u) != 0u)
        return 0;
    const int64_t window = (M_out + WINDOWS - 1) / WINDOWS;
    return 4 * ((M_src + 1) * PLACES + GROUPS + window * GROUPS);
}

hipError_t launch_quant_gather_lists(const uint8_t *x, const float *x_scale, int64_t M_src, int64_t K, const int32_t *gather_idx,
                                     int64_t M_out, uint8_t *q, int64_t ld_q, uint8_t *sf, int64_t ld_sf, void *workspace,
                                     hipStream_t stream)
{
    GatherListsArgs a;
    a.x = x;
    a.x_scale = x_scale;
    a.gather_idx = gather_idx;
    a.q = q;
    a.sf = sf;
    a.ld_q = ld_q;
    a.ld_sf = ld_sf;
    a.M_src = (uint32_t)M_src;
    a.M_out = (uint32_t)M_out;
    a.K = (uint32_t)K;
    a.window = (a.M_out + WINDOWS - 1u) / WINDOWS;
    a.counters = 1024;
    while (a.counters < COUNTERS_MOST && a.counters <= a.M_src / SHARES)
        a.counters *= 2u;
    a.lists = static_cast<uint32_t *>(workspace);
    a.n_rest = a.lists + (size_t)(a.M_src + 1u) * PLACES;
    a.rest = a.n_rest + GROUPS;
    auto build = [&](auto n) {
        hipLaunchKernelGGL(gather_lists_build_kernel<decltype(n)::value>, dim3(GROUPS), dim3(BUILD_THREADS), a.counters * 2u, stream, a);
    };
    if (a.window <= 2u * BUILD_THREADS)
        build(std::integral_constant<uint32_t, 2>{});
    else if (a.window <= 8u * BUILD_THREADS)
        build(std::integral_constant<uint32_t, 8>{});
    else if (a.window <= 16u * BUILD_THREADS)
        build(std::integral_constant<uint32_t, 16>{});
    else
        build(std::integral_constant<uint32_t, 0>{});
    const bool wide = K % 512 == 0 && ((reinterpret_cast<uintptr_t>(sf) | (uintptr_t)ld_sf) & 15u) == 0u;
    const uint32_t rec = (uint32_t)((K / 2 + K / 32 + 15) & ~(int64_t)15);
    // Rows of one segment by waves unless there are five copies of them: K = 7168 (us, waves / workgroups) 65536 x 2 copies 180 / 244,
    // x 4 293 / 317, 16384 x 3 65 / 75, 8192 x 5 51.5 / 49.4, 16384 x 6 110 / 101, 8192 x 8 71 / 61; K = 6144 x 8 56 / 56; K = 8192 x 3
    // 67 / 78, x 5 52.4 / 52.7, x 6 112 / 110, x 8 70.6 / 67.6; K = 14336 x 2 346 / 355, x 3 117 / 113, x 8 124 / 116.
    const bool rows = K > 6144 && (M_out >= 5 * M_src || (K >= 12288 && M_out >= 3 * M_src)) && rec <= 48u * 1024u;
    uint32_t segs_per_row;
    const uint32_t seg = wave_segment(K, &segs_per_row);
    if (rows) {
        const bool records = sf == q + K / 2 && ld_sf == ld_q;
        const uint32_t lds = std::max(rec, REST_WAVES * (uint32_t)WAVE_LDS);
        if (wide)
            hipLaunchKernelGGL(gather_lists_row_kernel<true>, dim3(a.M_src + 1u), dim3(ROW_THREADS), lds, stream, a, records, seg);
        else
            hipLaunchKernelGGL(gather_lists_row_kernel<false>, dim3(a.M_src + 1u), dim3(ROW_THREADS), lds, stream, a, records, seg);
    } else {
        const dim3 grid(((a.M_src + 1u) * segs_per_row + LIST_WAVES - 1u) / LIST_WAVES);
        if (wide)
            hipLaunchKernelGGL(gather_lists_wave_kernel<true>, grid, dim3(64 * LIST_WAVES), 0, stream, a, seg, segs_per_row);
        else
            hipLaunchKernelGGL(gather_lists_wave_kernel<false>, grid, dim3(64 * LIST_WAVES), 0, stream, a, seg, segs_per_row);
    }
    return hipGetLastError();
}

} // namespace mxfp4
