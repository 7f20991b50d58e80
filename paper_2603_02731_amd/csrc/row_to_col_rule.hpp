// Which flat row -> column conversions go by tiles that write whole 64-byte segments, and which grouped ones leave in aligned
// pieces.  Host code without HIP, so that the rules can be checked against the kernels' offsets wherever there is a C++ compiler.
#pragma once

#include <cstdint>

#include "col_small_rule.hpp"

namespace mxfp4 {
namespace row_to_col_seg {

constexpr uint32_t TILE_M = 256, TILE_K = 256, THREADS = 256, WAVES = 4;
constexpr uint32_t SEG = 64;                 // the segments of the output that a tile writes whole, in bytes
constexpr uint32_t TILE_BYTES = TILE_M / 2;  // of a k-row
constexpr int PASSES = 2, CPP = 8 / PASSES;  // the tile leaves in passes; columns of a lane per pass

// k-row that `lane` writes in step i, counted from its wave's first one.
template <class U>
constexpr U store_row(uint32_t lane, int i)
{
    return (U)(lane >> 3) * 8u + (U)i;
}

// Where the last piece of the last such k-row ends, counted as the kernel does from SEG bytes before the wave's first: its
// offsets have 32 bits.
constexpr uint64_t store_end(int64_t M) { return store_row<uint64_t>(63, CPP - 1) * (uint64_t)(M / 2) + SEG + TILE_BYTES; }

} // namespace row_to_col_seg

// One large matrix whose k-rows are no whole 64-byte segments: tiles that write whole ones, at the price of converting up to
// half as many rows once more.  Measured (us, own rows / segments): [65504, 7168] 146 / 119, [49120, 7168] 113 / 94,
// [32736, 7168] 75 / 66, [40032, 8192] 118 / 94, [57056, 5120] 93 / 80, [131040, 2048] 78 / 73, [49120, 4096] 65 / 57, but
// [32736, 4096] 41 / 42, [65504, 2048] 38 / 41, [16352, 7168] 36 / 40: what smaller ones leave half written meets in the
// memory-side cache.  Not for experts, whose last tiles cost as much as whole ones: 16 of 2585 rows, K = 7424, 81 / 92,
// [65533, 7168] in 32 Zipf-sized 139 / 134, in 128 142 / 157.  Nor from 145592128 rows on, where its store offsets would pass 2^32:
// those of the kernel that writes its own rows have 64 bits.
constexpr bool row_to_col_in_segments(int64_t M, int64_t K)
{
    return M % 128 != 0 && M * K >= (int64_t)176 << 20 && row_to_col_seg::store_end(M) <= (uint64_t)1 << 32;
}

// Experts whose k-rows begin at any byte, in at most one and a half tiles of 256 x 256 per compute unit: what an unaligned 16-byte
// store costs a wave to issue shows, and the pieces are put together on 16-byte boundaries (us, unaligned / aligned pieces, with every
// byte from and to HBM; of three matrices in turn: [22867,256] in 280 Zipf-sized 12.1 / 11.2 and 10.7 / 10.3, [13440,256] in 300
// 11.5 / 10.7 and 10.3 / 10.0, [1719,128] in 320 9.8 / 8.9 and 9.1 / 8.8, but [5966,256] in 300 10.0 / 10.3).  With more tiles the
// memory waits for the additional requests ([16384,2048] in 16 13.8 / 14.1, [65536,7168] in 32 158 / 170).  Up to as many experts as
// the small tiles take, which take nearly all such launches, it does not pay for the rest, totals that look padded and are not:
// [5760,3584] in 4 13.6 / 13.9 and 12.5 / 11.8, [6272,3456] in 2 13.3 / 14.1 and 11.8 / 12.1, sixteen of them 12.8 / 13.4 and 11.6 / 11.5.
constexpr bool row_to_col_in_aligned_pieces(int64_t M, int64_t K, int32_t num_experts, int64_t units)
{
    return num_experts > col_small::EXPERTS_MAX && 2 * ((M + 255) / 256 + num_experts) * ((K + 255) / 256) <= 3 * units;
}

static_assert(row_to_col_in_segments(145592096, 128) && !row_to_col_in_segments(145592128, 128), "offsets of 32 bits");

} // namespace mxfp4
