// Which transposing conversions go by tiles of 128 x 128 (col_small.hip).  Host code without HIP, so that the rule can be checked
// wherever there is a C++ compiler.
#pragma once

#include <cstdint>

namespace mxfp4 {

enum ColKind { COL_MXFP4, COL_ALIGN, COL_REQUANT };

namespace col_small {

constexpr uint32_t THREADS = 256, TILE = 128;
constexpr int EXPERTS_MAX = 256; // the lookup of more takes registers that cost a third of the waves

} // namespace col_small

// num_experts 0: one matrix.  units: compute units.
//
// All figures are us by tiles of 256 x 256 / by small ones, with every byte from and to HBM; of three matrices in turn; 256 compute units.
//
// One matrix: about three tiles per compute unit.
//    tiles                    row->col               alignment              re-quantization
//     704  [ 2816,4096]       6.89/6.89; 6.19/5.08   7.29/7.30; 6.63/5.28
//     704  [22528, 512]       6.55/5.66; 6.11/4.55   7.00/6.19; 6.50/5.07
//     768  [ 3072,4096]       6.99/7.22; 6.35/5.23                          8.07/7.30; 7.39/6.29
//     896                     7.07/8.68; 6.35/6.46   7.63/9.20; 6.80/8.06   8.35/8.79; 7.60/7.07
//
// Experts: the number of half tiles that their splits are expected to have per compute unit (h/u; each split ends in half a tile).  The
// larger tiles waste more on last ones, and in what splits at any row make of the k-rows, so that the lines lie higher; a total of whole
// groups of 128 rows may be that of padded splits, which waste less.
//   256 rows on the average and more, lines at 14, 12 and 12:
//     8.5  [ 8192,2048] in   8   12.2/ 9.5; 10.1/ 8.0   12.7/10.5; 11.5/ 9.6   15.7/11.6; 14.4/10.1
//    16.3  [16384,2048] in   4   15.9/16.5; 14.5/15.1   16.8/19.7; 14.6/18.5
//    17.0  [16384,2048] in  16                                                 19.4/18.7; 17.4/17.5
//    20.0  [ 8192,4096] in  32   16.5/15.5; 15.6/15.0
//   the same, padded, 10, 10 and 8:
//     9.0  [ 8704,2048] in   8                                                 10.6/ 9.4;  9.3/ 8.0
//    10.0  [18432,1024] in  32    9.1/ 8.1;  8.0/ 7.0   10.0/ 8.9;  8.9/ 8.6
//    16.4  [16512,2048] in   4                          14.4/16.8; 11.8/16.1   17.3/16.9; 16.0/16.2
//    18.0  [17408,2048] in  16   12.0/13.4; 10.7/12.7
//   less than 256 rows, which are no whole tile of the larger kind, 24, 12 and 15:
//    11.5  [ 7700,2048] in  64                          15.2/14.4; 13.5/13.8                          Zipf-sized
//    12.0  [ 8192,2048] in  64                          15.1/10.8; 13.3/10.2   21.4/11.6; 20.5/11.0
//    15.6  [12000,2048] in  64                          16.6/20.0; 14.4/18.8   19.0/18.1; 16.8/17.0   Zipf-sized
//    24.9  [17392,2048] in 128   19.9/15.3; 18.7/14.4   23.4/19.6; 18.8/18.4   25.8/20.2; 21.1/18.9
//   the same, padded, 15, 12 and 15:
//     7.6  [11392,1024] in  64                                                  9.4/ 6.4;  8.5/ 6.3
//    15.1  [11392,2048] in  64   11.1/ 9.0;  9.9/ 8.3   12.3/10.7; 11.0/10.6   13.7/10.2; 12.5/10.1
//    24.3  [16640,2048] in 128   12.5/12.2; 10.8/11.9   16.7/17.2; 14.5/16.0
//   64 rows and less waste three quarters of a larger tile and half of a small one; the lines, 56, 24 and 32, are where Zipf-sized
//   splits, most of whose rows are in a few experts, lose nothing either:
//    15.8  [ 2048,8064] in  32                          20.0/17.6; 17.5/16.5                          Zipf-sized, and these
//    28.0  [ 4096,7168] in  64                          30.7/29.4; 24.9/27.8   32.7/30.0; 29.0/28.5
//    55.6  [ 8190,7168] in 128     49/45;     45/43                              61/60;     54/56
//   112.0  [16384,7168] in 256     83/92;     78/89
//   32 rows and less, 336, 96 and 336, for alignment 336 up to 24 rows.  As far as was measured small tiles gain where the rows are
//   spread evenly (exponent 0.8 and less), 25 to 40 %; the lines are where Zipf-sized splits of exponent 1.2 lose on a first pass:
//    48.0  [ 4096,8192] in 128   42.9/33.1; 41.4/31.4   46.5/41.2; 41.2/39.4   53.4/43.9; 49.1/41.8   exponent 1.2, and these
//    84.0  [ 8192,7168] in 256   63.6/56.9; 65.0/57.5   71.5/72.0; 66.9/71.5   81.8/74.8; 79.9/74.3
//    96.0  [ 8192,8192] in 256   72.2/64.1; 72.8/64.7   80.0/81.0; 75.2/80.9   92.1/84.6; 90.2/84.2
//   168.0  [8192,14336] in 256    120/ 114;  120/ 115    138/ 148;  143/ 155    157/ 151;  163/ 160
//   336.0  [8192,28672] in 256    232/ 230;  238/ 234    276/ 300;  285/ 310    308/ 305;  319/ 319
//   154.0  [6144,14336] in 256    117/  97;  117/  99    128/ 126;  131/ 131    151/ 133;  152/ 137   24 rows
//   320.0  [4096,32768] in 256    238/ 181;  240/ 183    252/ 235;  257/ 243    304/ 251;  305/ 259   16 rows
//    84.0  [ 8192,7168] in 256   49.8/37.7; 49.7/36.9   68.8/42.2; 67.6/40.9   75.2/49.6; 74.9/48.3   equal, and these
//   336.0  [8192,28672] in 256    182/ 138;  181/ 133    255/ 156;  252/ 153    282/ 184;  280/ 181
// Every line also keeps the launch far below the 2^32 work items that one may have (col_small_workgroups).
constexpr bool col_in_small_tiles(int64_t M, int64_t K, int32_t num_experts, ColKind kind, int64_t units)
{
    const int64_t tiles_k = K / col_small::TILE, E = num_experts;
    auto pick = [kind](int64_t mxfp4, int64_t align, int64_t requant) {
        return kind == COL_MXFP4 ? mxfp4 : kind == COL_ALIGN ? align : requant;
    };
    if (E == 0) // quarters of a tile per compute unit
        return 4 * ((M + col_small::TILE - 1) / col_small::TILE * tiles_k) <= pick(11, 11, 12) * units;
    if (E > col_small::EXPERTS_MAX)
        return false;
    const bool padded = M % 128 == 0;
    const int64_t line = M <= 32 * E    ? pick(336, M <= 24 * E ? 336 : 96, 336)
                         : M <= 64 * E  ? pick(56, 24, 32)
                         : M < 256 * E  ? (padded ? pick(15, 12, 15) : pick(24, 12, 15))
                                        : (padded ? pick(10, 10, 8) : pick(14, 12, 12));
    return (2 * (M / col_small::TILE) + E) * tiles_k <= line * units;
}

// Workgroups of the launch: every expert may end in part of a tile.
constexpr int64_t col_small_workgroups(int64_t M, int64_t K, int32_t num_experts)
{
    return ((M + col_small::TILE - 1) / col_small::TILE + num_experts) * (K / col_small::TILE);
}

} // namespace mxfp4
