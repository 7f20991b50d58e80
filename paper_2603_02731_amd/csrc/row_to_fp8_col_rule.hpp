// Which FP8-column conversions of ragged experts go by tiles that write whole 64-byte segments (row_to_fp8_col_grouped.hip).  Host
// code without HIP, so that the rule can be checked wherever there is a C++ compiler.
#pragma once

#include <cstdint>

namespace mxfp4 {

// Of the launches that col_in_small_tiles leaves, those of about one round of the other kernels' workgroups (two per compute unit, one
// pass), as far as the number of tiles can be told, whose total row count says that the splits may be padded, are left to them: nothing
// is shared or the pieces are aligned, and what a workgroup takes longer here is not made up for.  Measured (us, own rows / segments,
// re-quantization): [10752, 2432] padded to 128 in one expert 10.9 / 11.3, [26112, 1152] in one 11.8 / 12.8, [18560, 1280] in 32
// 10.6 / 11.4, [9216, 2560] in 8 10.5 / 11.3, padded to 16 [17024, 1536] in 16 13.4 / 14.2; above the line, [16128, 2048] in 16
// 18.6 / 16.1, [11136, 3968] in one 18.8 / 15.6; not padded, [6180, 1280] in 16 12.1 / 10.6.  For scale alignment only totals that
// are multiples of 16 and not of 128: one of 128 may as well be that of un-padded splits, which lose more by their own rows than padded
// ones by segments ([4224, 3072] in 4 7.3 / 7.5, the same un-padded 11.9 / 10.1; [14208, 2048] in 4 10.2 / 9.8, 14.5 / 12.8).  Padded to
// 16: [5792, 4736] in 2 12.0 / 13.1, [46832, 512] in 100 11.9 / 13.0, [16624, 1536] in 2 11.3 / 11.8, but close to the line, in a second
// round, [17376, 1664] in 16 18.1 / 16.2.  Those kernels look for one of at most 128 experts: the longer lookup costs their flat form 1 %.
constexpr bool fp8_col_in_segments(int64_t M, int64_t K, int32_t num_experts, bool requant, int64_t units)
{
    const int64_t half_tiles = (M / 128 + num_experts) * ((K + 255) / 256); // experts end in half a tile each
    const bool padded = M % 16 == 0 && (requant || M % 128 != 0);
    return num_experts > 128 || !padded || 10 * half_tiles > 43 * units;
}

} // namespace mxfp4
