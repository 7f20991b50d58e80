// Device-side helpers shared by the gfx950 conversion kernels.
//
// Hardware facts the kernels rely on (each checked exhaustively by the GPU parity tests):
//  * v_cvt_pk_f32_fp8 decodes OCP E4M3 exactly, subnormals and NaN included.
//  * v_cvt_scalef32_pk_fp4_f32 computes RTNE(src / 2^(E-127)) onto E2M1 with gradual
//    underflow and saturation, E being bits 30:23 of the scale operand (sign and mantissa
//    of the scale are ignored, E = 0 means 2^-127), keeps the sign of zero results, and
//    honours FP32 subnormal sources.
//  * v_cvt_scalef32_pk_f32_fp4 returns e2m1 * 2^(E-127) exactly, as FP32 subnormals where
//    needed.
//  * v_cvt_scalef32_pk_fp8_f32 computes RTNE(src / 2^(E-127)) onto OCP E4M3 with gradual
//    underflow, keeps the sign of zero results, and puts its first source in the low byte.
//  * v_maximum3_f32 propagates NaN.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace mxfp4 {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// The same through pointers of any alignment (global memory takes unaligned vector accesses).
typedef u32x4 __attribute__((aligned(1))) u32x4_unaligned;
typedef u32x2 __attribute__((aligned(1))) u32x2_unaligned;
typedef uint64_t __attribute__((aligned(1))) u64_unaligned;
typedef uint32_t __attribute__((aligned(1))) u32_unaligned;
typedef uint16_t __attribute__((aligned(1))) u16_unaligned;

__device__ __forceinline__ uint32_t f2u(float f) { return __builtin_bit_cast(uint32_t, f); }
__device__ __forceinline__ float u2f(uint32_t u) { return __builtin_bit_cast(float, u); }

// Byte permute: the result's byte i is byte sel[i] of the 8-byte pool {hi:lo}
// (selector values 0..3 pick from lo, 4..7 from hi).
__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel)
{
    return __builtin_amdgcn_perm(hi, lo, sel);
}

// Value of another lane of the same row of 16, selected by a DPP control.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_read(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
constexpr int DPP_QUAD_XOR1 = 0xB1; // quad_perm [1,0,3,2]
constexpr int DPP_QUAD_XOR2 = 0x4E; // quad_perm [2,3,0,1]
constexpr int DPP_ROW_HALF_MIRROR = 0x141; // lane i <-> lane 7-i inside each group of 8
constexpr int DPP_ROW_MIRROR = 0x140;      // lane i <-> lane 15-i inside each row of 16

// Value of lane i+4 of the same row of 16 lanes (0 where there is none), by DPP.
__device__ __forceinline__ uint32_t row_shift_left4(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x104 /* row_shl:4 */, 0xF, 0xF, true);
}

// Value of lane i+8 of the same row of 16 lanes (0 where there is none), by DPP.
__device__ __forceinline__ uint32_t row_shift_left8(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x108 /* row_shl:8 */, 0xF, 0xF, true);
}

// Bytes that lanes of a wave exchange through its LDS: what is in front of this is done before what follows.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// NaN-propagating maximum of |a|, |b| and c.
__device__ __forceinline__ float max3_abs_nan(float a, float b, float c)
{
    return __builtin_elementwise_maximum(
        __builtin_elementwise_maximum(__builtin_fabsf(a), __builtin_fabsf(b)), c);
}

// UE8M0 byte of the block scale for a block maximum given as FP32 bits (sign clear):
// the smallest k with gmax <= 6 * 2^k, biased by 127 and clamped to [0,254]
// (paper sec. 3.1, evaluated on the exponent field as in sec. 3.4).
// gmax = 1.f * 2^(e-127): gmax <= 6 * 2^k = 1.5 * 2^(k+2)  <=>  k = e-127-2 when f <= 1.5,
// one more otherwise.  Zero and FP32 subnormals land on byte 0 through the clamp,
// +inf gives 254, NaN gives 0xFF.
__device__ __forceinline__ uint32_t ue8m0_of_block_max(uint32_t gmax_bits)
{
    int e = (int)(gmax_bits >> 23);
    uint32_t mant = gmax_bits & 0x7FFFFFu;
    int b = e - 2 + (mant > 0x400000u ? 1 : 0);
    b = b < 0 ? 0 : b;
    b = gmax_bits == 0x7F800000u ? 254 : b;
    b = gmax_bits > 0x7F800000u ? 255 : b;
    return (uint32_t)b;
}

// Scale operand of row I of a 32-row slice whose UE8M0 bytes are packed four to a dword (byte
// I%4 of dword I/4): the byte moved into bits 30:23 with one shift.  What lands in the sign and
// mantissa bits belongs to the neighbouring bytes; the conversion instructions read the exponent
// field only.
template <int I>
__device__ __forceinline__ float row_scale_operand(const uint32_t (&sb)[8])
{
    constexpr int j = I & 3;
    return u2f(j == 3 ? sb[I >> 2] >> 1 : sb[I >> 2] << (23 - 8 * j));
}

// The row scales of a tile go to LDS as [k-block][row].  Lane t holds the 8 bytes of row `row`, rows of a quad of lanes being
// four consecutive ones on a multiple of 4: the four are byte-transposed inside the quad, so that lane q stores k-blocks q and
// 4 + q of all of them as a dword each (eight byte stores per lane otherwise).
template <uint32_t STRIDE>
__device__ __forceinline__ void store_row_scales(uint8_t *s_row_sf, const u32x2 v, uint32_t row, uint32_t lane)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t t = perm(dpp_read<DPP_QUAD_XOR1>(v[h]), v[h], (lane & 1u) ? 0x03070105u : 0x06020400u);
        t = perm(dpp_read<DPP_QUAD_XOR2>(t), t, (lane & 2u) ? 0x03020706u : 0x05040100u);
        *reinterpret_cast<uint32_t *>(&s_row_sf[(4u * h + (lane & 3u)) * STRIDE + (row & ~3u)]) = t;
    }
}

// Bit 7 of byte i is set where that byte of x is 256 - ADD or more: its top bit is set and its low seven bits plus ADD reach 128.
template <uint32_t ADD>
__device__ __forceinline__ uint32_t bytes_from(uint32_t x)
{
    return ((x & 0x7F7F7F7Fu) + ADD * 0x01010101u) & x & 0x80808080u;
}

// Workgroup -> tile for the transposing kernels.  The hardware deals consecutive workgroup ids
// round-robin to the 8 XCDs, each with its own L2.  Id i therefore takes entry i/8 of XCD (i%8)'s
// own contiguous share of a tile order in which mbm x MBK tiles form a macro block walked
// m-fastest: the tiles an XCD has in flight together are neighbours along m (their output pieces
// and their few-byte scale pieces complete whole lines in that L2) and along k (they share the
// 32-byte sectors of the row scales).  Returns false for the ids that round the grid up.
// mbm is chosen by the launch (macro_block_rows) so that an XCD's share is a whole number of macro
// rows: every XCD then walks its own band of row tiles from the first k tile to the last, all of
// them are at the same k at the same time, and the chip writes whole rows of the output together.
constexpr uint32_t NUM_XCD = 8;
__device__ __forceinline__ bool order_entry_of_workgroup(uint32_t id, uint32_t total, uint32_t *entry)
{
    const uint32_t per_xcd = (total + NUM_XCD - 1) / NUM_XCD;
    *entry = (id % NUM_XCD) * per_xcd + id / NUM_XCD;
    return id / NUM_XCD < per_xcd && *entry < total;
}

// Entry l of the macro-block walk over tiles_m x tiles_k tiles.
template <uint32_t MBK>
__device__ __forceinline__ void tile_of_order_entry(uint32_t l, uint32_t tiles_m, uint32_t tiles_k, uint32_t MBM,
                                                    uint32_t *tile_m, uint32_t *tile_k)
{
    const uint32_t per_macro_row = MBM * tiles_k;
    const uint32_t mg = l / per_macro_row;
    const uint32_t rem = l - mg * per_macro_row;
    const uint32_t mb_rows = min(MBM, tiles_m - mg * MBM);
    const uint32_t kg = rem / (MBK * mb_rows);
    const uint32_t rem2 = rem - kg * MBK * mb_rows;
    const uint32_t k_in = rem2 / mb_rows;
    *tile_m = mg * MBM + (rem2 - k_in * mb_rows);
    *tile_k = kg * MBK + k_in;
}

template <uint32_t MBK>
__device__ __forceinline__ bool tile_of_workgroup(uint32_t id, uint32_t tiles_m, uint32_t tiles_k, uint32_t mbm,
                                                  uint32_t *tile_m, uint32_t *tile_k)
{
    uint32_t l;
    if (!order_entry_of_workgroup(id, tiles_m * tiles_k, &l))
        return false;
    tile_of_order_entry<MBK>(l, tiles_m, tiles_k, mbm, tile_m, tile_k);
    return true;
}

// Row tiles per macro block for a matrix of tiles_m row tiles: an eighth of them, one band per XCD; halved
// while it exceeds 64 (a share is then 2, 4, ... macro rows).  Measured with row_to_col at K = 7168 over rotated
// buffers against a fixed 32: M = 49152 0.63 -> 0.67 of the HBM peak, 61440 0.58 -> 0.67, 73728 0.62 -> 0.685,
// 98304 0.67 -> 0.69; 65536 and 131072 (where an eighth, or a sixteenth, is 32) unchanged; a quarter or a
// sixteenth of the row tiles instead of an eighth: 1-4 % behind wherever they differ from this rule's choice,
// 6-18 % at M = 65536 and 131072.
inline uint32_t macro_block_rows(uint32_t tiles_m)
{
    uint32_t b = (tiles_m + NUM_XCD - 1) / NUM_XCD;
    while (b > 64u)
        b = (b + 1u) / 2u;
    return b ? b : 1u;
}

// Inclusive prefix sum over the 64 lanes of a wave, in the lanes' own registers (DPP): a scan
// inside each row of 16 lanes, then the last lane of row 0 (2) is added to row 1 (3), and lane 31
// to the upper half.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);  // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false); // row_bcast:15 -> rows 1, 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false); // row_bcast:31 -> rows 2, 3
    return v;
}

// n / d for a divisor known at launch, exact for every 32-bit n (Granlund and Montgomery, "Division by invariant
// integers using multiplication", 1994): a high multiplication and four cheap instructions instead of the 20 to 25 of a
// division, which the kernels over row-strided buffers would pay for every 16 elements.
struct FastDiv {
    uint32_t mul, shift; // shift = ceil(log2 d) - 1, d >= 2
    FastDiv() = default;
    explicit FastDiv(uint32_t d)
    {
        uint32_t l = 1;
        while (l < 32u && ((uint64_t)1 << l) < d)
            ++l;
        mul = (uint32_t)((((((uint64_t)1 << l) - d) << 32) / d) + 1u);
        shift = l - 1u;
    }
    __device__ __forceinline__ uint32_t operator()(uint32_t n) const
    {
        const uint32_t t = __umulhi(mul, n);
        return (t + ((n - t) >> 1)) >> shift;
    }
};

// Ragged inputs: workgroup -> (expert, row tile inside it, k tile).  Expert e contributes
// ceil(T_e / TILE_ROWS) row tiles, T_e = off[e+1] - off[e].  The order is expert after expert, each
// expert's tiles in the macro-block walk of tile_of_workgroup over its own row tiles: a macro block
// never spans two experts, whose outputs are separate matrices (a run of m-neighbours that crosses
// into the next expert continues at an unrelated address; measured with a kernel that only moves
// the nibbles of 32 experts of 2048 rows, K = 7168, every byte from and to HBM: 84 us with the
// macro blocks inside the experts, 96 us with 32 concatenated row tiles per block; 83 against 103 us
// at 512 rows per expert).  An expert that extends over several XCD shares gets macro blocks of its width over
// that number (mover: one expert of 61440 rows 95 -> 76 us, two of 30720 81 -> 76, the Zipf-sized and the equal
// experts of the configurations unchanged, three of 21760 82 -> 85).  The XCD shares are cut from this order with the number of tiles that
// really exist (the launch can only bound it: with the bound in its place the ids that round the
// grid up would all fall into the last XCD's share and the others would carry its tiles).
// Uniform per workgroup; every wave evaluates it on its own, 64 experts per lane-parallel step:
// the offsets of all experts (CHUNKS = 1, 2, 4 or 16 times 64) are requested at once and without branches
// between the requests, so the lookup waits for memory once, then wave prefix sums of the tile counts and
// a ballot find the expert.  It is in front of every load of the tile: with branches between the requests (a
// wait at each), the column tiles divided by and two more divisions in the macro block it took 2400 cycles
// of a lone workgroup, now 1600 (small splits 0.3-0.5 us, 128 experts of 65536 x 7168 4 %).
// On success `tile_m` is the tile index inside the expert and, for a non-zero UNIT_A / UNIT_B,
// `a_before` / `b_before` the sum of ceil(T_j / UNIT) over the experts before it (where its
// outputs start when the splits are not padded).
constexpr int MAX_EXPERTS = 1024; // MXFP4_MAX_EXPERTS of the C ABI

struct ExpertTile {
    uint32_t tile_m, tile_k; // tile_m: inside the expert
    uint32_t row_base, rows;
    uint32_t a_before, b_before;
};

// n / d for uniform n below 2^24 and d below 2^12: the compiler then divides in a few FP32 instructions.
__device__ __forceinline__ uint32_t small_div(uint32_t n, uint32_t d) { return (n & 0xFFFFFFu) / (d & 0xFFFu); }

template <int CHUNKS, uint32_t TILE_ROWS, uint32_t UNIT_A, uint32_t UNIT_B, uint32_t MBM_MAX>
__device__ __forceinline__ bool expert_tile(const int32_t *off, uint32_t num_experts, uint32_t id, uint32_t tiles_k,
                                            FastDiv by_tiles_k, ExpertTile *t)
{
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t lo[CHUNKS], len[CHUNKS];
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) { // all at once; lanes past the last expert see an empty one
        const uint32_t e = c * 64 + lane;
        lo[c] = (uint32_t)off[min(e, num_experts)];
        len[c] = (uint32_t)off[min(e + 1u, num_experts)];
    }
    uint32_t nt[CHUNKS], incl[CHUNKS], before[CHUNKS]; // tiles, their prefix sums inside the chunk, those of earlier chunks
    uint32_t total = 0;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        len[c] -= lo[c];
        nt[c] = (len[c] + TILE_ROWS - 1u) / TILE_ROWS;
        incl[c] = wave_inclusive_sum(nt[c]);
        before[c] = total;
        total += (uint32_t)__builtin_amdgcn_readlane((int)incl[c], 63);
    }
    uint32_t entry;
    if (!order_entry_of_workgroup(id, total * tiles_k, &entry))
        return false;
    const uint32_t tile = tiles_k == 1u ? entry : by_tiles_k(entry); // the expert whose row tiles include it holds the entry
    uint32_t a_chunks = 0, b_chunks = 0;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const uint32_t na = UNIT_A ? (len[c] + UNIT_A - 1u) / (UNIT_A ? UNIT_A : 1u) : 0u;
        const uint32_t nb = UNIT_B ? (len[c] + UNIT_B - 1u) / (UNIT_B ? UNIT_B : 1u) : 0u;
        const uint32_t a_incl = UNIT_A ? wave_inclusive_sum(na) : 0u, b_incl = UNIT_B ? wave_inclusive_sum(nb) : 0u;
        const uint64_t hit = __ballot(before[c] + incl[c] > tile);
        if (CHUNKS == 1 || hit != 0ull) {
            const int l = __ffsll((unsigned long long)hit) - 1;
            const uint32_t nt_e = (uint32_t)__builtin_amdgcn_readlane((int)nt[c], l);
            const uint32_t tiles_before = before[c] + (uint32_t)__builtin_amdgcn_readlane((int)incl[c], l) - nt_e;
            t->row_base = (uint32_t)__builtin_amdgcn_readlane((int)lo[c], l);
            t->rows = (uint32_t)__builtin_amdgcn_readlane((int)len[c], l);
            if (UNIT_A)
                t->a_before = a_chunks + (uint32_t)__builtin_amdgcn_readlane((int)(a_incl - na), l);
            if (UNIT_B)
                t->b_before = b_chunks + (uint32_t)__builtin_amdgcn_readlane((int)(b_incl - nb), l);
            // macro block: the expert's width over the number of XCD shares it extends over (one expert is
            // then walked like a single matrix, see macro_block_rows), halved while above MBM_MAX
            // (the divisions only for an expert of at least 1.5 shares)
            uint32_t mbm = nt_e;
            if (2u * NUM_XCD * nt_e >= 3u * total) {
                const uint32_t spans = (NUM_XCD * nt_e + total / 2u) / total;
                mbm = (nt_e + spans - 1u) / spans;
            }
            while (mbm > MBM_MAX)
                mbm = (mbm + 1u) / 2u;
            // the m-fastest walk of the macro row; that it goes by blocks of a few column tiles does not show in it
            const uint32_t l_in = entry - tiles_before * tiles_k, per_macro_row = mbm * tiles_k;
            const uint32_t mg = l_in < per_macro_row ? 0u : l_in / per_macro_row;
            const uint32_t rem = l_in - mg * per_macro_row, mb_rows = min(mbm, nt_e - mg * mbm);
            t->tile_k = per_macro_row <= 0xFFFFFFu ? small_div(rem, mb_rows) : rem / mb_rows;
            t->tile_m = mg * mbm + rem - t->tile_k * mb_rows;
            return true;
        }
        if (UNIT_A)
            a_chunks += (uint32_t)__builtin_amdgcn_readlane((int)a_incl, 63);
        if (UNIT_B)
            b_chunks += (uint32_t)__builtin_amdgcn_readlane((int)b_incl, 63);
    }
    return false; // not reached: tile < total
}

template <uint32_t TILE_ROWS, uint32_t UNIT_A, uint32_t UNIT_B, uint32_t MBM_MAX>
__device__ __forceinline__ bool tile_of_expert_workgroup(const int32_t *off, int32_t num_experts, uint32_t id, uint32_t tiles_k,
                                                         FastDiv by_tiles_k, ExpertTile *t)
{
    if (num_experts <= 64)
        return expert_tile<1, TILE_ROWS, UNIT_A, UNIT_B, MBM_MAX>(off, (uint32_t)num_experts, id, tiles_k, by_tiles_k, t);
    if (num_experts <= 256)
        return expert_tile<4, TILE_ROWS, UNIT_A, UNIT_B, MBM_MAX>(off, (uint32_t)num_experts, id, tiles_k, by_tiles_k, t);
    return expert_tile<MAX_EXPERTS / 64, TILE_ROWS, UNIT_A, UNIT_B, MBM_MAX>(off, (uint32_t)num_experts, id, tiles_k,
                                                                             by_tiles_k, t);
}

// Streaming stores for outputs that this kernel does not read again: the non-temporal hint together
// with the sc1 bit of the gfx940-family vector stores (the write goes through at device scope
// instead of waiting in the L2 for an eviction).  Measured at [65536,7168] with every byte going to HBM:
// the 16-byte E4M3 stores of the de-quantizer, written in address order by the whole grid, 115 -> 111 us
// against the non-temporal hint alone.  Where neighbouring workgroups complete each other's lines (the
// transposed rows of row_to_col: 93 -> 97 us) or the pieces are small, the hint alone is the better form.
// The builtin non-temporal store only sets the hint, hence the asm.
__device__ __forceinline__ void store_streaming(void *p, u32x4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc1 nt" : : "v"(p), "v"(v) : "memory");
}

// A packed matrix (its nibble bytes) up to this size is expected to be read again from the 256 MB memory-side cache:
// what is quantized is then de-quantized and transposed.  The dense quantizer sends such nibbles off with
// store_through, which passes them on like a streaming store but leaves them in that cache, and the de-quantizer reads
// them without the non-temporal hint, so that they stay there for the next reader.  Measured cold, rotated buffers of 900 MB
// (us, hints everywhere -> this):
//   nibbles         quantize, de-quantize, transpose   quantizer alone   de-quantizer alone
//    7.9 MiB [2304,7168]    21.6 -> 21.5 if it applied    7.25 ->  7.23     7.17 ->  7.15
//   10   MiB [2912,7168]    27.2 -> 24.8 if it applied    7.79 ->  7.98     7.98 ->  8.02
//   12   MiB [3520,7168]    29.5 -> 26.8                  8.81 ->  9.09     9.02 ->  9.03
//   14   MiB [4096,7168]    29.1 -> 26.0                  9.75 -> 10.01     9.94 -> 10.11
//   16   MiB [4672,7168]    35.3 -> 32.5                 10.44 -> 10.80    11.36 -> 11.39
//   28   MiB [8192,7168]    50.9 -> 42.3                 16.30 -> 16.29    17.09 -> 17.29
//   56   MiB [16384,7168]   88.0 -> 76.4                 29.5  -> 29.7     30.3  -> 30.9
// A program that only quantizes loses up to 3 % at 12 to 16 MiB, one that reads the matrix again gains three to eight
// times that and more.  Below 12 MiB the quantizer keeps its non-temporal stores: nothing is gained at 8 MiB and the gain
// of the chain between was not taken for the single kernel's sake.  Above 64 MiB the chain still gains but the single
// kernels lose: [32768,7168] 55.6 -> 57.9 and 57.1 -> 58.8.
constexpr int64_t KEEP_BYTES = (int64_t)64 << 20;
constexpr int64_t KEEP_FROM = (int64_t)12 << 20; // of the quantizer's output

// Write-through at device scope (sc1) without the non-temporal hint.
__device__ __forceinline__ void store_through(void *p, u32x2 v)
{
    asm volatile("global_store_dwordx2 %0, %1, off sc1" : : "v"(p), "v"(v) : "memory");
}

// The first n (1..15) bytes of v to dst, any alignment, in at most four pieces.
__device__ __forceinline__ void store_head_bytes(uint8_t *dst, const u32x4 v, uint32_t n)
{
    uint32_t pos = 0; // bytes done
    if (n & 8u) {
        *reinterpret_cast<u64_unaligned *>(dst) = ((uint64_t)v.y << 32) | v.x;
        pos = 8;
    }
    if (n & 4u) {
        *reinterpret_cast<u32_unaligned *>(dst + pos) = pos ? v.z : v.x;
        pos += 4;
    }
    const uint32_t d = pos == 0u ? v.x : pos == 4u ? v.y : pos == 8u ? v.z : v.w; // the dword still open
    if (n & 2u)
        *reinterpret_cast<u16_unaligned *>(dst + pos) = (uint16_t)d;
    if (n & 1u)
        dst[pos + (n & 2u)] = (uint8_t)(d >> (8u * (n & 2u)));
}

// Compile-time loop: f(std::integral_constant<int, 0>) ... f(std::integral_constant<int, N-1>).
// The conversion builtins take their byte selector as an immediate.
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(static_cast<F &&>(f), std::make_integer_sequence<int, N>{});
}

} // namespace mxfp4
