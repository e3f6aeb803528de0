// Pieces shared by the two matrix-core Hadamard kernels (the fused quantizer and the trust-masked
// inverse transform): a row is cut into tiles of 1024 elements seen as 32 x 32 matrices X[p][q]
// (element 32 p + q).  Index bits 0..4 (q) go through one exact +-1 MFMA product per tile, after
// which lane (m = l & 31, h = l >> 5) holds column q' = m and register r holds
// p = 8 (r >> 2) + 4 h + (r & 3); the other stages run on those registers.
#pragma once

#include "quest_device.h"

namespace quest {

typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// In-lane element index iota = b6 + 2 b7 + 4 b8 + 8 b9 + 16 tile (bN = index bit N of the
// element) -> accumulator register within its tile, after the half-wave swap:
// b7 = r & 1, b6 = (r >> 1) & 1, b8 = (r >> 2) & 1, b9 = r >> 3.
__host__ __device__ constexpr int reg_of_iota(int iota)
{
    return ((iota >> 1) & 1) | ((iota & 1) << 1) | (((iota >> 2) & 1) << 2) |
           (((iota >> 3) & 1) << 3);
}

__device__ __forceinline__ void bfly(float &a, float &b)
{
    const float t = a;
    a = t + b;
    b = t - b;
}

// B operand of the tile product D = X . (I (x) H_min(n,32)): rows q = 16 h + 8 s + e (s = which of
// the two 32 x 32 x 16 instructions, e = element) of that matrix, column q' = m, as bf16 +-1 / 0.
// FULL: the block is at least 32 wide, every entry is +-1: the signs of eight consecutive rows are
// parity(base & m) ^ parity(e & m), the second factor one of eight byte patterns.
template <bool FULL>
__device__ __forceinline__ void hadamard_operand(int log2n, int m, int h, v8bf (&bmat)[2])
{
    if constexpr (FULL) {
        const uint32_t pattern = ((m & 1) ? 0xAAu : 0u) ^ ((m & 2) ? 0xCCu : 0u) ^ ((m & 4) ? 0xF0u : 0u);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int base = 16 * h + 8 * s;
            const uint32_t minus = (__builtin_popcount(base & m) & 1) ? pattern ^ 0xFFu : pattern;   // bit e: entry is -1
            uint32_t w[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                w[k] = 0x3F803F80u | ((minus << (15 - 2 * k)) & 0x8000u) | ((minus << (30 - 2 * k)) & 0x80000000u);
            __builtin_memcpy(&bmat[s], w, 16);
        }
        return;
    }
    // column m has entries in the 2^nb rows of its block only: of the eight rows base .. base + 7 those whose bit is set in
    // `there` (all or none for blocks of eight or more), with the signs of the block's own pattern
    const int nb = log2n < 5 ? log2n : 5;
    const int low = (1 << nb) - 1, own = m & low, first = m & ~low;
    const uint32_t pattern = ((own & 1) ? 0xAAu : 0u) ^ ((own & 2) ? 0xCCu : 0u) ^ ((own & 4) ? 0xF0u : 0u);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int base = 16 * h + 8 * s;
        const uint32_t there = nb >= 3 ? ((base & ~low) == first ? 0xFFu : 0u)
                                       : (first >> 3 == base >> 3 ? ((1u << (1 << nb)) - 1u) << (first & 7) : 0u);
        const uint32_t minus = (__builtin_popcount(base & own) & 1) ? pattern ^ 0xFFu : pattern;   // bit e: entry is -1
        uint32_t w[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            w[k] = ((there >> (2 * k)) & 1u) * (0x3F80u | ((minus << (15 - 2 * k)) & 0x8000u)) |
                   ((there >> (2 * k + 1)) & 1u) * (0x3F800000u | ((minus << (30 - 2 * k)) & 0x80000000u));
        __builtin_memcpy(&bmat[s], w, 16);
    }
}

// The same for a block size known only at run time (wave-uniform); the general form is needed for blocks below 32 only.
__device__ __forceinline__ void hadamard_operand_any(int log2n, int m, int h, v8bf (&bmat)[2])
{
    if (log2n >= 5)
        hadamard_operand<true>(log2n, m, h, bmat);
    else
        hadamard_operand<false>(log2n, m, h, bmat);
}

// 1 / sqrt(n) and sqrt(n), correctly rounded: powers of two, times sqrt(2) for odd log2(n).
__device__ __forceinline__ float inv_sqrt_pow2(int log2n)
{
    return (log2n & 1) ? 0.70710678118654752440f / (float)(1 << (log2n >> 1)) : 1.0f / (float)(1 << (log2n >> 1));
}

__device__ __forceinline__ float sqrt_pow2(int log2n)
{
    return (log2n & 1) ? 1.41421356237309504880f * (float)(1 << (log2n >> 1)) : (float)(1 << (log2n >> 1));
}

// Per-row constants of the projection from the row's sum of squares, in the un-normalised domain
// (x_h = raw / sqrt(n)), every operation correctly rounded.
struct RowConstants {
    float scale;       // alpha rms / (L - 1); E2M1: alpha rms / 6
    float to_cell;     // raw -> position in grid cells; E2M1: raw -> units of the format
    float trust_raw;   // trusted iff |raw| <= trust_raw
    bool zero_row;     // scale 0, code k = 0 (E2M1: +0), all trusted, also where the entries are not zero but their squares are
};

template <int LEVELS, bool FP4>
__device__ __forceinline__ RowConstants row_constants(float total, int cols, float alpha, float trust_edge,
                                                      float inv_sqrt_n, float sqrt_n)
{
    RowConstants c;
    const float rms = sqrtf(__fdiv_rn(total, (float)cols));
    const float clip = __fmul_rn(alpha, rms);
    c.zero_row = !(rms > 0.0f);
    c.trust_raw = c.zero_row ? __builtin_inff() : __fmul_rn(__fmul_rn(trust_edge, rms), sqrt_n);
    const float inv_step = c.zero_row ? 0.0f : FP4 ? __fdiv_rn(6.0f, clip) : __fdiv_rn((float)(LEVELS - 1), __fmul_rn(2.0f, clip));
    c.to_cell = __fmul_rn(inv_step, inv_sqrt_n);
    c.scale = __fdiv_rn(clip, FP4 ? 6.0f : (float)(LEVELS - 1));
    return c;
}

// The code of one element in the top BITS bits of a byte (before its saturation to 0 .. 255): 2^(8-b) (cell + L/2), the cell
// being the floor of the product itself.  By the sum of product and 127.5, whose fp32 spacing is coarser than
// the product's near zero, more codes differ from a 64-bit evaluation (of 3.5e8 bf16 elements, 4 and 8
// bits: by the sum 116 and 1945, by the product 74 and 533; the general kernel 72 and 516).
template <int BITS>
__device__ __forceinline__ float cell_byte(float raw, float to_cell)
{
    return __fmaf_rn(floorf(__fmul_rn(raw, to_cell)), (float)(256 >> BITS), 128.0f);
}

// How a row's sum of squares is made up, the same in every kernel that may get a shape, so that a row's scale
// and codes do not depend on the number of rows: partial sum c is that of tiles c, c + n, .. (a fused multiply-add
// per element in order, then wave_sum_dpp), and the n partial sums are added in order.
__host__ __device__ constexpr int partial_sums_of_row(int tiles, int tiles_per_group)
{
    const int groups = (tiles + tiles_per_group - 1) / tiles_per_group;
    return groups < 4 ? groups : 4;
}

// The stages on index bits 5 .. LOG2N - 1 of G tiles held as MFMA accumulators: bits 5, 6, 8, 9 are
// register-to-register, bit 7 is the half-wave index and is swapped with register bit 0 first
// (after which h holds bit 5; the swap is made for every block size so that the element order of
// the registers does not depend on it), bits >= 10 pair whole tiles.  PAIRED: the stage on bit 10
// (tile 2 j with tile 2 j + 1) has already been applied by the caller.
template <int LOG2N, int G, bool PAIRED = false>
__device__ __forceinline__ void tile_stages(float (&acc)[G][16])
{
    if (LOG2N > 5) {  // bit 5 = register bit 0
#pragma unroll
        for (int u = 0; u < G; ++u)
#pragma unroll
            for (int r = 0; r < 16; r += 2)
                bfly(acc[u][r], acc[u][r + 1]);
    }
    if (LOG2N > 6) {  // bit 6 = register bit 1
#pragma unroll
        for (int u = 0; u < G; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (!(r & 2))
                    bfly(acc[u][r], acc[u][r + 2]);
    }
#pragma unroll
    for (int u = 0; u < G; ++u)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[u][r]),
                                                             __float_as_uint(acc[u][r + 1]), false, false);
            acc[u][r] = __uint_as_float(sw[0]);
            acc[u][r + 1] = __uint_as_float(sw[1]);
        }
    if (LOG2N > 7) {
#pragma unroll
        for (int u = 0; u < G; ++u)
#pragma unroll
            for (int r = 0; r < 16; r += 2)
                bfly(acc[u][r], acc[u][r + 1]);
    }
    if (LOG2N > 8) {  // bit 8 = register bit 2
#pragma unroll
        for (int u = 0; u < G; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (!(r & 4))
                    bfly(acc[u][r], acc[u][r + 4]);
    }
    if (LOG2N > 9) {  // bit 9 = register bit 3
#pragma unroll
        for (int u = 0; u < G; ++u)
#pragma unroll
            for (int r = 0; r < 8; ++r)
                bfly(acc[u][r], acc[u][r + 8]);
    }
#pragma unroll
    for (int k = PAIRED ? 1 : 0; (1 << k) < G; ++k) {  // bits >= 10 pair whole tiles
        if (LOG2N > 10 + k) {
#pragma unroll
            for (int u = 0; u < G; ++u)
                if (!(u & (1 << k)) && (u | (1 << k)) < G) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        bfly(acc[u][r], acc[u | (1 << k)][r]);
                }
        }
    }
}

// Sixteen floats as three packed bf16 pieces each, x = hi + mid + lo exactly: each piece is the top 16
// bits of what the pieces before it leave (the remainders have 16 and 8 significant bits).  Remainders
// come from the two-way bf16 dot product, packed piece times (1, 0) or (0, 1) minus the value:
// s1 = hi - x = -(mid + lo), s2 = top16(s1) - s1 = lo.  `mid` holds -mid.
__device__ __forceinline__ void split_bf16(const float (&f)[16], uint32_t (&hi)[8], uint32_t (&mid)[8], uint32_t (&lo)[8])
{
    // (1, 0) and (0, 1) as bf16 pairs, held in registers the compiler cannot see through: written
    // as literals the pair (1, 0) reaches the instruction as (0, 1)
    uint32_t first_bits = 0x00003F80u, second_bits = 0x3F800000u;
    asm volatile("" : "+v"(first_bits), "+v"(second_bits));
    v2bf first, second;
    __builtin_memcpy(&first, &first_bits, 4);
    __builtin_memcpy(&second, &second_bits, 4);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float a = f[2 * i], b = f[2 * i + 1];
        hi[i] = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
        v2bf hp;
        __builtin_memcpy(&hp, &hi[i], 4);
        const float s1a = __builtin_amdgcn_fdot2_f32_bf16(hp, first, -a, false);
        const float s1b = __builtin_amdgcn_fdot2_f32_bf16(hp, second, -b, false);
        mid[i] = __builtin_amdgcn_perm(__float_as_uint(s1b), __float_as_uint(s1a), 0x07060302u);
        v2bf mp;
        __builtin_memcpy(&mp, &mid[i], 4);
        const float s2a = __builtin_amdgcn_fdot2_f32_bf16(mp, first, -s1a, false);
        const float s2b = __builtin_amdgcn_fdot2_f32_bf16(mp, second, -s1b, false);
        lo[i] = __builtin_amdgcn_perm(__float_as_uint(s2b), __float_as_uint(s2a), 0x07060302u);
    }
}

template <int XOR>
__device__ __forceinline__ uint32_t swizzle_xor(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (XOR << 10) | 0x1f);
}

// Per-lane constants of the lane <-> field transposes.  In stage s a lane keeps the fields whose
// index bit s equals its own lane bit s and takes the others from lane ^ (1 << s), moved by
// FIELD << s bits.  Moves of 8 or 16 bits are one byte permute; smaller ones a rotate and a
// three-input select.
template <int STAGES, int FIELD>
struct TransposePlan {
    uint32_t keep[STAGES];   // bit mask of the fields kept            (sub-byte stages)
    uint32_t rot[STAGES];    // right-rotation applied to the partner  (sub-byte stages)
    uint32_t sel[STAGES];    // v_perm selector {own, partner}         (byte and halfword stages)

    __device__ __forceinline__ void init(int lane)
    {
#pragma unroll
        for (int s = 0; s < STAGES; ++s) {
            const int sh = FIELD << s;
            uint32_t lo = 0;  // field positions whose index has bit s clear
#pragma unroll
            for (int f = 0; f < (1 << STAGES); ++f)
                if (((f >> s) & 1) == 0)
                    lo |= ((1u << FIELD) - 1u) << (f * FIELD);
            const bool up = (lane >> s) & 1;
            keep[s] = up ? ~lo : lo;
            rot[s] = up ? (uint32_t)sh : (uint32_t)(32 - sh);
            // v_perm_b32(partner, own, sel): selector bytes 0..3 pick from own, 4..7 from partner
            if (sh == 8)
                sel[s] = up ? 0x03070105u : 0x06020400u;
            else if (sh == 16)
                sel[s] = up ? 0x03020706u : 0x05040100u;
            else
                sel[s] = 0;
        }
    }

    // After the call, field i of lane a holds what field a of lane i held (lanes modulo 2^STAGES).
    __device__ __forceinline__ uint32_t apply(uint32_t d) const
    {
#pragma unroll
        for (int s = 0; s < STAGES; ++s) {
            uint32_t partner;
            if (s == 0) partner = swizzle_xor<1>(d);
            else if (s == 1) partner = swizzle_xor<2>(d);
            else if (s == 2) partner = swizzle_xor<4>(d);
            else if (s == 3) partner = swizzle_xor<8>(d);
            else partner = swizzle_xor<16>(d);
            if ((FIELD << s) >= 8) {
                d = __builtin_amdgcn_perm(partner, d, sel[s]);
            } else {
                const uint32_t rotated = __builtin_amdgcn_alignbit(partner, partner, rot[s]);
                // (keep & d) | (~keep & rotated) as one three-input bit operation
                d = __builtin_amdgcn_bitop3_b32(keep[s], d, rotated, 0xCA);
            }
        }
        return d;
    }
};

// tile_stages for a block size known only at run time: the stages on index bits 5 .. 9 of one tile, and the
// stages that pair whole tiles, bits 10 and up, of G tiles (wave-uniform branches).  One tile's are straight code for
// each size: with a branch for each stage the values come together behind every one of them, a move per
// butterfly.  (Not more tiles than one: of 32 values from eight such pieces of code, nine to eighteen went to scratch.)
__device__ __forceinline__ void one_tile_stages(int log2n, float (&tile)[16])
{
    float (&acc)[1][16] = *reinterpret_cast<float (*)[1][16]>(&tile);
    if (log2n >= 10)
        tile_stages<10, 1>(acc);
    else if (log2n == 9)
        tile_stages<9, 1>(acc);
    else if (log2n == 8)
        tile_stages<8, 1>(acc);
    else if (log2n == 7)
        tile_stages<7, 1>(acc);
    else if (log2n == 6)
        tile_stages<6, 1>(acc);
    else
        tile_stages<5, 1>(acc);
}

template <int G>
__device__ __forceinline__ void tile_pair_stages(int log2n, float (&acc)[G][16])
{
#pragma unroll
    for (int k = 0; (1 << k) < G; ++k)
        if (log2n > 10 + k) {
#pragma unroll
            for (int u = 0; u < G; ++u)
                if (!(u & (1 << k))) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        bfly(acc[u][r], acc[u | (1 << k)][r]);
                }
        }
}

// ---- the inverse transform's inputs and outputs

__device__ __forceinline__ uint32_t pack_bf16_pair(float lo, float hi)
{
    v2bf p;
    p[0] = (__bf16)lo;
    p[1] = (__bf16)hi;
    uint32_t u;
    __builtin_memcpy(&u, &p, 4);
    return u;
}

// zero the halves of `pair` whose mask bits (bit 0: low half, bit 1: high half) are clear
__device__ __forceinline__ uint32_t keep_trusted(uint32_t pair, uint32_t mask_bits, int first_bit)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_sbfe((int)mask_bits, first_bit, 1);      // 0 or ~0
    const uint32_t hi = (uint32_t)__builtin_amdgcn_sbfe((int)mask_bits, first_bit + 1, 1);
    return pair & __builtin_amdgcn_perm(hi, lo, 0x07060100u);   // low half from lo, high half from hi
}

}  // namespace quest
