// The 16-bit products with a code-packed operand for outputs of few tiles (small layers, short
// batches): the gradient matmuls of Algorithm 2 and the weight-only forward product (Sec. 4.4).
//
// The 256 x 256 tiles of the main path leave most compute units without work there (2048 x 640: 24
// tiles for 256 units), and expanding the packed operand is a launch of its own.  Here a workgroup
// owns 64 or 128 rows by 64 or 128 columns, and expands its share of the codes to bf16(fp32(s u)) on the way
// into LDS: an operand element is expanded once per tile row or column that needs it, which is a few
// times at these sizes, and nothing but the codes is read.
//
// 64 contraction elements per step, two LDS stages, one barrier per step; global loads run PF steps
// ahead in registers (with one workgroup per compute unit nobody else covers their latency).
//
// LDS forms of an operand of one step (T rows or columns by 64 contraction elements):
//   row form     (contraction-contiguous in memory) [T rows][8 chunks of 8 contraction elements], chunk
//                c of row r in slot c ^ ((r >> 1) & 7); 128-bit fragment reads
//   column form  (rows of memory are contraction rows) [64 contraction rows][T / 8 chunks of 8 columns],
//                chunk c of contraction row q in slot c ^ swz(q); read with the transposing LDS load (16 lanes
//                point at a 4 x 16 block, lane i receives column i), two per fragment.  swz moves the four
//                contraction rows of a block to different quarters of the 64 banks (bits 2, 3 of the chunk;
//                rows of 128 bytes: bit 2) and the low bits with the block's number: sixteen lanes that write
//                one chunk each of four rows, four apart in their row, then meet sixteen different slots.
#include <utility>

#include "gemm_tile.h"
#include "quest_internal.h"

namespace quest {
namespace {

typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;   // of one group: four waves
constexpr int GC = 64;          // contraction elements per step
constexpr int PF = 2;           // register sets for a group's loads, one step each (4 measured the same)

template <int T>
__device__ __forceinline__ int column_swz(int crow)
{
    static_assert(T == 64 || T == 128, "tile edge");
    return T == 128 ? ((crow & 3) << 2) | ((crow >> 2) & 3) : (((crow >> 1) & 1) << 2) | ((crow >> 2) & 1);
}

// NE packed codes (NE = 16 or 32) of one scale, as they come from memory
template <int GRID, int NE>
struct PackedCodes {
    static constexpr int kContainer = GRID == 0 || GRID == 3 ? 4 : GRID;   // bits; GRID 0 = E2M1
    static constexpr int kBytes = NE * kContainer / 8;
    uint32_t w[(kBytes + 3) / 4];

    __device__ __forceinline__ void load(const uint8_t *p)
    {
        if constexpr (kBytes == 16) {
            const v4u v = *reinterpret_cast<const v4u *>(p);
            w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
        } else if constexpr (kBytes == 8) {
            const v2u v = *reinterpret_cast<const v2u *>(p);
            w[0] = v.x; w[1] = v.y;
        } else if constexpr (kBytes == 4) {
            w[0] = *reinterpret_cast<const uint32_t *>(p);
        } else {
            w[0] = *reinterpret_cast<const uint16_t *>(p);
        }
    }

    // elements 2 p, 2 p + 1 as bf16(fp32(s u)) (E2M1: s v); `scaled` is scale(s)
    static __device__ __forceinline__ float scale(float s)
    {
        return GRID == 0 ? s : s * (1.0f / (float)(1 << (GRID == 0 ? 0 : 7 - GRID)));
    }
    static constexpr int kPerByte = 8 / kContainer;
    // The eight codes of group g as signed bytes: bytes[d] holds, in byte i, element kPerByte i + d of the group as
    // 2^(7 - b) u: the code at the top of its byte, top bit inverted, the bit below the code set.  (The power of
    // two goes into the scale: s u exactly as by fp32(s u), for scales of 2^-120 or more.  Below, the scale is
    // subnormal and rounded by at most 2^-150, the product by 127 times that, 2^-10 of the spacing of bf16 there.)
    template <int g, bool WHOLE>
    __device__ __forceinline__ void to_bytes(uint32_t (&bytes)[8]) const
    {
        if constexpr (GRID != 0) {
            constexpr uint32_t field = ((0xffu << (8 - GRID)) & 0xffu) * 0x01010101u;
            constexpr uint32_t flip = (0x80u | (0x80u >> GRID)) * 0x01010101u;
            const uint32_t word = kContainer == 4 ? w[g] : w[g * kContainer / 4] >> (8 * ((g * kContainer) & 3));
            static_for<kPerByte>([&](auto d) {
                constexpr int up = 8 - GRID - decltype(d)::value * kContainer;
                bytes[decltype(d)::value] = ((up >= 0 ? word << (up & 31) : word >> (-up & 31)) & field) ^ flip;
                if constexpr (WHOLE)   // computed here as a word, not byte by byte at each use
                    asm("" : "+v"(bytes[decltype(d)::value]));
            });
        }
    }
    template <int P>
    __device__ __forceinline__ uint32_t expand_pair(const uint32_t (&bytes)[8], float scaled) const
    {
        if constexpr (GRID == 0) {
            const v2f v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w[P / 4], 1.0f, P % 4);
            return pack_bf16(__fmul_rn(scaled, v[0]), __fmul_rn(scaled, v[1]));
        } else {
            constexpr int e = 2 * P % 8;
            return pack_bf16(__fmul_rn((float)(int8_t)(bytes[e % kPerByte] >> (8 * (e / kPerByte))), scaled),
                             __fmul_rn((float)(int8_t)(bytes[(e + 1) % kPerByte] >> (8 * ((e + 1) / kPerByte))), scaled));
        }
    }
};

/*
 * MODE as in grad_gemm.hip: 0: out[M, K] = dy what (left row form, right column form), 1: out[N, K] =
 * dy^T xhat (both column form), 2: out[M, N] = x what^T (both row form).
 * `left` has row pitch ld_left elements, the packed operand row pitch q_row_bytes; out is [R, K].
 * Waves 2 x 2, each 32 WI x 32 WJ outputs.  R and K are multiples of 64 and may end inside a tile of
 * 128: the loads then take what exists in place of what does not, and the stores are predicated.
 */
template <int MODE, int GRID, int WI, int WJ, int GROUPS>
__global__ __launch_bounds__(kThreads * GROUPS, GROUPS == 1 ? 2 : 1) void grad_gemm_mid_kernel(
    const uint16_t *__restrict__ left, int64_t ld_left, const uint8_t *__restrict__ q_codes, int64_t q_row_bytes,
    const float *__restrict__ q_scales, int C, int R, int K, int tiles_r, int tiles_k, uint16_t *__restrict__ out)
{
    constexpr bool kLeftColumns = MODE == 1, kRightRows = MODE == 2;
    constexpr int TR = 64 * WI, TC = 64 * WJ;
    constexpr int kLeftBytes = TR * GC * 2, kRightBytes = TC * GC * 2, kStage = kLeftBytes + kRightBytes;
    constexpr int kLeftChunks = TR * 8 / kThreads;   // 16-byte chunks per thread and step
    constexpr int NE = TC * GC / kThreads;           // codes per thread and step
    typedef PackedCodes<GRID, NE> Packed;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    // one contiguous run of tiles per XCD, eight tile-rows deep
    const int total = tiles_r * tiles_k, per_xcd = (total + 7) / 8;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= total)
        return;
    const int band = logical / (8 * tiles_k), band_rows = min(8, tiles_r - band * 8);
    const int in_band = logical - band * 8 * tiles_k;
    const int r0 = (band * 8 + in_band % band_rows) * TR, k0 = (in_band / band_rows) * TC;

    // groups of four waves share the tile's steps in turn: group g takes steps g, g + GROUPS, ..
    const int group = GROUPS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads);
    uint8_t *const stages = smem + group * (2 * kStage);
    const int tid = threadIdx.x % kThreads, lane = tid & 63, wave = tid >> 6;
    const int wr = wave >> 1, wc = wave & 1;
    const int lm = lane & 31, lh = lane >> 5, l16 = lane & 15, lg = lane >> 4;
    const int steps = C / GC, rounds = (steps + GROUPS - 1) / GROUPS;

    // ---- this thread's share of a step: byte offsets from the operands' positions of the step
    // (wave-uniform), and where it goes in a stage
    uint32_t left_src[kLeftChunks];
    int left_dst[kLeftChunks];
#pragma unroll
    for (int i = 0; i < kLeftChunks; ++i) {
        const int chunk = i * kThreads + tid;
        if constexpr (kLeftColumns) {
            const int crow = chunk / (TR / 8), c = chunk % (TR / 8);
            left_src[i] = ((uint32_t)crow * (uint32_t)ld_left + (uint32_t)min(8 * c, R - 8 - r0)) * 2u;
            left_dst[i] = crow * (TR * 2) + ((c ^ column_swz<TR>(crow)) << 4);
        } else {
            const int row = chunk >> 3, c = chunk & 7;
            left_src[i] = ((uint32_t)min(row, R - 1 - r0) * (uint32_t)ld_left + 8u * c) * 2u;
            left_dst[i] = row * 128 + ((c ^ ((row >> 1) & 7)) << 4);
        }
    }
    const char *const left_base = reinterpret_cast<const char *>(left + (kLeftColumns ? (int64_t)r0 : r0 * ld_left));
    const int64_t left_step = (kLeftColumns ? GC * ld_left : GC) * 2;
    uint32_t code_src, scale_src;
    int right_dst[NE / 8];
    if constexpr (kRightRows) {
        constexpr int kPerRow = GC / NE;   // threads per output column
        const int row = tid / kPerRow, part = tid % kPerRow;
        scale_src = (uint32_t)min(row, K - 1 - k0) * 4u;
        code_src = (uint32_t)min(row, K - 1 - k0) * (uint32_t)q_row_bytes + (uint32_t)(part * Packed::kBytes);
#pragma unroll
        for (int g = 0; g < NE / 8; ++g)
            right_dst[g] = kLeftBytes + row * 128 + (((part * (NE / 8) + g) ^ ((row >> 1) & 7)) << 4);
    } else {
        // (the four contraction rows of sixteen lanes are four apart, T = 64: 0, 1, 4, 5 of eight; see column_swz)
        const int part = tid & 3, four = (tid >> 2) & 3, rest = tid >> 4;
        const int crow = TC == 128 ? 16 * (rest >> 2) + 4 * four + (rest & 3)
                                   : 8 * (rest >> 1) + 4 * (four >> 1) + 2 * (rest & 1) + (four & 1);
        scale_src = (uint32_t)crow * 4u;
        code_src = (uint32_t)crow * (uint32_t)q_row_bytes + (uint32_t)min(part * NE, K - NE - k0) * Packed::kContainer / 8u;
#pragma unroll
        for (int g = 0; g < NE / 8; ++g)
            right_dst[g] = kLeftBytes + crow * (TC * 2) + (((part * (NE / 8) + g) ^ column_swz<TC>(crow)) << 4);
    }
    const uint8_t *const code_base = q_codes + (kRightRows ? k0 * q_row_bytes : (int64_t)k0 * Packed::kContainer / 8);
    const char *const scale_base = reinterpret_cast<const char *>(q_scales + (kRightRows ? k0 : 0));
    const int64_t code_step = kRightRows ? GC * Packed::kContainer / 8 : GC * q_row_bytes;
    const int64_t scale_step = kRightRows ? 0 : GC * 4;

    v4u left_reg[PF][kLeftChunks];
    Packed code_reg[PF];
    float scale_reg[PF];
    // operand positions of the round being fetched (past the end: the last step again, not used)
    const char *left_at = left_base, *scale_at = scale_base;
    const uint8_t *code_at = code_base;
    auto position = [&](int round) {
        const int at = min(round * GROUPS + group, steps - 1);
        left_at = left_base + at * left_step;
        code_at = code_base + at * code_step;
        scale_at = scale_base + at * scale_step;
    };
    auto fetch_left = [&](auto set, auto i) {
        left_reg[decltype(set)::value][decltype(i)::value] =
            *reinterpret_cast<const v4u *>(left_at + left_src[decltype(i)::value]);
    };
    auto fetch_codes = [&](auto set) {
        code_reg[decltype(set)::value].load(code_at + code_src);
        scale_reg[decltype(set)::value] = *reinterpret_cast<const float *>(scale_at + scale_src);
    };
    auto fetch = [&](auto set, int round) {
        position(round);
        static_for<kLeftChunks>([&](auto i) { fetch_left(set, i); });
        fetch_codes(set);
    };
    // Blocks of 128 x 128 pin the staging of the next round between a round's matrix instructions: a wave
    // that multiplies first and expands afterwards leaves the matrix unit and the vector unit idle in turn,
    // and two waves on a SIMD, in step by the barriers, do little about it (weight-only 512 x 5632 x 2048
    // 23.1 -> 20.7 us, 2560 x 1024 x 2816 28.2 -> 24.5; G_w 2688 x 384 x 5632 28.5 -> 24.7).  Smaller blocks have
    // half or a quarter of the matrix instructions per expanded code; there the order is left to the
    // compiler, with all loads issued ahead of the multiplication (G_w 2048 x 1792 x 640 16.6 us, pinned 17.9).
    constexpr bool kPinned = WI * WJ == 4;
    // The staging of a round in kSlices slices: slice e expands pair e of the codes and, with a chunk's last
    // pair, writes the chunk; the left operand's chunks go in between, each replaced at once by the load of
    // the same chunk for two rounds later, if REFILL (`position` says which).
    constexpr int kSlices = NE / 2;
    v4u chunk;
    uint32_t bytes[8];
    auto stage_slice = [&](auto set, uint8_t *stage, auto slice, auto refill) __attribute__((always_inline)) {
        constexpr int p = decltype(set)::value, e = decltype(slice)::value;
        if constexpr (e % 4 == 0)
            code_reg[p].template to_bytes<e / 4, kPinned>(bytes);
        chunk[e % 4] = code_reg[p].template expand_pair<e>(bytes, Packed::scale(scale_reg[p]));
        if constexpr (e % 4 == 3)
            *reinterpret_cast<v4u *>(stage + right_dst[e / 4]) = chunk;
        if constexpr (kPinned && e % 4 == 1)
            static_for<kLeftChunks>([&](auto i) {
                if constexpr (decltype(i)::value * (kSlices / 4) / kLeftChunks == e / 4) {
                    *reinterpret_cast<v4u *>(stage + left_dst[decltype(i)::value]) = left_reg[p][decltype(i)::value];
                    if constexpr (decltype(refill)::value)
                        fetch_left(set, i);
                }
            });
        if constexpr (e == kSlices - 1 && decltype(refill)::value)
            fetch_codes(set);
    };
    auto stage_in = [&](auto set, uint8_t *stage, auto refill) {
        if constexpr (!kPinned)
            static_for<kLeftChunks>([&](auto i) {
                *reinterpret_cast<v4u *>(stage + left_dst[decltype(i)::value]) =
                    left_reg[decltype(set)::value][decltype(i)::value];
            });
        static_for<kSlices>([&](auto e) { stage_slice(set, stage, e, refill); });
    };

    // ---- fragment reads
    auto row_fragment = [&](const uint8_t *operand, int row0, int ks) {
        const int row = row0 + lm;
        return *reinterpret_cast<const v8bf *>(operand + row * 128 + (((2 * ks + lh) ^ ((row >> 1) & 7)) << 4));
    };
    auto column_fragment = [&](auto edge, const uint8_t *operand, int col0, int ks) __attribute__((always_inline)) {
        constexpr int T = decltype(edge)::value;
        const int col = col0 + 16 * (lg & 1) + 4 * (l16 & 3), row = 8 * (lg >> 1) + (l16 >> 2);
        auto at = [&](int more) {   // contraction row of the k-step: row + more (swz has period 16)
            return operand + (16 * ks + row + more) * (T * 2) + (((col >> 3) ^ column_swz<T>(row + more)) << 4) +
                   (col & 7) * 2;
        };
        typedef __attribute__((address_space(3))) v4bf LdsV4;
        const v4bf lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LdsV4 *)at(0));
        const v4bf hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LdsV4 *)at(4));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };

    v16f acc[WI][WJ];
#pragma unroll
    for (int i = 0; i < WI; ++i)
#pragma unroll
        for (int j = 0; j < WJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][j][r] = 0.0f;
    // Fragments of k-step ks in set ks % 2; read number n of a k-step (transposing reads come in pairs).
    v8bf lf[2][WI], rf[2][WJ];
    constexpr int kFragments = WI + WJ, kBlocks = WI * WJ, kMatrix = (GC / 16) * kBlocks;
    auto read_fragment = [&](const uint8_t *stage, auto ksc, auto fc) __attribute__((always_inline)) {
        constexpr int ks = decltype(ksc)::value, f = decltype(fc)::value;   // R0 L0 then the others
        constexpr bool is_left = f == 1 || f > WJ;
        constexpr int i = is_left ? (f == 1 ? 0 : f - WJ) : (f == 0 ? 0 : f - 1);
        if constexpr (is_left) {
            if constexpr (kLeftColumns)
                lf[ks & 1][i] = column_fragment(std::integral_constant<int, TR>{}, stage, wr * 32 * WI + 32 * i, ks);
            else
                lf[ks & 1][i] = row_fragment(stage, wr * 32 * WI + 32 * i, ks);
        } else {
            if constexpr (kRightRows)
                rf[ks & 1][i] = row_fragment(stage + kLeftBytes, wc * 32 * WJ + 32 * i, ks);
            else
                rf[ks & 1][i] = column_fragment(std::integral_constant<int, TC>{}, stage + kLeftBytes,
                                                wc * 32 * WJ + 32 * i, ks);
        }
    };
    // The matrix instructions of a round out of `stage`.  Pinned: each is followed by its share of the next
    // k-step's fragment reads and, if STAGING, of the next round's staging.  (Right fragment as the row
    // operand: transposed accumulator tiles.)
    auto multiply = [&](auto staging, auto refill, const uint8_t *stage, auto next_set, uint8_t *next_stage)
                        __attribute__((always_inline)) {
        static_for<GC / 16>([&](auto ksc) {
            constexpr int ks = decltype(ksc)::value;
            typedef std::integral_constant<int, ks + 1> NextStep;
            if constexpr (ks == 0 || !kPinned)
                static_for<kFragments>([&](auto f) { read_fragment(stage, ksc, f); });
            static_for<kBlocks>([&](auto bc) {
                constexpr int b = decltype(bc)::value, i = b / WJ, j = b % WJ;
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rf[ks & 1][j], lf[ks & 1][i], acc[i][j], 0, 0, 0);
                if constexpr (kPinned) {
                    if constexpr (ks + 1 < GC / 16)
                        static_for<kFragments>([&](auto f) {
                            if constexpr (decltype(f)::value * kBlocks / kFragments == b)
                                read_fragment(stage, NextStep{}, f);
                        });
                    if constexpr (decltype(staging)::value)
                        static_for<kSlices>([&](auto e) {
                            if constexpr (decltype(e)::value * kMatrix / kSlices == ks * kBlocks + b)
                                stage_slice(next_set, next_stage, e, refill);
                        });
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
        });
    };

    typedef std::integral_constant<int, 0> Set0;
    typedef std::integral_constant<int, 1> Set1;
    static_for<PF>([&](auto p) { fetch(p, decltype(p)::value); });
    int s = 0;
    if constexpr (kPinned) {
        // Round s reads stage s % 2 and stages round s + 1 in the other one (last read in round s - 1, which
        // every wave had left when it passed the barrier of round s).
        position(PF);
        stage_in(Set0{}, stages, std::true_type{});
        for (; s + PF < rounds; s += PF) {
            static_for<PF>([&](auto p) {
                constexpr int now = decltype(p)::value;
                typedef std::integral_constant<int, 1 - now> Next;
                __syncthreads();
                position(s + now + 1 + PF);
                multiply(std::true_type{}, std::true_type{}, stages + now * kStage, Next{}, stages + (1 - now) * kStage);
            });
        }
        // the last one or two rounds
        __syncthreads();
        const bool second = s + 1 < rounds;
        if (second)   // (then every group has this round)
            multiply(std::true_type{}, std::false_type{}, stages, Set1{}, stages + kStage);
        else if (GROUPS == 1 || s * GROUPS + group < steps)
            multiply(std::false_type{}, std::false_type{}, stages, Set1{}, stages + kStage);
        if (second) {
            __syncthreads();
            if (GROUPS == 1 || (s + 1) * GROUPS + group < steps)
                multiply(std::false_type{}, std::false_type{}, stages + kStage, Set0{}, stages);
        }
    } else {
        // Round s: into stage s % 2 (last read in round s - 2, which every wave had left when it passed the
        // barrier of round s - 1), loads of round s + PF, barrier, multiply.
        for (; s + PF < rounds; s += PF) {
            static_for<PF>([&](auto p) {
                uint8_t *const stage = stages + decltype(p)::value * kStage;
                stage_in(p, stage, std::false_type{});
                fetch(p, s + decltype(p)::value + PF);
                // the next round's expansion may move up to here, not above the loads: its wait would cover them
                __builtin_amdgcn_sched_barrier(0);
                __syncthreads();
                multiply(std::false_type{}, std::false_type{}, stage, p, stage);
            });
        }
        static_for<PF>([&](auto p) {
            if (s + decltype(p)::value < rounds) {
                uint8_t *const stage = stages + decltype(p)::value * kStage;
                stage_in(p, stage, std::false_type{});
                __syncthreads();
                if (GROUPS == 1 || (s + decltype(p)::value) * GROUPS + group < steps)
                    multiply(std::false_type{}, std::false_type{}, stage, p, stage);
            }
        });
    }

    // the groups' sums meet in the first group, in order
    if constexpr (GROUPS > 1) {
        constexpr int kPerGroup = WI * WJ * 4 * kThreads;   // float4
        v4f *sums = reinterpret_cast<v4f *>(smem);
        __syncthreads();
        if (group != 0) {
            static_for<WI * WJ * 4>([&](auto n) {
                constexpr int i = decltype(n)::value / (4 * WJ), j = decltype(n)::value / 4 % WJ, r = decltype(n)::value % 4 * 4;
                sums[(group - 1) * kPerGroup + decltype(n)::value * kThreads + tid] =
                    v4f{acc[i][j][r], acc[i][j][r + 1], acc[i][j][r + 2], acc[i][j][r + 3]};
            });
        }
        __syncthreads();
        if (group != 0)
            return;
#pragma unroll
        for (int g = 0; g < GROUPS - 1; ++g)
            static_for<WI * WJ * 4>([&](auto n) {
                constexpr int i = decltype(n)::value / (4 * WJ), j = decltype(n)::value / 4 % WJ, r = decltype(n)::value % 4 * 4;
                const v4f v = sums[g * kPerGroup + decltype(n)::value * kThreads + tid];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[i][j][r + e] += v[e];
            });
    }

    // Epilogue: lane l of an accumulator tile holds output row l % 32 and, in register r, column
    // 8 (r / 4) + 4 (l / 32) + r % 4.  Each wave parks its block as bf16 and writes 16-byte chunks.
    if constexpr (GROUPS == 1)
        __syncthreads();   // every wave is done with the stages
    constexpr int kRowBytes = 64 * WJ, kRowChunks = 4 * WJ;
    // (several groups: behind the sums, which other waves may still be reading)
    constexpr int kParkAt = GROUPS == 1 ? 0 : (GROUPS - 1) * WI * WJ * 4 * kThreads * 16;
    static_assert(kParkAt + 4 * 32 * WI * kRowBytes <= GROUPS * 2 * kStage, "sums and parked blocks fit the stages");
    uint8_t *park = smem + kParkAt + wave * (32 * WI * kRowBytes);
#pragma unroll
    for (int i = 0; i < WI; ++i)
#pragma unroll
        for (int j = 0; j < WJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = 32 * i + lm, chunk = (4 * j + q) ^ (row & (kRowChunks - 1));
                *reinterpret_cast<uint2 *>(park + row * kRowBytes + chunk * 16 + 8 * lh) =
                    make_uint2(pack_bf16(acc[i][j][4 * q + 0], acc[i][j][4 * q + 1]),
                               pack_bf16(acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]));
            }
    // (a wave reads back only what it parked itself)
    const int row_base = r0 + wr * 32 * WI, col_base = k0 + wc * 32 * WJ;
#pragma unroll
    for (int pass = 0; pass < 32 * WI * kRowChunks / 64; ++pass) {
        const int at = pass * 64 + lane, row = at / kRowChunks, c = at % kRowChunks;
        const uint4 v = *reinterpret_cast<const uint4 *>(park + row * kRowBytes + ((c ^ (row & (kRowChunks - 1))) << 4));
        if (row_base + row < R && col_base + 8 * c < K)
            *reinterpret_cast<uint4 *>(out + (int64_t)(row_base + row) * K + col_base + 8 * c) = v;
    }
}

template <int MODE, int GRID, int WI, int WJ, int GROUPS>
hipError_t launch(const GradMidArgs &a, hipStream_t stream)
{
    auto kernel = grad_gemm_mid_kernel<MODE, GRID, WI, WJ, GROUPS>;
    const int tiles_r = (int)((a.R + 64 * WI - 1) / (64 * WI)), tiles_k = (int)((a.K + 64 * WJ - 1) / (64 * WJ));
    constexpr int kLds = GROUPS * 2 * (64 * WI + 64 * WJ) * GC * 2;
    if (kLds > 64 * 1024) {
        static OncePerDevice once;
        const hipError_t err = once([&] { return allow_dynamic_lds(reinterpret_cast<const void *>(kernel), kLds); });
        if (err != hipSuccess)
            return err;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)((tiles_r * tiles_k + 7) / 8 * 8)), dim3(kThreads * GROUPS), kLds, stream,
                       static_cast<const uint16_t *>(a.left), a.ld_left, a.q_codes, a.q_row_bytes, a.q_scales,
                       (int)a.C, (int)a.R, (int)a.K, tiles_r, tiles_k, static_cast<uint16_t *>(a.out));
    return hipGetLastError();
}

// The block shapes there are, with what one costs (us, measured on G_x, G_w and weight-only products of
// 128 .. 16384 tokens): `alone` per round of GROUPS steps with one workgroup on a compute unit, `shared` per
// workgroup and round when several take turns.  What bounds a round is a wave's issue rate (expansion:
// three vector instructions per code) and the LDS traffic, so small blocks are cheap per round and dear
// per operation; several groups halve or quarter the number of rounds where a unit has one workgroup.
// One-bit codes (eight to a byte, each expanded by itself in blocks whose order is the compiler's) make a round of
// the smaller blocks dearer, by `one_bit`: measured / estimated without it 1.2 to 1.45 (G_x 384 x 9792 x 3136 with
// 64 x 128 blocks of two groups: 63.8 us at 4 bits, 92.5 at one).  Those, at 1.45, would never be the
// cheapest and are not built for one bit (0).
struct Shape {
    int wi, wj, groups;
    double alone, shared, one_bit;
};
constexpr Shape kShapes[] = {{1, 1, 2, 0.56, 0.44, 1.20}, {1, 1, 4, 1.00, 1.00, 1.25}, {1, 2, 1, 0.53, 0.39, 1.30},
                             {1, 2, 2, 0.79, 0.79, 0.00}, {2, 2, 1, 0.70, 0.61, 1.00}, {2, 2, 2, 1.08, 1.30, 1.05}};

double shape_cost(const Shape &s, int grid, int64_t C, int64_t R, int64_t K, int cus)
{
    if (grid == 1 && s.one_bit == 0.0)
        return 1e30;
    const int64_t blocks = ((R + 64 * s.wi - 1) / (64 * s.wi)) * ((K + 64 * s.wj - 1) / (64 * s.wj));
    const int64_t per_cu = (blocks + cus - 1) / cus, rounds = (C / GC + s.groups - 1) / s.groups;
    const double round = (per_cu == 1 ? s.alone : (double)per_cu * s.shared) * (grid == 1 ? s.one_bit : 1.0);
    return 3.0 + (double)per_cu * 1.0 + (double)rounds * round;
}

int cheapest_shape(int grid, int64_t C, int64_t R, int64_t K, int cus)
{
    int best = 0;
    for (int i = 1; i < (int)(sizeof(kShapes) / sizeof(kShapes[0])); ++i)
        if (shape_cost(kShapes[i], grid, C, R, K, cus) < shape_cost(kShapes[best], grid, C, R, K, cus))
            best = i;
    return best;
}

template <int MODE, int GRID>
hipError_t launch_shape(const GradMidArgs &a, int shape, hipStream_t stream)
{
    switch (shape) {
    case 0: return launch<MODE, GRID, 1, 1, 2>(a, stream);
    case 1: return launch<MODE, GRID, 1, 1, 4>(a, stream);
    case 2: return launch<MODE, GRID, 1, 2, 1>(a, stream);
    case 3:
        if constexpr (GRID != 1)
            return launch<MODE, GRID, 1, 2, 2>(a, stream);
        return hipErrorInvalidValue;
    case 4: return launch<MODE, GRID, 2, 2, 1>(a, stream);
    default: return launch<MODE, GRID, 2, 2, 2>(a, stream);
    }
}

template <int MODE>
hipError_t launch_mode(const GradMidArgs &a, int shape, hipStream_t stream)
{
    switch (a.grid) {
    case 0:
        if constexpr (MODE != 2)
            return launch_shape<MODE, 0>(a, shape, stream);
        return hipErrorInvalidValue;   // no weight-only product on E2M1 codes
    case 1: return launch_shape<MODE, 1>(a, shape, stream);
    case 2: return launch_shape<MODE, 2>(a, shape, stream);
    case 3: return launch_shape<MODE, 3>(a, shape, stream);
    default: return launch_shape<MODE, 4>(a, shape, stream);
    }
}

template <int MODE, int GRID>
hipError_t prepare_grid()
{
    // the shapes with more than 64 KiB of LDS
    const auto limit = [](auto kernel, int wi, int wj, int groups) {
        return allow_dynamic_lds(reinterpret_cast<const void *>(kernel), groups * 2 * (64 * wi + 64 * wj) * GC * 2);
    };
    hipError_t err = limit(grad_gemm_mid_kernel<MODE, GRID, 1, 1, 4>, 1, 1, 4);
    if constexpr (GRID != 1) {
        if (err == hipSuccess)
            err = limit(grad_gemm_mid_kernel<MODE, GRID, 1, 2, 2>, 1, 2, 2);
    }
    if (err == hipSuccess)
        err = limit(grad_gemm_mid_kernel<MODE, GRID, 2, 2, 2>, 2, 2, 2);
    return err;
}

template <int MODE>
hipError_t prepare_mode()
{
    hipError_t err = prepare_grid<MODE, 1>();
    if (err == hipSuccess)
        err = prepare_grid<MODE, 2>();
    if (err == hipSuccess)
        err = prepare_grid<MODE, 3>();
    if (err == hipSuccess)
        err = prepare_grid<MODE, 4>();
    if constexpr (MODE != 2) {
        if (err == hipSuccess)
            err = prepare_grid<MODE, 0>();
    }
    return err;
}

}  // namespace

quest_plan grad_gemm_mid_plan(int grid, int64_t C, int64_t R, int64_t K, int cus)
{
    const Shape &s = kShapes[cheapest_shape(grid, C, R, K, cus)];
    return {QUEST_PLAN_MID, 64 * s.wi, 64 * s.wj, s.groups};
}

double grad_gemm_mid_cost(int grid, int64_t C, int64_t R, int64_t K, int cus)
{
    return shape_cost(kShapes[cheapest_shape(grid, C, R, K, cus)], grid, C, R, K, cus);
}

hipError_t prepare_grad_gemm_mid_kernels()
{
    hipError_t err = prepare_mode<0>();
    if (err == hipSuccess)
        err = prepare_mode<1>();
    if (err == hipSuccess)
        err = prepare_mode<2>();
    return err;
}

hipError_t launch_grad_gemm_mid(const GradMidArgs &a, hipStream_t stream)
{
    const int shape = cheapest_shape(a.grid, a.C, a.R, a.K, device_compute_units());
    return a.mode == 0   ? launch_mode<0>(a, shape, stream)
           : a.mode == 1 ? launch_mode<1>(a, shape, stream)
                         : launch_mode<2>(a, shape, stream);
}

}  // namespace quest
