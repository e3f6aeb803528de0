// The forward product for few activation rows (decoding, short prompts): y = xhat_h what_h^T on packed
// codes (Algorithm 1, last step), integer grid and E2M1 grid.
//
// With a few dozen rows the product is a pass over the packed weights (5.8 MB for 5632 x 2048, 1 us
// at the memory's rate) and everything else is latency, so the work is cut for as many loads in
// flight as possible and no staging: a workgroup owns 16 NT weight rows and all of its waves split the
// contraction between them in units of 128 elements, wave w taking units w, w + W, ..; a lane loads
// its share of a unit (32 codes of one row, 16 bytes at 4 bits) straight into registers, where it is
// the matrix instruction's operand after widening, and the waves' partial sums meet once in LDS.
// The sums are exact (int32, or fp32 multiples of 1/4 below 2^24), so their order does not matter.
//
// Every container width is read as it is (no re-coding pass for 1 and 2 bits), and any K that is a
// multiple of 64 is taken: the last half unit is one matrix instruction on half as many codes.
#include "gemm_tile.h"
#include "quest_internal.h"

namespace quest {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kUnit = 128;   // contraction elements per unit: 32 codes per lane, lanes l, l + 16, l + 32, l + 48 share a row

// GRID: 1, 2, 3, 4 = bits of the Eq. 1 grid, 0 = E2M1.
template <int GRID>
struct Codes {
    static constexpr int kContainer = GRID == 0 || GRID == 3 ? 4 : GRID;   // bits
    static constexpr int kWords = kContainer;                              // dwords of 32 codes
    // The integer codes become signed bytes 2^shift u: the code at the top of its byte, the top bit
    // inverted (offset binary to two's complement), the bit below the code set.  Products carry
    // 2^(2 shift); 2^(2 shift) (L - 1)^2 K stays below 2^31 for K <= 65536.
    static constexpr int kCarry = GRID == 0 ? 0 : 2 * (7 - GRID);
    uint32_t w[kWords];

    __device__ __forceinline__ void load(const uint8_t *p)
    {
        if constexpr (kWords == 4) {
            const uint4 v = *reinterpret_cast<const uint4 *>(p);
            w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
        } else if constexpr (kWords == 2) {
            const uint2 v = *reinterpret_cast<const uint2 *>(p);
            w[0] = v.x; w[1] = v.y;
        } else {
            w[0] = *reinterpret_cast<const uint32_t *>(p);
        }
    }
    // sixteen codes; what is above them in the registers is zero
    __device__ __forceinline__ void load_half(const uint8_t *p)
    {
        if constexpr (kWords == 4) {
            const uint2 v = *reinterpret_cast<const uint2 *>(p);
            w[0] = v.x; w[1] = v.y; w[2] = 0; w[3] = 0;
        } else if constexpr (kWords == 2) {
            w[0] = *reinterpret_cast<const uint32_t *>(p);
            w[1] = 0;
        } else {
            w[0] = *reinterpret_cast<const uint16_t *>(p);
        }
    }
    // The 32 codes as two operands of sixteen signed bytes.  The order of the elements is permuted
    // the same way in both factors of the product.
    __device__ __forceinline__ void widen(v4i (&op)[2]) const
    {
        static_assert(GRID != 0, "E2M1 codes are an operand as they are");
        constexpr uint32_t top = (0xffu << (8 - GRID)) & 0xffu;
        constexpr uint32_t field = top * 0x01010101u;
        constexpr uint32_t flip = (0x80u | (0x80u >> GRID)) * 0x01010101u;
        constexpr int kPerWord = 8 / kContainer;   // dwords of bytes per dword of codes
        int d[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int position = (i % kPerWord) * kContainer;       // the code's lowest bit in its byte
            const int up = 8 - GRID - position;
            const uint32_t v = w[i / kPerWord];
            d[i] = (int)(((up >= 0 ? v << up : v >> -up) & field) ^ flip);
        }
        op[0] = v4i{d[0], d[1], d[2], d[3]};
        op[1] = v4i{d[4], d[5], d[6], d[7]};
    }
};

template <bool FLOAT>
struct Sum {
    typedef v4i type;
};
template <>
struct Sum<true> {
    typedef v4f type;
};

/*
 * blockIdx.x: weight rows 16 NT blockIdx.x .., blockIdx.y: activation rows 16 MT blockIdx.y ..
 * Dynamic LDS: WAVES * MT * NT * 1 KiB.
 * The weights are the row operand, so a lane's four sums are four consecutive outputs of one row.
 */
template <int GRID, int MT, int NT, int BATCH, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 2) void skinny_gemm_kernel(
    const uint8_t *__restrict__ a_codes, const float *__restrict__ a_scales, const uint8_t *__restrict__ b_codes,
    const float *__restrict__ b_scales, int M, int N, int K, uint16_t *__restrict__ y, int64_t ld_y,
    void *__restrict__ acc_out)
{
    constexpr bool kFloat = GRID == 0;
    typedef typename Sum<kFloat>::type Acc;
    typedef Codes<GRID> C;
    constexpr int kContainer = C::kContainer;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    // The largest block's loop over one-bit codes wants its step unknown: as a constant the compiler carries the codes that are
    // fetched ahead through seven moves per 32 matrix instructions (us: 988 x 2816 x 10816 57.4, so 47.4; 3637 x 768 x 5568 32.1, 27.4).
    // With two bits it is better either way, by up to 5 % unknown where a compute unit has two of the blocks at most, by up to
    // 14 % known where it has more; with the others it makes no difference.
    int waves = WAVES;
    if constexpr (MT * NT == 16 && GRID == 1)
        asm("" : "+s"(waves));
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row16 = lane & 15, quarter = lane >> 4;
    const int n0 = blockIdx.x * 16 * NT, m0 = blockIdx.y * 16 * MT;
    const int64_t row_bytes = (int64_t)K * kContainer / 8;

    const uint8_t *a_row[MT], *b_row[NT];   // rows beyond the edge read the last row; their sums are not stored
#pragma unroll
    for (int i = 0; i < MT; ++i)
        a_row[i] = a_codes + min(m0 + 16 * i + row16, M - 1) * row_bytes;
#pragma unroll
    for (int j = 0; j < NT; ++j)
        b_row[j] = b_codes + min(n0 + 16 * j + row16, N - 1) * row_bytes;

    Acc acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
            acc[i][j] = Acc{0, 0, 0, 0};

    auto multiply = [&](const C (&a)[MT], const C (&b)[NT], int operands, bool half) {
        if constexpr (kFloat) {
            constexpr int one = 0x7f7f7f7f;   // block scales 2^0
            auto op = [](const C &c) { return v8i{(int)c.w[0], (int)c.w[1], (int)c.w[2], (int)c.w[3], 0, 0, 0, 0}; };
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(op(b[j]), op(a[i]), acc[i][j], 4, 4, 0,
                                                                                 one, 0, one);
        } else {
            v4i bw[NT][2];
#pragma unroll
            for (int j = 0; j < NT; ++j)
                b[j].widen(bw[j]);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                v4i aw[2];
                a[i].widen(aw);
                if (half && GRID == 1) {   // 16 one-bit codes sit in the low halves of all eight dwords
#pragma unroll
                    for (int o = 0; o < 2; ++o)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            aw[o][e] &= 0xffff;
                }
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int o = 0; o < 2; ++o)
                        if (o < operands)
                            acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bw[j][o], aw[o], acc[i][j], 0, 0, 0);
            }
        }
    };

    const int units = K / kUnit;
    if (wave < units) {
        C a[BATCH][MT], b[BATCH][NT];
        auto fetch = [&](int s, int unit) {   // past the end: the last unit again, not used
            const int off = min(unit, units - 1) * (16 * kContainer) + quarter * 4 * kContainer;
#pragma unroll
            for (int j = 0; j < NT; ++j)
                b[s][j].load(b_row[j] + off);
#pragma unroll
            for (int i = 0; i < MT; ++i)
                a[s][i].load(a_row[i] + off);
        };
#pragma unroll
        for (int s = 0; s < BATCH; ++s)
            fetch(s, wave + s * waves);
        int u = wave;
        for (; u + BATCH * waves < units; u += BATCH * waves) {
#pragma unroll
            for (int s = 0; s < BATCH; ++s) {
                multiply(a[s], b[s], 2, false);
                fetch(s, u + (s + BATCH) * waves);
            }
        }
#pragma unroll
        for (int s = 0; s < BATCH; ++s)
            if (u + s * waves < units)
                multiply(a[s], b[s], 2, false);
    }
    if constexpr (!kFloat) {
        if ((K & 64) && wave == units % waves) {   // the half unit at the end
            C a[MT], b[NT];
            const int off = units * (16 * kContainer) + quarter * 2 * kContainer;
#pragma unroll
            for (int j = 0; j < NT; ++j)
                b[j].load_half(b_row[j] + off);
#pragma unroll
            for (int i = 0; i < MT; ++i)
                a[i].load_half(a_row[i] + off);
            multiply(a, b, GRID == 1 ? 2 : 1, true);
        }
    }

    // The waves' sums: [wave][i][j][lane].  (Their number is a constant: the reads of a sum are then in flight together, which
    // makes a call 0.1 to 0.4 us shorter.)
    Acc *park = reinterpret_cast<Acc *>(smem);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
            park[((wave * MT + i) * NT + j) * 64 + lane] = acc[i][j];
    __syncthreads();
    const bool quad_ok = y && (ld_y & 3) == 0 && (reinterpret_cast<uintptr_t>(y) & 7) == 0;
    for (int t = tid; t < MT * NT * 64; t += 64 * WAVES) {
        Acc sum = park[t];
#pragma unroll
        for (int v = 1; v < WAVES; ++v)
            sum += park[v * (MT * NT * 64) + t];
        const int tile = t >> 6, l = t & 63;
        const int m = m0 + 16 * (tile / NT) + (l & 15), n = n0 + 16 * (tile % NT) + 4 * (l >> 4);
        if (m >= M || n >= N)
            continue;
        if constexpr (!kFloat) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                sum[e] >>= C::kCarry;   // exact: multiples of 2^kCarry
        }
        const float sa = a_scales[m];
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = __fmul_rn(__fmul_rn((float)sum[e], sa), b_scales[min(n + e, N - 1)]);
        if (acc_out) {
            typedef typename std::remove_reference<decltype(sum[0])>::type Raw;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < N)
                    static_cast<Raw *>(acc_out)[(int64_t)m * N + n + e] = sum[e];
        }
        if (!y)
            continue;
        uint16_t *dst = y + (int64_t)m * ld_y + n;
        if (quad_ok && n + 4 <= N) {
            *reinterpret_cast<uint2 *>(dst) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
        } else {
            for (int e = 0; e < 4; ++e)
                if (n + e < N)
                    dst[e] = (uint16_t)float_to_bf16_bits(v[e]);
        }
    }
}

template <int GRID, int MT, int NT, int BATCH, int WAVES>
hipError_t launch(const SkinnyGemmArgs &a, hipStream_t stream)
{
    const dim3 grid((unsigned)((a.N + 16 * NT - 1) / (16 * NT)), (unsigned)((a.M + 16 * MT - 1) / (16 * MT)));
    hipLaunchKernelGGL((skinny_gemm_kernel<GRID, MT, NT, BATCH, WAVES>), grid, dim3(64 * WAVES), WAVES * MT * NT * 1024, stream,
                       a.a_codes, a.a_scales, a.b_codes, a.b_scales, (int)a.M, (int)a.N, (int)a.K,
                       static_cast<uint16_t *>(a.y), a.ld_y, a.acc_out);
    return hipGetLastError();
}

int64_t block_count(int64_t M, int64_t N, int mt, int nt)
{
    return ((M + 16 * mt - 1) / (16 * mt)) * ((N + 16 * nt - 1) / (16 * nt));
}

// The block: the smallest one that leaves no more than a workgroup per compute unit.  Small blocks
// spread the loads over the chip, large ones read each operand less often; a workgroup more than the
// chip holds costs a second round of latency.  Measured (us, block / waves; 4 bits):
//   2048 x 5632, 24 rows: 1x1/8 4.9, 1x1/4 6.2, 1x2/8 6.3   4096 x 1024, 64 rows: 2x2/4 3.3, 1x2/4 3.6, 1x1/4 4.0
//   4096 x 1024, 128 rows: 4x2/8 4.0, 2x2/4 4.2, 4x4/4 4.4  5632 x 2048, 128 rows: 4x4/4 7.8, 2x2/4 8.2, 4x2/8 8.4
// With 16 rows or fewer the activations are next to nothing, and 1x1 is within 3 % of the best
// everywhere (11008 x 4096, 8 rows: 1x1 6.9, 1x2 7.4).  Where blocks are many the largest one pays when the
// contraction is long enough for what it saves in reads (5632 x 5632, 128 rows: 4x4/4 14.1, 4x2/8 17.6), from 16 units
// on (E2M1 of 14: 256 x 1792, 2346 rows 7.5, 8.5; of 13 and 15, whose rows start within lines, 4 to 20 % more); else 4x2 with
// its shorter summation, by eight waves as long as a compute unit has two of its blocks at most (2048 x 1664, 512 rows: 4x2/8 5.6,
// 4x2/4 6.2, 4x4/4 6.3).  Of more blocks the compute unit with most of them decides: 4x4, of which it holds two at a time, where it
// has no more sixteens so and most places of the last round are taken (2 bits: 1664 x 1664, 972 rows, 2 x 16 and 4 x 8: 4x4/4 8.7,
// 4x2/4 9.5; 11008 x 1664, 97 rows, 2 x 16 and 3 x 8: 8.2, 7.8), with 8 units in one round (1 bit: 1024 x 1024, 1600 rows 8.2, 9.1; 512
// x 1024, 3000 rows, 2 x 16 and 3 x 8: 8.1, 7.8; 4 bits: 9920 x 1088, 807 rows, four rounds, 27.5, 25.8), with fewer not.  Two units of
// a wave in flight pay where it has just two (2 bits: 4096 x 1024, 333 rows 7.66, 7.75; 1664 x 1664, 972 rows 10.8, 9.5).  At 1671
// shapes of 33 .. 4096 rows with more than 256 blocks of 4x2 the one chosen takes 1.5 % more than the best of them in the mean.
quest_plan_few choose_block(int64_t M, int64_t N, int64_t K, int grid)
{
    constexpr int64_t kUnitsOfChip = 256;
    auto blocks = [&](int mt, int nt) { return block_count(M, N, mt, nt); };
    auto fits = [&](int mt, int nt) { return blocks(mt, nt) <= kUnitsOfChip; };
    auto block = [](int mt, int nt, int in_flight, int waves) { return quest_plan_few{16 * mt, 16 * nt, in_flight, waves}; };
    const int64_t units = K / kUnit;
    if (M <= 16 || fits(1, 1)) {
        // two units of a wave in flight when workgroups are few and the contraction is long (2048 x 5632, 1 row: 4.2
        // against 4.3; 24 rows, a workgroup for each compute unit, 5.1 against 4.9), by four waves for large E2M1 weights, two to four
        // workgroups for a compute unit (11008 x 11008, 10 rows: 18.0 against 20.3; integer codes take 3 % more so)
        if (units >= 32 && 2 * blocks(1, 1) <= kUnitsOfChip)
            return block(1, 1, 2, 8);
        if (grid == 0 && units >= 64 && blocks(1, 1) > 2 * kUnitsOfChip && blocks(1, 1) <= 4 * kUnitsOfChip)
            return block(1, 1, 2, 4);
        return block(1, 1, 1, 8);
    }
    if (fits(1, 2))
        return block(1, 2, 2, 4);
    if (M <= 32 || fits(2, 2))
        return block(2, 2, 2, 4);
    if (!fits(4, 2) && (units >= 16 || (grid == 0 && units == 14)))
        return block(4, 4, 1, 4);
    if (blocks(4, 2) <= 2 * kUnitsOfChip)
        return block(4, 2, 1, 8);
    auto most = [&](int mt, int nt) { return (blocks(mt, nt) + kUnitsOfChip - 1) / kUnitsOfChip; };   // of a compute unit
    const int64_t rounds = (most(4, 4) + 1) / 2;
    if (2 * most(4, 4) <= most(4, 2) &&
        (units > 8 ? 2 * blocks(4, 4) >= 3 * rounds * kUnitsOfChip : units == 8 && rounds == 1))
        return block(4, 4, 1, 4);
    return block(4, 2, units == 8 ? 2 : 1, 4);
}

template <int GRID>
hipError_t launch_grid(const SkinnyGemmArgs &a, hipStream_t stream)
{
    const quest_plan_few b = choose_block(a.M, a.N, a.K, GRID);
    if (b.block_rows == 16 && b.block_cols == 16) {
        if constexpr (GRID == 0) {
            if (b.waves == 4)
                return launch<GRID, 1, 1, 2, 4>(a, stream);
        }
        return b.in_flight == 2 ? launch<GRID, 1, 1, 2, 8>(a, stream) : launch<GRID, 1, 1, 1, 8>(a, stream);
    }
    if (b.block_rows == 16)
        return launch<GRID, 1, 2, 2, 4>(a, stream);
    if (b.block_rows == 32)
        return launch<GRID, 2, 2, 2, 4>(a, stream);
    if (b.block_cols == 64)
        return launch<GRID, 4, 4, 1, 4>(a, stream);
    if (b.waves == 8)
        return launch<GRID, 4, 2, 1, 8>(a, stream);
    return b.in_flight == 2 ? launch<GRID, 4, 2, 2, 4>(a, stream) : launch<GRID, 4, 2, 1, 4>(a, stream);
}

}  // namespace

// Whether this kernel is the one for the shape.  With few rows always; beyond that as long as its
// largest block leaves about one workgroup per compute unit: the tile kernels with their staging
// need whole tiles for every compute unit to be better (us, this kernel / tile kernels, 4 bits:
// 2048 x 5632 with 512 rows 14.2 / 20.7, 4096 x 1024 with 256 rows 5.8 / 6.9 and with 512 rows
// 8.2 / 7.2, 5632 x 2048 with 256 rows 11.8 / 10.5).  The tile kernels take 1 and 2 bits only after a
// re-coding pass, which moves the line (2 bits: 5632 x 2048 with 512 rows 17.0 / 19.2, 11008 x 4096
// with 512 rows 51 / 45).  Where no tile kernel covers the shape the alternative is a general kernel
// at a third of their rate.
bool skinny_gemm_preferred(int64_t M, int64_t N, int64_t K, int grid)
{
    if (M <= 64)
        return true;
    const bool tiles = K % 128 == 0 && (grid == 0 || (N >= 128 && (grid >= 3 || M >= 128)));
    return block_count(M, N, 4, 4) <= (!tiles ? 2048 : grid == 1 || grid == 2 ? 768 : 256);
}

// Makes the runtime load this file's code object now (a query of one kernel's attributes does), so
// that the first launch, which may be under graph capture, does not.
hipError_t prepare_skinny_gemm_kernels()
{
    hipFuncAttributes attr;
    return hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(skinny_gemm_kernel<4, 1, 1, 1, 8>));
}

hipError_t launch_skinny_gemm(const SkinnyGemmArgs &a, hipStream_t stream)
{
    switch (a.grid) {
    case 0: return launch_grid<0>(a, stream);
    case 1: return launch_grid<1>(a, stream);
    case 2: return launch_grid<2>(a, stream);
    case 3: return launch_grid<3>(a, stream);
    default: return launch_grid<4>(a, stream);
    }
}

}  // namespace quest

quest_plan_few quest_plan_forward_few(int32_t bits, int64_t M, int64_t N, int64_t K)
{
    return quest::choose_block(M, N, K, bits);
}
