// The fused quantizer on the matrix cores for row lengths and block sizes that hadamard_quantize_mfma.hip
// has no instantiation for: any row of a multiple of 64 elements, any block up to 4096, every grid,
// bf16 rows, and fp32 rows in blocks of 16 or more (Algorithm 1, one operand or both; Sec. 3.1, 3.2 and 4.4 of arXiv 2502.05003).
//
// Data flow per row as in that file (which see for the index bookkeeping), with the row length and the
// block size as run-time values: a wave brings a row into its own LDS buffer by global -> LDS transfers,
// takes the sum of squares from there, and then transforms, rounds and stores the row in groups of G
// tiles of 1024 elements (two, or four for the block of 4096), reading each tile out of LDS when its turn
// comes.  The next row is requested as soon as the last group's tiles have been read.  When there are
// fewer rows than waves to fill the chip, a workgroup shares a row instead.  A tile that the row
// does not reach is skipped; one that it ends in is transformed whole, with zeros.
//
// Measured against the general kernel (b = 4, us): bf16 8192 x 2560 48.7 -> 15.6, 8192 x 5120 94 -> 29.7,
// 333 x 2560 7.2 -> 5.1; fp32 8192 x 2560 48.9 -> 26.7.  What bounds it is the vector unit: of 11008 x 2560, b = 4 with its
// mask, 25.9 us for 1045 vector instructions per row.  Hence straight code where the row fills a group of tiles (no test
// for its end, no zeroing of what is not there) and for each block size (see one_tile_stages): 21.9 us in the same run (22.7 and
// 20.8 in another), and 8192 elements in blocks of 4096, 4096 rows, 33.1 -> 23.0.
#include "hadamard_tile.h"
#include "quest_internal.h"
#include "row_staging.h"

#include <type_traits>

namespace quest {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// GRID: bits of the Eq. 1 grid (1, 2, 3, 4, 8), or 0 for E2M1.
template <int GRID, typename In, int G>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(G == 2 || sizeof(In) == 2 ? 4 : 3)))
void hq_rows_kernel(const In *__restrict__ x_a, int64_t rows_a, int64_t ld_a, int cols, int log2n, float alpha,
                    float trust_edge, uint8_t *__restrict__ codes_a, float *__restrict__ scales_a,
                    uint8_t *__restrict__ mask_a, float *__restrict__ xh_out, const In *__restrict__ x_b,
                    int64_t rows_b, int64_t ld_b, uint8_t *__restrict__ codes_b, float *__restrict__ scales_b,
                    uint8_t *__restrict__ mask_b, int row_buffer, bool shared_row)
{
    constexpr bool kF32 = sizeof(In) == 4, kFp4 = GRID == 0;
    constexpr int BITS = kFp4 ? 4 : GRID, CB = BITS == 3 ? 4 : BITS, kLevels = 1 << BITS;
    // Whether a row can end within a group of tiles: not where a block is as long as a group
    constexpr bool kCanEnd = G == 2;
    typedef std::true_type Whole;
    typedef std::false_type Ending;
    extern __shared__ __attribute__((aligned(16))) uint8_t row_buffers[];
    __shared__ float wave_sums[4];

    const int lane = threadIdx.x & 63, m = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int64_t rows = rows_a + rows_b;     // the second operand's rows follow the first one's
    const int row_bytes = cols * (int)sizeof(In);
    const int tiles = (cols + 1023) >> 10, per_lane = cols >> 6;   // elements per lane
    // A row is one wave's, or (shared_row, wave-uniform like everything that follows from it) its
    // workgroup's: the waves then take transfers and groups of tiles in turn.
    const int sums = partial_sums_of_row(tiles, G);
    const int part = shared_row ? wave : 0, parts = shared_row ? waves : 1;
    const uint8_t *const buffer = row_buffers + (shared_row ? 0 : wave * row_buffer);
    const uint32_t buffer_addr = lds_address(row_buffers) + (uint32_t)(shared_row ? 0 : wave * row_buffer);

    typedef RowStaging<(int)sizeof(In)> Staging;
    auto request_row = [&](int64_t row_of_launch) {
        const bool from_b = row_of_launch >= rows_a;
        const char *base = reinterpret_cast<const char *>(from_b ? x_b + (row_of_launch - rows_a) * ld_b
                                                                 : x_a + row_of_launch * ld_a);
        for (int at = 1024 * part; at < row_bytes; at += 1024 * parts)
            lds_dma16_stream(base, (uint32_t)Staging::source(at, lane, row_bytes), buffer_addr + (uint32_t)at);
    };
    const int64_t row_stride = shared_row ? gridDim.x : (int64_t)gridDim.x * waves;
    int64_t row_of_launch = shared_row ? blockIdx.x : (int64_t)blockIdx.x * waves + wave;
    if (row_of_launch < rows)
        request_row(row_of_launch);

    v8bf bmat[2], bneg[2];
    hadamard_operand_any(log2n, m, h, bmat);
#pragma unroll
    for (int s = 0; kF32 && s < 2; ++s) {   // -H, for the middle piece of fp32 values
        uint32_t w[4];
        __builtin_memcpy(w, &bmat[s], 16);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            w[i] ^= (w[i] & 0x00800080u) << 8;   // bit 7 is set in +-1 and clear in 0: flip the sign of the former
        __builtin_memcpy(&bneg[s], w, 16);
    }
    TransposePlan<3, 4> nibble_plan;
    TransposePlan<2, 8> byte_plan;
    TransposePlan<4, 2> pair_plan;
    TransposePlan<5, 1> bit_plan;
    if (CB == 4)
        nibble_plan.init(lane);
    if (CB == 8)
        byte_plan.init(lane);
    if (CB == 2)
        pair_plan.init(lane);
    bit_plan.init(lane);
    const float inv_sqrt_n = inv_sqrt_pow2(log2n), sqrt_n = sqrt_pow2(log2n);
    const int code_word = ((lane >> 3) & 3) + 4 * h + 8 * (lane & 7);

    // This lane's share of a tile: 16 consecutive elements of tile row m (zeros beyond the row's end, which
    // only the tile past the last whole one can reach)
    const int whole_tiles = cols >> 10;
    auto read_bf16 = [&](auto whole, int t, uint32_t (&w)[8]) __attribute__((always_inline)) {
        const v4u a = *reinterpret_cast<const v4u *>(buffer + Staging::read(t, m, h, 0, row_buffer));
        const v4u b = *reinterpret_cast<const v4u *>(buffer + Staging::read(t, m, h, 1, row_buffer));
        const bool there = whole() || 1024 * t + 32 * m < cols;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            w[i] = there ? a[i] : 0u;
            w[4 + i] = there ? b[i] : 0u;
        }
    };
    auto read_f32 = [&](auto whole, int t, float (&f)[16]) __attribute__((always_inline)) {
        const bool there = whole() || 1024 * t + 32 * m < cols;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const v4u v = *reinterpret_cast<const v4u *>(buffer + Staging::read(t, m, h, i, row_buffer));
#pragma unroll
            for (int e = 0; e < 4; ++e)
                f[4 * i + e] = there ? __uint_as_float(v[e]) : 0.0f;
        }
    };

    for (; row_of_launch < rows; row_of_launch += row_stride) {
        const bool from_b = row_of_launch >= rows_a;
        const int64_t row = from_b ? row_of_launch - rows_a : row_of_launch;
        uint8_t *mask = from_b ? mask_b : mask_a;
        wait_vmcnt<0>();   // the row has landed
        asm volatile("" ::: "memory");
        if (shared_row)
            __syncthreads();

        // The block transform is orthonormal: the sum of squares of the inputs, in as many partial sums as a shared
        // row has waves (see partial_sums_of_row)
        auto partial_sum = [&](int c) {
            float sumsq = 0.0f;
            auto add_tile = [&](auto whole, int t) __attribute__((always_inline)) {
                if constexpr (kF32) {
                    float f[16];
                    read_f32(whole, t, f);
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        sumsq = __fmaf_rn(f[i], f[i], sumsq);
                } else {
                    uint32_t w[8];
                    read_bf16(whole, t, w);
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        v2bf pair;
                        __builtin_memcpy(&pair, &w[i], 4);
                        sumsq = __builtin_amdgcn_fdot2_f32_bf16(pair, pair, sumsq, false);
                    }
                }
            };
            int t = c;
            for (; t < whole_tiles; t += sums)
                add_tile(Whole(), t);
            if (kCanEnd && t < tiles)
                add_tile(Ending(), t);
            return wave_sum_dpp(sumsq);
        };
        float total = partial_sum(part);   // shared_row: parts = sums
        if (shared_row) {
            if (lane == 0)
                wave_sums[wave] = total;
            __syncthreads();
            total = wave_sums[0];
            for (int c = 1; c < sums; ++c)
                total += wave_sums[c];
        } else {
            for (int c = 1; c < sums; ++c)
                total += partial_sum(c);
        }
        const RowConstants row_is = row_constants<kLevels, kFp4>(total, cols, alpha, trust_edge, inv_sqrt_n, sqrt_n);
        const float to_cell = row_is.to_cell, trust_raw = row_is.trust_raw;
        const bool zero_row = row_is.zero_row;
        if (lane == 0 && part == 0)
            (from_b ? scales_b : scales_a)[row] = row_is.scale;
        uint32_t *code_row = reinterpret_cast<uint32_t *>((from_b ? codes_b : codes_a) + row * (cols * CB / 8));
        uint32_t *mask_row = reinterpret_cast<uint32_t *>(mask + row * (cols / 8));

        // A group of tiles that the row fills has no test in it; the one that it ends in skips what is not there
        auto group = [&](auto whole, int g0) __attribute__((always_inline)) {
            float acc[G][16];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const int t = g0 + u;
                if (whole() || t < tiles) {   // wave-uniform
                    v16f z;
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        z[r] = 0.0f;
                    v8bf p0, p1;
                    if constexpr (kF32) {
                        float f[16];
                        read_f32(whole, t, f);
                        uint32_t hi[8], mid[8], lo[8];
                        split_bf16(f, hi, mid, lo);
                        __builtin_memcpy(&p0, &lo[0], 16);      // smallest piece first
                        __builtin_memcpy(&p1, &lo[4], 16);
                        z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p0, bmat[0], z, 0, 0, 0);
                        z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p1, bmat[1], z, 0, 0, 0);
                        __builtin_memcpy(&p0, &mid[0], 16);     // holds -mid
                        __builtin_memcpy(&p1, &mid[4], 16);
                        z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p0, bneg[0], z, 0, 0, 0);
                        z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p1, bneg[1], z, 0, 0, 0);
                        __builtin_memcpy(&p0, &hi[0], 16);
                        __builtin_memcpy(&p1, &hi[4], 16);
                    } else {
                        uint32_t w[8];
                        read_bf16(whole, t, w);
                        __builtin_memcpy(&p0, &w[0], 16);
                        __builtin_memcpy(&p1, &w[4], 16);
                    }
                    z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p0, bmat[0], z, 0, 0, 0);
                    z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p1, bmat[1], z, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        acc[u][r] = z[r];
                    if (G == 2)
                        one_tile_stages(log2n, acc[u]);
                }
            }
            if (!shared_row && g0 + G >= tiles) {   // the last tiles of the row have been read: the buffer may be refilled
                __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
                asm volatile("" ::: "memory");
                if (row_of_launch + row_stride < rows)
                    request_row(row_of_launch + row_stride);
            }
            if constexpr (G == 4)   // blocks of 4096
                tile_stages<12, G>(acc);
            else if (whole())   // (blocks of several tiles are in whole groups only)
                tile_pair_stages<G>(log2n, acc);

            // in-lane elements of this group: 16 g0 .. , as far as the row goes
            constexpr int kGroupI = 16 * G;
            const int first = 16 * g0, count_i = whole() ? kGroupI : per_lane - first;
            auto elem = [&](int i) { return acc[i >> 4][reg_of_iota(i & 15)]; };
            if (xh_out && !from_b) {   // debug output of the first operand only: element = lane + 64 iota
                float *dst = xh_out + row * cols + lane + 64 * first;
#pragma unroll
                for (int i = 0; i < kGroupI; ++i)
                    if (i < count_i)
                        dst[64 * i] = __fmul_rn(elem(i), inv_sqrt_n);
            }
            auto store = [&](uint32_t *p, uint32_t v) { __builtin_nontemporal_store(v, p); };
            // Codes: see hq_mfma_kernel for the bit tricks
            auto code_byte = [&](int i) { return cell_byte<BITS>(elem(i), to_cell); };
            if constexpr (CB == 4) {
#pragma unroll
                for (int dd = 0; dd < 2 * G; ++dd) {
                    if (8 * dd < count_i) {
                        uint32_t packed;
                        if (kFp4) {
                            // (+ 0: the zero row's products are -0 for negative entries)
                            auto scaled = [&](int i) { return __fmaf_rn(elem(8 * dd + i), to_cell, 0.0f); };
                            packed = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, scaled(0), scaled(1), 1.0f, 0);
                            packed = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(packed, scaled(2), scaled(3), 1.0f, 1);
                            packed = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(packed, scaled(4), scaled(5), 1.0f, 2);
                            packed = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(packed, scaled(6), scaled(7), 1.0f, 3);
                        } else {
                            uint32_t even = 0, odd = 0;
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                const float t = code_byte(8 * dd + i);
                                if (i & 1)
                                    odd = __builtin_amdgcn_cvt_pk_u8_f32(t, i >> 1, odd);
                                else
                                    even = __builtin_amdgcn_cvt_pk_u8_f32(t, i >> 1, even);
                            }
                            packed = BITS == 4 ? ((even >> 4) & 0x0f0f0f0fu) | (odd & 0xf0f0f0f0u)
                                               : ((even >> 5) & 0x07070707u) | ((odd >> 1) & 0x70707070u);
                        }
                        const uint32_t word = nibble_plan.apply(packed);
                        if (8 * dd + (lane & 7) < count_i)
                            store(code_row + code_word + 64 * (2 * g0 + dd), word);
                    }
                }
            } else if constexpr (CB == 8) {
#pragma unroll
                for (int w = 0; w < 4 * G; ++w) {
                    if (4 * w < count_i) {
                        uint32_t packed = 0;
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            packed = __builtin_amdgcn_cvt_pk_u8_f32(code_byte(4 * w + i), i, packed);
                        packed = byte_plan.apply(packed);
                        if (4 * w + (lane & 3) < count_i)
                            store(code_row + (lane >> 2) + 16 * (lane & 3) + 64 * (4 * g0 + w), packed);
                    }
                }
            } else if constexpr (CB == 2) {
#pragma unroll
                for (int t16 = 0; t16 < G; ++t16) {
                    if (16 * t16 < count_i) {
                        uint32_t packed = 0;
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            uint32_t e = 0;
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                e = __builtin_amdgcn_cvt_pk_u8_f32(code_byte(16 * t16 + k + 4 * j), j, e);
                            packed |= ((e >> 6) & 0x03030303u) << (2 * k);
                        }
                        packed = pair_plan.apply(packed);
                        if (16 * t16 + (lane & 15) < count_i)
                            store(code_row + (lane >> 4) + 4 * (lane & 15) + 64 * (g0 + t16), packed);
                    }
                }
            }
            // One bit per element in iota order (the code for b = 1: not negative; the mask: the sign of
            // trust_raw - |raw|), then the 32 x 32 bit transpose.  Bits of elements the row does not have
            // land in lanes that do not store.
#pragma unroll
            for (int cc = 0; cc * 32 < kGroupI; ++cc) {
                if (32 * cc < count_i) {
                    const bool mine = 32 * cc + m < count_i;
                    const int at = h + 2 * (m + 32 * (g0 / 2 + cc));
                    if constexpr (CB == 1) {
                        uint32_t negative = 0;
#pragma unroll
                        for (int half = 1; half >= 0; --half)
                            if (32 * cc + 16 * half < count_i) {
#pragma unroll
                                for (int i = 15; i >= 0; --i)
                                    negative = __builtin_amdgcn_alignbit(
                                        negative, __float_as_uint(elem(32 * cc + 16 * half + i)), 31);
                            }
                        const uint32_t code = bit_plan.apply(zero_row ? ~0u : ~negative);
                        if (mine)
                            store(code_row + at, code);
                    }
                    if (mask) {
                        uint32_t untrusted = 0;
#pragma unroll
                        for (int half = 1; half >= 0; --half)
                            if (32 * cc + 16 * half < count_i) {
#pragma unroll
                                for (int i = 15; i >= 0; --i) {   // slack negative <=> untrusted
                                    const float slack = trust_raw - fabsf(elem(32 * cc + 16 * half + i));
                                    untrusted = __builtin_amdgcn_alignbit(untrusted, __float_as_uint(slack), 31);
                                }
                            }
                        const uint32_t trusted = bit_plan.apply(~untrusted);
                        if (mine)
                            store(mask_row + at, trusted);
                    }
                }
            }
        };
        int g0 = G * part;
        for (; g0 + G <= whole_tiles; g0 += G * parts)
            group(Whole(), g0);
        if (kCanEnd && g0 < tiles)
            group(Ending(), g0);
        if (shared_row && row_of_launch + row_stride < rows) {
            __syncthreads();   // every wave has read its tiles and the sums
            request_row(row_of_launch + row_stride);
        }
    }
}

template <int GRID, typename In, int G>
hipError_t launch(const QuantizeArgs &a, hipStream_t stream)
{
    auto kernel = hq_rows_kernel<GRID, In, G>;
    const int buffer = RowStaging<(int)sizeof(In)>::buffer_bytes((int)a.cols), groups = (int)((a.cols + 1024 * G - 1) / (1024 * G));
    const int64_t rows = a.rows + a.rows2;
    // A workgroup shares a row when there are few rows, and when sixteen waves' rows would not fit a compute
    // unit's LDS (us, a row per wave / shared: 333 x 5120 7.7 / 5.5, 1000 x 2560 6.1 / 5.3, 1400 x 2560 6.8 / 6.8,
    // 8192 x 2560 15.7 / 19.2, 8192 x 5120 29.1 / 29.7, 8192 x 6144 33.2 / 32.0, 4096 x 8192 in blocks of 4096 26.4 / 21.8;
    // fp32 8192 x 5120 79 / 44).
    const bool shared_row = groups > 1 && (rows <= 1024 || buffer > 10 * 1024);
    // waves per workgroup: four, fewer when a shared row has fewer groups of tiles (one partial sum each); sixteen
    // per compute unit at most.  LDS: a shared row's buffer or, of rows of one group or of 10 KiB, four: 64 KiB at most.
    const int waves = shared_row ? partial_sums_of_row((int)((a.cols + 1023) / 1024), G) : 4;
    const int lds = shared_row ? buffer : waves * buffer;
    if (lds > 48 * 1024) {
        static OncePerDevice once;
        const hipError_t err = once([&] { return allow_dynamic_lds(reinterpret_cast<const void *>(kernel), 64 * 1024); });
        if (err != hipSuccess)
            return err;
    }
    const int64_t needed = shared_row ? rows : (rows + waves - 1) / waves, resident = 256 * (16 / waves);
    const dim3 grid((unsigned)(needed < resident ? needed : resident));
    hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), lds, stream, static_cast<const In *>(a.x), a.rows, a.ld,
                       (int)a.cols, a.log2n, a.alpha, a.trust_edge, a.codes, a.scales, a.mask, a.xh_out,
                       static_cast<const In *>(a.x2), a.rows2, a.ld2, a.codes2, a.scales2, a.mask2, buffer, shared_row);
    return hipGetLastError();
}

template <int GRID>
hipError_t launch_grid(const QuantizeArgs &a, hipStream_t stream)
{
    if (a.dtype == QUEST_F32)
        return a.log2n <= 11 ? launch<GRID, float, 2>(a, stream) : launch<GRID, float, 4>(a, stream);
    return a.log2n <= 11 ? launch<GRID, uint16_t, 2>(a, stream) : launch<GRID, uint16_t, 4>(a, stream);
}

template <int GRID>
hipError_t prepare_grid()
{
    hipError_t err = allow_dynamic_lds(reinterpret_cast<const void *>(hq_rows_kernel<GRID, uint16_t, 2>), 64 * 1024);
    if (err == hipSuccess)
        err = allow_dynamic_lds(reinterpret_cast<const void *>(hq_rows_kernel<GRID, uint16_t, 4>), 64 * 1024);
    if (err == hipSuccess)
        err = allow_dynamic_lds(reinterpret_cast<const void *>(hq_rows_kernel<GRID, float, 2>), 64 * 1024);
    if (err == hipSuccess)
        err = allow_dynamic_lds(reinterpret_cast<const void *>(hq_rows_kernel<GRID, float, 4>), 64 * 1024);
    return err;
}

}  // namespace

hipError_t prepare_quantize_rows_kernels()
{
    hipError_t err = prepare_grid<0>();
    if (err == hipSuccess)
        err = prepare_grid<1>();
    if (err == hipSuccess)
        err = prepare_grid<2>();
    if (err == hipSuccess)
        err = prepare_grid<3>();
    if (err == hipSuccess)
        err = prepare_grid<4>();
    if (err == hipSuccess)
        err = prepare_grid<8>();
    return err;
}

// Which calls come here (`rows`: of both operands).  Everything that hadamard_quantize_mfma.hip has no instantiation
// for, up to blocks of 4096: faster than the general kernel, in most shapes at every number of rows (us, here / there, 24
// rows: 2560 elements 4.6 / 6.6, 5120 4.6 / 11.0, 64 3.6 / 4.3).  The exceptions are blocks of 8 or less, which the
// general kernel has in registers straight from its loads: bf16 rows still come here (50 x 1280 4.6 / 4.0, 750 x 1280
// 4.8 / 4.9, 8192 x 1280 10.8 / 21.8), fp32 rows, which gain little, do not (50 x 1344 5.7 / 4.0, 8192 x 3584 30 / 35).
// Of the fp32 shapes that it has, which it holds in registers as
// a whole: long rows, and many rows (here / there: 24 rows of 2816 5.4 / 5.5, 3584 5.4 / 6.3, 5632 5.5 / 7.9;
// 768 x 2048 5.6 / 5.3, 1024 x 2048 5.8 / 6.6, 8192 x 2048 18.6 / 25.2; 1024 x 1024 4.6 / 4.3, 2048 x 1024 5.2 / 6.4;
// blocks of 4096, 24 rows 6.9 / 6.3, 1024 rows 8.7 / 9.2, 8192 rows 38.6 / 50.9).  Both kernels make the same bits of these
// rows, so the number of rows may decide; for bf16 rows they do not, and the shape alone does.
bool quantize_rows_preferred(const QuantizeArgs &a, int64_t rows)
{
    if (a.cols % 64 != 0 || a.log2n > 12 || a.mode == kQuantAbsMax)
        return false;
    if (!launch_hadamard_quantize_mfma(a, nullptr, true))
        return a.dtype == QUEST_BF16 || a.log2n > 3;
    return a.dtype == QUEST_F32 && a.cols >= 1024 &&
           (rows >= 2048 || (rows >= 1024 && a.cols >= 2048) || (a.cols > 2816 && a.log2n < 12));
}

hipError_t launch_hadamard_quantize_rows(const QuantizeArgs &a, hipStream_t stream)
{
    if (a.mode == kQuantFp4)
        return launch_grid<0>(a, stream);
    switch (a.bits) {
    case 1: return launch_grid<1>(a, stream);
    case 2: return launch_grid<2>(a, stream);
    case 3: return launch_grid<3>(a, stream);
    case 4: return launch_grid<4>(a, stream);
    default: return launch_grid<8>(a, stream);
    }
}

}  // namespace quest
