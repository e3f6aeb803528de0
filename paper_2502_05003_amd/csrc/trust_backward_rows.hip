// The trust-masked inverse transform on the matrix cores for row lengths and block sizes that
// trust_backward_mfma.hip has no instantiation for: bf16 rows of any multiple of 64 elements, blocks
// of 16 to 4096, bf16 or fp32 out (Algorithm 2, out = IHT(M (.) g); Sec. 3.2 of arXiv 2502.05003).
//
// Rows are contiguous and made of whole blocks, and nothing but the blocks couples elements, so the rows do
// not matter: a gradient is cut into units of T tiles of 1024 consecutive elements, whatever rows they belong to (T = 2, or
// 4 for the block of 4096; units are whole blocks, and tiles start at a row start or a multiple of 64 from it, so that
// an infinity or a NaN stays in its row).  Only a gradient's last unit can be partial.
//
// Data flow of a unit as in that file: a wave brings it into its own LDS buffer by global -> LDS transfers, one
// unit ahead of the one that it transforms; the stores are issued by hand and counted, and the wait for a unit is for "all
// but that many", or but 24 where a unit has 32 or 64 (fp32 outputs, blocks of 4096), whose oldest stores have long gone
// (us, so / all but 32 or 63: fp32 11008 x 2560 32.0 / 32.0, blocks of 4096 8192 x 12288 72.9 / 72.7, to fp32 111.8 /
// 112.5).  Bound by the memory (4.1 bytes per element).  Cut at rows instead, in units of the one tile that a block
// spans, loaded into registers (us, so / now): 18432 x 5632 81.7 -> 71.9 = 6.0 TB/s, 11008 x 2560 23.7 -> 21.9,
// 2000 x 3584 8.3 -> 6.4, 8192 x 6144 block 2048 40.5 -> 35.9, 1000 x 12288 block 4096 12.0 -> 9.8.
#include "gemm_tile.h"
#include "hadamard_tile.h"
#include "quest_internal.h"

namespace quest {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// A unit: up to 1024 T consecutive elements of a gradient
struct Unit {
    bool from_b;     // of the second gradient
    int64_t first;   // element of its gradient
    int exists;      // elements of the unit that exist: a multiple of 64
};

template <int T>
__device__ __forceinline__ Unit unit_at(uint32_t unit, uint32_t units_a, int64_t elements_a, int64_t elements_b)
{
    Unit w;
    w.from_b = unit >= units_a;
    w.first = (int64_t)(w.from_b ? unit - units_a : unit) * (1024 * T);
    const int64_t left = (w.from_b ? elements_b : elements_a) - w.first;
    w.exists = left < 1024 * T ? (int)left : 1024 * T;
    return w;
}

// A lane's sixteen elements of tile row m of a tile, the untrusted ones zeroed, as operands of the two instructions
__device__ __forceinline__ void masked_operand(const v4u &n0, const v4u &n1, uint32_t bits, v8bf (&frag)[2])
{
    uint32_t w[8] = {n0.x, n0.y, n0.z, n0.w, n1.x, n1.y, n1.z, n1.w};
#pragma unroll
    for (int i = 0; i < 8; ++i)
        w[i] = keep_trusted(w[i], bits, 2 * i);
    __builtin_memcpy(&frag[0], &w[0], 16);
    __builtin_memcpy(&frag[1], &w[4], 16);
}

template <int T>
__device__ __forceinline__ void transform(int log2n, const v8bf (&frag)[T][2], const v8bf (&bmat)[2], float (&acc)[T][16])
{
#pragma unroll
    for (int u = 0; u < T; ++u) {
        v16f z;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            z[r] = 0.0f;
        z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[u][0], bmat[0], z, 0, 0, 0);
        z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[u][1], bmat[1], z, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r)
            acc[u][r] = z[r];
        if constexpr (T < 4)
            one_tile_stages(log2n, acc[u]);
    }
    if constexpr (T == 4)   // blocks of 4096
        tile_stages<12, T>(acc);
    else
        tile_pair_stages<T>(log2n, acc);
}

// Scales, rounds and stores a unit (WHOLE) or the part of it that exists, in order and by instructions that the compiler
// does not move; the number of them.  Element = lane + 64 iota.
template <bool WHOLE, typename Out, int T>
__device__ __forceinline__ int store_unit(const float (&acc)[T][16], float inv_sqrt_n, Out *out, int exists, int lane)
{
    const int m = lane & 31, h = lane >> 5, count = WHOLE ? 16 * T : exists >> 6;
    if constexpr (sizeof(Out) == 4) {
        static_for<16 * T>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if (WHOLE || i < count)
                store_word_counted<256 * (i & 15)>(out + 1024 * (i >> 4), 4u * lane,
                                                   __float_as_uint(__fmul_rn(acc[i >> 4][reg_of_iota(i & 15)], inv_sqrt_n)));
        });
        return count;
    } else {
        // (iota, iota + 1) as a bf16 pair, halves exchanged with lane ^ 1: an even lane (low halves) stores elements
        // (l, l + 1) of iota, an odd one (high halves) (l - 1, l) of iota + 1
        const uint32_t pair_sel = (lane & 1) ? 0x03020706u : 0x05040100u;
        const uint32_t lane_offset = 4u * ((m >> 1) + 16 * h + 32 * (lane & 1));
        static_for<8 * T>([&](auto pair) {
            constexpr int i = 2 * decltype(pair)::value;
            if (WHOLE || i < count) {
                const uint32_t own = pack_bf16_pair(__fmul_rn(acc[i >> 4][reg_of_iota(i & 15)], inv_sqrt_n),
                                                    __fmul_rn(acc[(i + 1) >> 4][reg_of_iota((i + 1) & 15)], inv_sqrt_n));
                const uint32_t other = (uint32_t)__builtin_amdgcn_ds_swizzle((int)own, (1 << 10) | 0x1f);
                if (WHOLE || i + (lane & 1) < count)
                    store_word_counted<128 * (i & 31)>(out + 64 * (i & ~31), lane_offset,
                                                       __builtin_amdgcn_perm(other, own, pair_sel));
            }
        });
        return (count + 1) / 2;
    }
}

// LDS of a wave: the gradient's elements of a unit of T tiles, then their mask bits
constexpr int buffer_bytes(int tiles)
{
    return tiles * (2048 + 128);
}

template <typename Out, int T>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
void tb_rows_kernel(const uint16_t *__restrict__ g_a, const uint8_t *__restrict__ mask_a, int64_t elements_a,
                    uint32_t units_a, uint32_t units, int log2n, Out *__restrict__ out_a, const uint16_t *__restrict__ g_b,
                    const uint8_t *__restrict__ mask_b, int64_t elements_b, Out *__restrict__ out_b)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t buffers[];
    const int lane = threadIdx.x & 63, m = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint8_t *const buffer = buffers + wave * buffer_bytes(T);
    const uint32_t buffer_addr = lds_address(buffers) + (uint32_t)(wave * buffer_bytes(T));

    // the second gradient's units follow the first one's; a wave takes every (number of waves)-th one
    const uint32_t stride = gridDim.x * kWaves;
    uint32_t unit = blockIdx.x * kWaves + wave;
    // Pieces of 16 tile rows of 64 bytes, chunk c of tile row r in slot c ^ ((r >> 2) & 3).  Lanes beyond the end fetch the
    // last bytes that exist.
    const int piece_offset = 64 * (lane >> 2) + 16 * ((lane & 3) ^ ((lane >> 4) & 3));
    auto request = [&](const Unit &w) {
        const char *base = reinterpret_cast<const char *>((w.from_b ? g_b : g_a) + w.first);
#pragma unroll
        for (int i = 0; i < 2 * T; ++i)
            lds_dma16_stream(base, (uint32_t)min(1024 * i + piece_offset, 2 * w.exists - 16), buffer_addr + 1024 * i);
        if (mask_a) {   // both masks or neither
            const char *mask = reinterpret_cast<const char *>((w.from_b ? mask_b : mask_a) + (w.first >> 3));
#pragma unroll
            for (int i = 0; i < T / 2; ++i)
                lds_dma4_stream(mask, (uint32_t)min(256 * i + 4 * lane, w.exists / 8 - 4), buffer_addr + 2048 * T + 256 * i);
        }
    };
    Unit next = {};
    if (unit < units) {
        next = unit_at<T>(unit, units_a, elements_a, elements_b);
        request(next);   // before anything else is set up
    }

    v8bf bmat[2];
    hadamard_operand_any(log2n, m, h, bmat);
    const float inv_sqrt_n = inv_sqrt_pow2(log2n);
    const int slot0 = 16 * ((2 * h) ^ ((m >> 2) & 3)), slot1 = 16 * ((2 * h + 1) ^ ((m >> 2) & 3));

    int stores_after_request = 0;   // stores issued since the transfers of the unit about to be read
    while (unit < units) {
        const Unit now = next;
        wait_vmcnt_upto(stores_after_request);
        v8bf frag[T][2];
#pragma unroll
        for (int u = 0; u < T; ++u) {
            const v4u n0 = *reinterpret_cast<const v4u *>(buffer + 2048 * u + 64 * m + slot0);
            const v4u n1 = *reinterpret_cast<const v4u *>(buffer + 2048 * u + 64 * m + slot1);
            const uint32_t bits = mask_a ? *reinterpret_cast<const uint16_t *>(buffer + 2048 * T + 128 * u + 4 * m + 2 * h)
                                         : 0xffffu;
            masked_operand(n0, n1, 1024 * u + 32 * m < now.exists ? bits : 0u, frag[u]);
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the buffer has been read, it may be refilled
        asm volatile("" ::: "memory");
        unit += stride;
        if (unit < units) {
            next = unit_at<T>(unit, units_a, elements_a, elements_b);
            request(next);
        }
        float acc[T][16];
        transform<T>(log2n, frag, bmat, acc);
        Out *out = (now.from_b ? out_b : out_a) + now.first;
        stores_after_request = now.exists == 1024 * T ? store_unit<true>(acc, inv_sqrt_n, out, now.exists, lane)
                                                      : store_unit<false>(acc, inv_sqrt_n, out, now.exists, lane);
    }
}

// Few units: one of a single tile for each wave, straight from its loads
template <typename Out>
__global__ __launch_bounds__(kThreads) void tb_few_kernel(
    const uint16_t *__restrict__ g_a, const uint8_t *__restrict__ mask_a, int64_t elements_a, uint32_t units_a,
    uint32_t units, int log2n, Out *__restrict__ out_a, const uint16_t *__restrict__ g_b,
    const uint8_t *__restrict__ mask_b, int64_t elements_b, Out *__restrict__ out_b)
{
    const int lane = threadIdx.x & 63, m = lane & 31, h = lane >> 5;
    const uint32_t unit = blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (unit >= units)
        return;
    const Unit w = unit_at<1>(unit, units_a, elements_a, elements_b);
    const int from = min(32 * m, w.exists - 32) + 16 * h;   // beyond the end: others, not trusted
    const uint16_t *src = (w.from_b ? g_b : g_a) + w.first + from;
    const v4u n0 = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(src));
    const v4u n1 = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(src + 8));
    const uint32_t bits =
        mask_a ? *reinterpret_cast<const uint16_t *>((w.from_b ? mask_b : mask_a) + ((w.first + from) >> 3)) : 0xffffu;
    v8bf bmat[2], frag[1][2];
    hadamard_operand_any(log2n, m, h, bmat);
    masked_operand(n0, n1, 32 * m < w.exists ? bits : 0u, frag[0]);
    float acc[1][16];
    transform<1>(log2n, frag, bmat, acc);
    store_unit<false>(acc, inv_sqrt_pow2(log2n), (w.from_b ? out_b : out_a) + w.first, w.exists, lane);
}

// Units of T tiles of both gradients
int64_t unit_count(const BackwardArgs &a, int tiles, int64_t *of_first)
{
    *of_first = (a.rows * a.cols + 1024 * tiles - 1) / (1024 * tiles);
    return *of_first + (a.rows2 * a.cols + 1024 * tiles - 1) / (1024 * tiles);
}

template <typename Out, int T>
hipError_t launch(const BackwardArgs &a, hipStream_t stream)
{
    int64_t units_a;
    const int64_t units = unit_count(a, T, &units_a);
    const int64_t needed = (units + kWaves - 1) / kWaves, resident = 256 * 4;
    auto kernel = T == 1 ? tb_few_kernel<Out> : tb_rows_kernel<Out, T == 1 ? 2 : T>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(T == 1 || needed < resident ? needed : resident)), dim3(kThreads),
                       T == 1 ? 0 : kWaves * buffer_bytes(T), stream, static_cast<const uint16_t *>(a.g), a.mask,
                       a.rows * a.cols, (uint32_t)units_a, (uint32_t)units, a.log2n, static_cast<Out *>(a.out),
                       static_cast<const uint16_t *>(a.g2), a.mask2, a.rows2 * a.cols, static_cast<Out *>(a.out2));
    return hipGetLastError();
}

// Which kernel: blocks of up to 1024 in few units go straight through the registers, a wave having just one or two loads
// to wait for (us, that / staged in LDS: 333 x 2560 3.4 / 3.9, 300 x 448 2.9 / 3.3; 1024 x 2560, 1280 units of two tiles,
// 4.3 / 4.4; 1024 x 4864 6.2 / 5.4).
template <typename Out>
hipError_t launch_span(const BackwardArgs &a, hipStream_t stream)
{
    int64_t units_a;
    if (a.log2n <= 10 && unit_count(a, 2, &units_a) <= 1024)
        return launch<Out, 1>(a, stream);
    return a.log2n <= 11 ? launch<Out, 2>(a, stream) : launch<Out, 4>(a, stream);
}

}  // namespace

// Makes the runtime load this file's code object now (a query of one kernel's attributes does).
hipError_t prepare_trust_backward_rows_kernels()
{
    hipFuncAttributes attr;
    return hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(tb_rows_kernel<uint16_t, 2>));
}

// Not blocks of 8 or less, which the general kernel has in registers straight from its loads and never exchanges (us, here /
// there: block 8, 8192 x 3392 23.3 / 20.1, 8192 x 1280 to fp32 14.0 / 11.9, 300 x 448 3.2 / 2.6; 8192 x 448 6.4 / 7.3; block 16,
// 8192 x 3392 23.3 / 33.6, 300 x 448 3.2 / 3.0).  Nor rows of 1664, 1792 and 2816 in such blocks, for which there was an
// instantiation of the other matrix-core kernel (that / the general one, block 8: 333 x 1792 4.0 / 3.3, 1000 x 2816 5.5 / 5.0,
// 8192 x 1792 13.5 / 12.8, 8192 x 2816 20.1 / 20.8, 16384 x 1792 24.4 / 25.5, 16384 x 2816 37.5 / 38.8; block 1 16384 x
// 1792 24.4 / 25.0): the number of rows may not decide, as the two add in different orders in blocks of 4 and 8.
bool trust_backward_rows_covers(const BackwardArgs &a)
{
    return a.g_dtype == QUEST_BF16 && a.cols % 64 == 0 && a.log2n >= 4 && a.log2n <= 12;
}

hipError_t launch_trust_backward_rows(const BackwardArgs &a, hipStream_t stream)
{
    return a.out_dtype == QUEST_BF16 ? launch_span<uint16_t>(a, stream) : launch_span<float>(a, stream);
}

}  // namespace quest
