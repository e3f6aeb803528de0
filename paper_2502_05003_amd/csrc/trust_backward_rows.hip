// The trust-masked inverse transform on the matrix cores for row lengths and block sizes that
// trust_backward_mfma.hip has no instantiation for: bf16 rows of any multiple of 64 elements, blocks
// of 16 to 4096, bf16 or fp32 out (Algorithm 2, out = IHT(M (.) g); Sec. 3.2 of arXiv 2502.05003).
//
// Data flow as in that file, with the row length and the block size as run-time values: the unit of work is
// a group of G tiles of 1024 elements (G: the tiles one block spans), so that few long rows fill the chip
// as well as many short ones; a wave loads its next unit's inputs before it transforms the current one.  Bound by the memory (4.1 bytes
// per element): 8192 x 2560 18.4 us = 4.7 TB/s (general kernel 29), 8192 x 5120 33 us = 5.2 TB/s (84);
// with one tile per group the registers leave room for eight waves per SIMD.
#include "hadamard_tile.h"
#include "quest_internal.h"

namespace quest {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kRowsPerBlock = kThreads / 64;

template <typename Out, int G>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(G == 1 ? 8 : G == 2 ? 4 : 3)))
void tb_rows_kernel(const uint16_t *__restrict__ g_a, const uint8_t *__restrict__ mask_a, int64_t rows_a, int cols,
                    int log2n, Out *__restrict__ out_a, const uint16_t *__restrict__ g_b,
                    const uint8_t *__restrict__ mask_b, int64_t rows_b, Out *__restrict__ out_b)
{
    constexpr bool kF32Out = sizeof(Out) == 4;
    const int lane = threadIdx.x & 63, m = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t rows = rows_a + rows_b;   // the second gradient's rows follow the first one's
    const int tiles = (cols + 1023) >> 10, per_lane = cols >> 6;

    v8bf bmat[2];
    hadamard_operand_any(log2n, m, h, bmat);
    const float inv_sqrt_n = inv_sqrt_pow2(log2n);
    // exchange with lane ^ 1: even lanes keep the low halves, odd lanes the high halves
    const uint32_t pair_sel = (lane & 1) ? 0x03020706u : 0x05040100u;

    // Work is counted in groups of tiles: unit (row, group), a wave takes every (number of waves)-th one.
    const int groups = (tiles + G - 1) / G;
    const uint32_t stride = gridDim.x * kRowsPerBlock;
    const int stride_rows = (int)(stride / (uint32_t)groups), stride_groups = (int)(stride % (uint32_t)groups);
    const uint32_t first_unit = blockIdx.x * kRowsPerBlock + wave;
    int64_t at = first_unit / (uint32_t)groups;
    int group = (int)(first_unit % (uint32_t)groups);

    v4u raw[G][2];
    uint32_t bits[G];
    // this lane's 16 elements of tile row m of the unit's tiles; elements beyond the row's end: others, not trusted
    auto load = [&](int64_t row_of_launch, int g0) {
        const bool from_b = row_of_launch >= rows_a;
        const int64_t row = from_b ? row_of_launch - rows_a : row_of_launch;
        const uint8_t *mask = from_b ? mask_b : mask_a;
        const uint16_t *src = (from_b ? g_b : g_a) + row * cols;
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int p = 1024 * (g0 + u) + 32 * m;
            const int from = min(p, cols - 32) + 16 * h;
            raw[u][0] = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(src + from));
            raw[u][1] = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(src + from + 8));
            bits[u] = mask ? *reinterpret_cast<const uint16_t *>(mask + row * (cols / 8) + (from >> 3)) : 0xffffu;
            bits[u] = p < cols ? bits[u] : 0u;
        }
    };
    if (at < rows)
        load(at, G * group);
    while (at < rows) {
        const bool from_b = at >= rows_a;
        Out *out = from_b ? out_b + (at - rows_a) * cols : out_a + at * cols;
        const int g0 = G * group;
        v8bf frag[G][2];
#pragma unroll
        for (int u = 0; u < G; ++u) {
            uint32_t w[8] = {raw[u][0].x, raw[u][0].y, raw[u][0].z, raw[u][0].w,
                             raw[u][1].x, raw[u][1].y, raw[u][1].z, raw[u][1].w};
#pragma unroll
            for (int i = 0; i < 8; ++i)
                w[i] = keep_trusted(w[i], bits[u], 2 * i);
            __builtin_memcpy(&frag[u][0], &w[0], 16);
            __builtin_memcpy(&frag[u][1], &w[4], 16);
        }
        at += stride_rows;
        group += stride_groups;
        if (group >= groups) {
            group -= groups;
            ++at;
        }
        if (at < rows)
            load(at, G * group);
        float acc[G][16];
#pragma unroll
        for (int u = 0; u < G; ++u) {
            v16f z;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                z[r] = 0.0f;
            z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[u][0], bmat[0], z, 0, 0, 0);
            z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[u][1], bmat[1], z, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[u][r] = z[r];
            one_tile_stages(log2n, acc[u]);
        }
        tile_pair_stages<G>(log2n, acc);

        // element = lane + 64 iota; this group holds iota = 16 g0 .. as far as the row goes
        const int first = 16 * g0, count = min(per_lane - first, 16 * G);
        if constexpr (kF32Out) {
            float *dst = out + lane + 64 * first;
#pragma unroll
            for (int i = 0; i < 16 * G; ++i)
                if (i < count)
                    __builtin_nontemporal_store(__fmul_rn(acc[i >> 4][reg_of_iota(i & 15)], inv_sqrt_n), dst + 64 * i);
        } else {
            // (iota, iota + 1) as a bf16 pair, halves exchanged with lane ^ 1: an even lane stores elements
            // (l, l + 1) of iota, an odd one (l - 1, l) of iota + 1
            uint32_t *dst = reinterpret_cast<uint32_t *>(out) + (m >> 1) + 16 * h + 32 * (lane & 1) + 32 * first;
#pragma unroll
            for (int i = 0; i < 16 * G; i += 2) {
                if (i < count) {
                    const uint32_t own =
                        pack_bf16_pair(__fmul_rn(acc[i >> 4][reg_of_iota(i & 15)], inv_sqrt_n),
                                       __fmul_rn(acc[(i + 1) >> 4][reg_of_iota((i + 1) & 15)], inv_sqrt_n));
                    const uint32_t other = (uint32_t)__builtin_amdgcn_ds_swizzle((int)own, (1 << 10) | 0x1f);
                    if (i + (lane & 1) < count)
                        __builtin_nontemporal_store(__builtin_amdgcn_perm(other, own, pair_sel), dst + 32 * i);
                }
            }
        }
    }
}

template <typename Out, int G>
hipError_t launch(const BackwardArgs &a, hipStream_t stream)
{
    const int64_t units = (a.rows + a.rows2) * ((a.cols + 1024 * G - 1) / (1024 * G));
    const int64_t needed = (units + kRowsPerBlock - 1) / kRowsPerBlock, resident = 256 * (G == 1 ? 8 : G == 2 ? 4 : 3);
    hipLaunchKernelGGL((tb_rows_kernel<Out, G>), dim3((unsigned)(needed < resident ? needed : resident)), dim3(kThreads), 0,
                       stream, static_cast<const uint16_t *>(a.g), a.mask, a.rows, (int)a.cols, a.log2n,
                       static_cast<Out *>(a.out), static_cast<const uint16_t *>(a.g2), a.mask2, a.rows2,
                       static_cast<Out *>(a.out2));
    return hipGetLastError();
}

template <typename Out>
hipError_t launch_span(const BackwardArgs &a, hipStream_t stream)
{
    return a.log2n <= 10 ? launch<Out, 1>(a, stream) : a.log2n == 11 ? launch<Out, 2>(a, stream) : launch<Out, 4>(a, stream);
}

}  // namespace

// Makes the runtime load this file's code object now (a query of one kernel's attributes does).
hipError_t prepare_trust_backward_rows_kernels()
{
    hipFuncAttributes attr;
    return hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(tb_rows_kernel<uint16_t, 1>));
}

// Not blocks of 8 or less, which the general kernel has in registers straight from its loads and never exchanges (us, here /
// there: block 8, 8192 x 3392 23.3 / 20.1, 8192 x 1280 to fp32 14.0 / 11.9, 300 x 448 3.2 / 2.6; 8192 x 448 6.4 / 7.3; block 16,
// 8192 x 3392 23.3 / 33.6, 300 x 448 3.2 / 3.0).
bool trust_backward_rows_covers(const BackwardArgs &a)
{
    return a.g_dtype == QUEST_BF16 && a.cols % 64 == 0 && a.log2n >= 4 && a.log2n <= 12;
}

hipError_t launch_trust_backward_rows(const BackwardArgs &a, hipStream_t stream)
{
    return a.out_dtype == QUEST_BF16 ? launch_span<uint16_t>(a, stream) : launch_span<float>(a, stream);
}

}  // namespace quest
