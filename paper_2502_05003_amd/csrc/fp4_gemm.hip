// FP4 x FP4 GEMM with a dequantizing bf16 epilogue for the FP4 variant of the method (Sec. 4.4
// "The FP4 Format" of arXiv 2502.05003): y = xhat_h what_h^T on E2M1 codes, contracted on the FP4
// matrix instruction (v_mfma_scale_f32_32x32x64_f8f6f4 with unit block scales).  Products of
// E2M1 values are multiples of 1/4 below 36, so the fp32 accumulators hold sum_k v_a v_b exactly
// for K <= 65536.
//
// Same structure as the INT8 kernel for the integer grid (256 x 128 tile, four waves of 128 x 64,
// 128 contraction elements per step, three LDS stages filled by direct global -> LDS transfers, two
// workgroups per CU, transposed accumulator tiles, LDS-parked epilogue), minus the widening: the
// quantizer packs two codes per byte in element order, which is the instruction's operand layout
// (lane l: row l % 32, elements 32 (l / 32) .. + 32 of the 64-element sub-step), so a 16-byte LDS
// read is an operand.
#include <algorithm>

#include "gemm_tile.h"
#include "quest_internal.h"

namespace quest {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int TN = 128, TK = 128;
constexpr int kTileThreads = 256;
constexpr int kRowBytes = TK / 2;                      // packed bytes per tile row and step
constexpr int kStages = 3;

// AF: activation fragments of a wave.  4: tiles of 256 x 128, two workgroups per CU; 2: 128 x 128, three.
template <int AF>
struct Tile {
    static constexpr int kRows = 64 * AF;
    static constexpr int kStageBytes = (kRows + TN) * kRowBytes;   // 24 or 16 KiB
    static constexpr int kParkBytes = 4 * 32 * AF * 64 * 2;        // epilogue: four waves x 32 AF x 64 bf16
    static_assert(kParkBytes <= kStages * kStageBytes, "the epilogue parks in the stages");
    static constexpr int kLds = kStages * kStageBytes + TN * 4;    // + the tile's weight scales
};

// 16-byte chunk c (0..3) of tile row `row` lives at chunk c ^ swz(row): sixteen consecutive rows
// reading the same logical chunk hit sixteen different 16-byte slots modulo 256 bytes.
__device__ __forceinline__ int swz(int row)
{
    return (row >> 2) & 3;
}

template <int AF>
__global__ __launch_bounds__(kTileThreads, AF == 4 ? 2 : 3) void fp4_gemm_tile_kernel(
    const uint8_t *__restrict__ a_codes, const float *__restrict__ a_scales,
    const uint8_t *__restrict__ b_codes, const float *__restrict__ b_scales, int M, int N, int K,
    int tiles_m, int tiles_n, uint16_t *__restrict__ y, int64_t ld_y,
    float *__restrict__ acc_out)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    constexpr int TM = Tile<AF>::kRows, kStageBytes = Tile<AF>::kStageBytes;
    constexpr int kTransfers = AF + 2, kMatrix = 4 * AF;   // per wave and step

    // Workgroup -> tile.  Consecutive workgroup ids go to different XCDs (8 of them, each with
    // its own L2), so give each XCD one contiguous run of tiles, ordered four tile-rows deep:
    // the tiles an XCD works on at a time share a few row panels of A and column panels of B.
    const int total = tiles_m * tiles_n;
    const int per_xcd = (total + 7) / 8;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= total)
        return;
    const int band = logical / (4 * tiles_n);
    const int band_rows = min(4, tiles_m - band * 4);
    const int in_band = logical - band * 4 * tiles_n;
    const int tile_m = band * 4 + in_band % band_rows;
    const int tile_n = in_band / band_rows;
    const int m0 = tile_m * TM, n0 = tile_n * TN;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int lm = lane & 31, lh = lane >> 5;

    // Staging: codes go from global memory straight into LDS, 16 bytes per lane.  A wave's 64 lanes
    // fill 1 KiB = 16 tile rows x 64 bytes; lane l lands at offset 16 l, i.e. row l / 4, physical
    // chunk l % 4, so it fetches the logical chunk that belongs there.  Six such pieces per step and
    // wave (AF = 4): rows 64 i + 16 wave .. + 16 of A (i < 4) and of B (i = 4, 5).
    const int st_row = 16 * wave + (lane >> 2);                       // + 64 i
    const int st_chunk = (lane & 3) ^ swz(st_row);                    // swz(row + 64 i) = swz(row)
    const int64_t row_bytes = (int64_t)K / 2;
    uint32_t src_off[kTransfers];   // per-thread byte offsets from a_codes / b_codes (rows clamped at the edge)
#pragma unroll
    for (int i = 0; i < kTransfers; ++i) {
        const int row = st_row + 64 * (i < AF ? i : i - AF);
        const int64_t grow = i < AF ? min(m0 + row, M - 1) : min(n0 + row, N - 1);
        src_off[i] = (uint32_t)(grow * row_bytes + st_chunk * 16);
    }

    v16f acc[AF][2];
#pragma unroll
    for (int i = 0; i < AF; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][j][r] = 0.0f;

    const int steps = K / TK;
    // piece I of contraction step STEP -> stage at LDS byte address STAGE (wave-uniform)
    const uint32_t smem_addr = lds_address(smem);
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    // (WAVE_STAGE: LDS byte address of the stage plus this wave's 16 rows)
#define QUEST_DMA(WAVE_STAGE, I, STEP)                                                             \
    lds_dma16_at<((I) < AF ? 0 : TM * kRowBytes) + 64 * ((I) < AF ? (I) : (I)-AF) * kRowBytes>(       \
        ((I) < AF ? a_codes : b_codes) + (int64_t)min((STEP), steps - 1) * kRowBytes, src_off[I], (WAVE_STAGE))

    const uint32_t wave_smem = smem_addr + 16 * wave_u * kRowBytes;
    static_for<kTransfers>([&](auto i) { QUEST_DMA(wave_smem, decltype(i)::value, 0); });
    static_for<kTransfers>([&](auto i) { QUEST_DMA(wave_smem + kStageBytes, decltype(i)::value, 1); });
    // the epilogue's scales, fetched while the first stages are on their way: the weight scales of
    // the tile's columns into their own corner of LDS, this lane's activation scales into
    // registers
    float *scale_lds = reinterpret_cast<float *>(smem + kStages * kStageBytes);
    if (tid < TN)
        scale_lds[tid] = b_scales[min(n0 + tid, N - 1)];
    float sa_reg[AF];
#pragma unroll
    for (int i = 0; i < AF; ++i)
        sa_reg[i] = a_scales[min(m0 + wm * (32 * AF) + i * 32 + lm, M - 1)];
    wait_vmcnt<0>();
    __syncthreads();

    // fragment addresses: rows lm + 32 i share bits 2..3, hence one swizzle value per lane;
    // chunk 2 p + lh of a row feeds this lane's share of sub-steps 2 p and 2 p + 1
    const int x = swz(lm);
    const int a_off = (wm * (32 * AF) + lm) * kRowBytes;
    const int b_off = TM * kRowBytes + (wn * 64 + lm) * kRowBytes;
    uint4 af[2][AF], bf[2][2];   // packed fragments of the two sub-step pairs
    auto load_frag = [&](const uint8_t *stage, int p, int f) {
        const int off = ((2 * p + lh) ^ x) << 4;
        if (f < AF)
            af[p][f] = *reinterpret_cast<const uint4 *>(stage + a_off + f * 32 * kRowBytes + off);
        else
            bf[p][f - AF] = *reinterpret_cast<const uint4 *>(stage + b_off + (f - AF) * 32 * kRowBytes + off);
    };
    static_for<AF + 2>([&](auto f) { load_frag(smem, 0, decltype(f)::value); });

    // Main loop: 4 AF matrix instructions per step and wave.  A packed fragment (16 bytes per lane:
    // the 32 codes of its half of a 64-element sub-step) is the instruction's operand as it is.
    //   MFMA s: pair p = s / (2 AF), A fragment i = (s / 2) % AF, B fragment j = s % 2
    //   AF = 4:
    //   s = 0, 2, .. 10  start the transfers of step + 2 into the stage that was read in step - 1
    //   s = 1..6    load the fragments of pair 1 (first needed at s = 8)
    //   s = 10      wait for this wave's transfers of step + 1 (all but the six newest), barrier
    //   s = 11..15  load the fragments of pair 0 of step + 1
    //   AF = 2: transfers at s = 0..3, fragments of pair 1 two each at 0 and 1, wait and barrier at 4,
    //   fragments of pair 0 two each at 5 and 6
    // The barrier lets the other waves refill the stage that is being read, one step later, so a wave has all
    // of its reads back before it: the instructions up to s = 9 use every fragment of pair 1 (AF = 4);
    // with AF = 2 the second fragments are used behind the barrier, so those are read first, the first ones,
    // which s = 4 waits for, last, and the wait is spelled out.
    constexpr int kWaitAt = AF == 4 ? 10 : 4;
    const int one = 0x7f7f7f7f;   // block scales 2^0 (the codes carry no block scale)
    auto operand = [](const uint4 &f) { return v8i{(int)f.x, (int)f.y, (int)f.z, (int)f.w, 0, 0, 0, 0}; };
    int stage_cur = 0;   // byte offsets of the stages holding step, step + 1, step + 2
    int stage_one = kStageBytes, stage_two = 2 * kStageBytes;
    for (int step = 0; step < steps; ++step) {
        const uint8_t *cur = smem + stage_cur;
        const uint8_t *one_stage = smem + stage_one;
        static_for<kMatrix>([&](auto kc) {
            constexpr int s = decltype(kc)::value;
            constexpr int p = s / (2 * AF), i = (s >> 1) % AF, j = s & 1;
            // weight fragment as the row operand: transposed accumulator tiles
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand(bf[p][j]), operand(af[p][i]),
                                                                        acc[i][j], 4, 4, 0, one, 0, one);
            if constexpr (AF == 4 ? s <= 10 && (s & 1) == 0 : s < 4)
                QUEST_DMA(wave_smem + stage_two, (AF == 4 ? s / 2 : s), step + 2);
            if constexpr (AF == 4 && s >= 1 && s <= 6)
                load_frag(cur, 1, s - 1);
            if constexpr (AF == 2 && s < 2) {
                load_frag(cur, 1, s == 0 ? 1 : 0);
                load_frag(cur, 1, s == 0 ? AF + 1 : AF);
            }
            if constexpr (s == kWaitAt) {
                if constexpr (AF == 2)
                    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
                wait_vmcnt<kTransfers>();
                __builtin_amdgcn_s_barrier();
            }
            if constexpr (s == kWaitAt + 1) {
                load_frag(one_stage, 0, 0);
                load_frag(one_stage, 0, AF);
            }
            if constexpr (AF == 2 && s == kWaitAt + 2)
                load_frag(one_stage, 0, 1);
            if constexpr (s == kWaitAt + 2)
                load_frag(one_stage, 0, AF + 1);
            if constexpr (AF == 4 && s >= 13)
                load_frag(one_stage, 0, s - 12);
            __builtin_amdgcn_sched_barrier(0);
        });
        const int t = stage_cur;
        stage_cur = stage_one;
        stage_one = stage_two;
        stage_two = t;
    }
    wait_vmcnt<0>();   // all transfers landed before the stages are reused
#undef QUEST_DMA

    // Epilogue: each wave's 32 AF x 64 block (see store_wave_block), parked in the stages.  (Storing
    // 16-byte pieces straight from registers after a lane-pair exchange, without the detour through
    // LDS, measured 5 % slower here and 1 % slower in the INT8 kernels: whole 128-byte row segments
    // per store instruction matter more than the LDS round trip.)
    __syncthreads();   // every wave is done with the stages
    store_wave_block<AF, 0>(acc, sa_reg, scale_lds + wn * 64, smem + wave * (32 * AF * 128), m0 + wm * (32 * AF),
                            n0 + wn * 64, M, N, y, ld_y, acc_out, lane);
}

// Fewer tiles of 256 x 128 than three quarters of the chip's slots (two per CU), as for the integer kernels:
// tiles of 128 x 128 (us, 256 / 128 rows: 323 x 2992 x 4608, 24 tiles, 16.5 / 10.4; 768 x 2816 x 4096, 66 tiles,
// 14.5 / 10.5; 1728 x 1920 x 5760, 105 tiles, 26.3 / 19.3; 4096 x 2816 x 1024, 352 tiles, 14.7 / 14.4).  But not
// where each CU gets at most one large tile and some get two small ones: those CUs have the same products to do
// and read a third more for them, which a long contraction does not win back by its shorter prologue and
// epilogue (3072 x 1536, 144 tiles: K = 2048 11.4 / 11.1, K = 3072 15.4 / 15.5, K = 7296 31.6 / 36.7;
// 1815 x 4096, 256 tiles: K = 2048 14.8 / 14.5, K = 3072 18.8 / 19.7, K = 7296 36.9 / 39.7; beside it 121 tiles,
// all small ones in one round, K = 7296 31.1 / 23.2, and 288 tiles, two rounds either way, 60.2 / 55.9).
constexpr int64_t kFewTiles = 384, kUnits = 256, kLongContraction = 2560;

template <int AF>
hipError_t launch(const Fp4GemmArgs &a, hipStream_t stream)
{
    constexpr int TM = Tile<AF>::kRows;
    const int tiles_m = (int)((a.M + TM - 1) / TM), tiles_n = (int)((a.N + TN - 1) / TN);
    const int per_xcd = (tiles_m * tiles_n + 7) / 8;
    hipLaunchKernelGGL(fp4_gemm_tile_kernel<AF>, dim3((unsigned)(per_xcd * 8)), dim3(kTileThreads), Tile<AF>::kLds,
                       stream, a.a_codes, a.a_scales, a.b_codes, a.b_scales, (int)a.M, (int)a.N, (int)a.K,
                       tiles_m, tiles_n, static_cast<uint16_t *>(a.y), a.ld_y, a.acc_out);
    return hipGetLastError();
}

}  // namespace

hipError_t prepare_fp4_gemm_kernels()
{
    static OncePerDevice once;
    return once([] {
        const hipError_t err = allow_dynamic_lds(reinterpret_cast<const void *>(fp4_gemm_tile_kernel<4>), Tile<4>::kLds);
        return err != hipSuccess ? err
                                 : allow_dynamic_lds(reinterpret_cast<const void *>(fp4_gemm_tile_kernel<2>), Tile<2>::kLds);
    });
}

quest_plan plan_fp4_gemm(int64_t M, int64_t N, int64_t K)
{
    if (skinny_gemm_preferred(M, N, K, 0))
        return {QUEST_PLAN_FEW, 0, 0, 0};
    const auto tiles = [&](int rows) { return ((M + rows - 1) / rows) * ((N + TN - 1) / TN); };
    const int64_t large = tiles(Tile<4>::kRows);
    const bool one_large_each = large <= kUnits && tiles(Tile<2>::kRows) > kUnits && K >= kLongContraction;
    return {QUEST_PLAN_TILES, large < kFewTiles && !one_large_each ? Tile<2>::kRows : Tile<4>::kRows, TN, 0};
}

hipError_t launch_fp4_gemm(const Fp4GemmArgs &a, hipStream_t stream)
{
    if (a.M == 0 || a.N == 0)
        return hipSuccess;
    const quest_plan plan = plan_fp4_gemm(a.M, a.N, a.K);
    if (plan.kernel == QUEST_PLAN_FEW) {
        const SkinnyGemmArgs few = {a.a_codes, a.a_scales, a.b_codes, a.b_scales, a.M, a.N,
                                    a.K, 0, a.y, a.ld_y, a.acc_out};
        return launch_skinny_gemm(few, stream);
    }
    const hipError_t attr_err = prepare_fp4_gemm_kernels();
    if (attr_err != hipSuccess)
        return attr_err;
    return plan.block_rows == Tile<2>::kRows ? launch<2>(a, stream) : launch<4>(a, stream);
}

}  // namespace quest
