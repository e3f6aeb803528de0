// The two 16-bit gradient matmuls of Algorithm 2 (arXiv 2502.05003, Sec. 3.3): the upstream
// gradient dy against a code-packed operand whose value is bf16(s * u), contracted on the bf16
// matrix cores with fp32 accumulation.
//   which = 0:  out[M, K] = dy[M, N]   * what_h[N, K]   (contraction over N)
//   which = 1:  out[N, K] = dy[M, N]^T * xhat_h[M, K]   (contraction over M)
// and, with the same machinery, the weight-only forward product (Sec. 4.4):
//   which = 2:  out[M, N] = x[M, K]    * what_h[N, K]^T (contraction over K)
// This file: outputs of many tiles, and the choice between its kernels and those of grad_gemm_mid.hip.
#include <algorithm>
#include <numeric>
#include <utility>

#include "gemm_tile.h"
#include "quest_internal.h"

namespace quest {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------------
// Main path.  The code-packed operand is first expanded once to bf16(s u), [C, K] row-major, in
// the caller's workspace (every 256 x 256 output tile would otherwise repeat that work for the
// whole contraction); the matmul itself is then a plain bf16 x bf16 contraction whose main loop
// holds nothing but matrix instructions, LDS reads and global -> LDS transfers.
//
// 256 x 256 outputs per workgroup, four waves of 128 x 128 (sixteen 32 x 32 fp32 accumulator
// tiles, one wave per SIMD), 32 contraction elements per step, a ring of LDS stages of 32 KiB that
// the transfers fill several steps ahead of the step being multiplied.  An operand whose rows are
// contraction rows in memory ([c][k]: the expanded operand, and dy for which = 1) is staged as it
// is and read with the transposing LDS load, which hands each lane four contraction elements of
// one column; an operand whose rows are output rows (dy for which = 0) is read with 128-bit loads.
//
// The same with tiles of 192, 128 and 64 rows (TI = 3, 2, 1) for outputs whose tiles of 256 would leave compute
// units idle or need splitting: one and the same loop, fewer accumulators.  A step costs 0.78, 0.59, 0.41,
// 0.28 us with the chip full, so the smaller tiles give away 1, 5 and 40 % per operation.  Whole or split tiles of
// 256 only, and with the smaller ones (us per call, the expansion included; tokens x N x K):
//   G_w 16384 x 5632 x 2048: 341 (split) -> 318 (30 x 8 tiles of 192)    G_x 4096 x 6912 x 2560: 168 (split) -> 138 (192)
//   G_x 4096 x 5632 x 2048: 110 (split) -> 91 (128)                      weight-only 4096 x 5632 x 2048: 135 -> 107 (192)
//   G_w 4096 x 6912 x 2560: 181 (split) -> 153 (192)                     G_x 1088 x 4096 x 3648: 91 -> 55 (64)
// ------------------------------------------------------------------------------------------

constexpr int GT = 256;                        // tile columns, and rows of the largest tile
constexpr int GC = 32;                         // contraction elements per step
constexpr int kGemmThreads = 256;
constexpr int kRightBytes = GT * GC * 2;       // right operand of one step

// TI: accumulator tiles of a wave along the rows: tiles of 64 TI rows
template <int TI>
struct TileSizes {
    static constexpr int kRows = 64 * TI;
    static constexpr int kLeftBytes = kRows * GC * 2;
    static constexpr int kStage = kLeftBytes + kRightBytes;   // left operand, then right operand
    static constexpr int kStages = 160 * 1024 / kStage;       // ring of stages: 5 (TI = 4, 3), 6, 8
    static constexpr int kLds = kStages * kStage;
    static constexpr int kParkBytes = 32 * 128;               // epilogue: a wave's 32 rows by 64 columns
    static_assert(4 * kParkBytes <= kStage && kLds <= 160 * 1024, "the epilogue parks in the stage that was read last");
};

typedef __bf16 v4bf __attribute__((ext_vector_type(4)));

// One LDS read of the main loop: operand, fragment, and which half of the fragment's eight
// contraction elements a transposing read fetches (-1: a 128-bit read of the row form, both halves).
struct ReadOp {
    bool left;
    int idx, half;
};
// The reads of one k-step in the order the matrix instructions want them: right fragment j feeds
// instructions j, 4 + j, .., left fragment i instructions 4 i .. 4 i + 3.
template <int MODE, int TI>
struct ReadOrder {
    static constexpr bool kLeftHalves = MODE == 1, kRightHalves = MODE != 2;   // transposing reads come in halves
    static constexpr int kCount = TI * (kLeftHalves ? 2 : 1) + 4 * (kRightHalves ? 2 : 1);
    ReadOp op[kCount];
    constexpr ReadOrder() : op{}
    {
        int n = 0;
        for (int f = 0; f < TI + 4; ++f) {   // R0 L0 R1 R2 R3 L1 ..
            const bool left = f == 1 || f > 4;
            const int idx = left ? (f == 1 ? 0 : f - 4) : (f == 0 ? 0 : f - 1);
            if (left ? kLeftHalves : kRightHalves) {
                op[n++] = {left, idx, 0};
                op[n++] = {left, idx, 1};
            } else {
                op[n++] = {left, idx, -1};
            }
        }
    }
};

// Expands packed codes to bf16(fp32(s * u)), u = 2 c - (L - 1): eight elements per thread.
__global__ __launch_bounds__(256) void expand_codes_kernel(const uint8_t *__restrict__ codes,
                                                           const float *__restrict__ scales, int levels,
                                                           int cb, int K, int64_t groups,
                                                           uint16_t *__restrict__ qhat)
{
    // a workgroup takes 1024 consecutive groups of eight elements, a thread four of them, 256 apart:
    // every load instruction of a wave reads 256 contiguous bytes of codes (at 4 bits), every store
    // writes 1 KiB, and a thread has four independent chains in flight
    const int per_row = K / 8;
    const float offset = -(float)(levels - 1);
    const uint32_t field = (1u << cb) - 1u;
#pragma unroll
    for (int part = 0; part < 4; ++part) {
    const int64_t g = (int64_t)blockIdx.x * 1024 + part * 256 + threadIdx.x;   // group of eight elements
    if (g >= groups)
        continue;
    const int64_t row = g / per_row;
    const uint8_t *src = codes + g * cb;
    uint32_t bits = 0;
    if (cb == 4) {
        bits = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(src));
    } else {
        for (int byte = 0; byte < cb; ++byte)
            bits |= (uint32_t)src[byte] << (8 * byte);
    }
    const float s = scales[row];
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const uint32_t c = (bits >> (e * cb)) & field;
        v[e] = __fmul_rn(s, __fmaf_rn((float)c, 2.0f, offset));
    }
    *reinterpret_cast<uint4 *>(qhat + g * 8) = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]),
                                                          pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
    }
}

// The same for E2M1 codes, u then being the signed E2M1 value of the code (Sec. 4.4): converted in pairs by the
// hardware, a 32-bit division for the row, two groups per thread.  With the value computed from the
// code's bits in the kernel above (us): 5632 x 2048 12.3, now 8.0; 4096 x 2048 9.9, now 7.1.  (The integer codes stay
// above: this form was 5 to 10 % faster for them up to 7 MB of codes and 15 % slower at 16384 x 5632.)
__global__ __launch_bounds__(256) void expand_fp4_codes_kernel(const uint8_t *__restrict__ codes,
                                                               const float *__restrict__ scales, uint32_t per_row,
                                                               uint32_t groups, uint16_t *__restrict__ qhat)
{
    typedef float v2f __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        const uint32_t g = blockIdx.x * 512u + part * 256u + threadIdx.x;   // group of eight elements
        if (g >= groups)
            continue;
        const uint32_t bits = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(codes) + g);
        const float s = scales[g / per_row];
        uint32_t out[4];
        static_for<4>([&](auto pair) {
            const v2f u = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(bits, 1.0f, decltype(pair)::value);
            out[decltype(pair)::value] = pack_bf16(__fmul_rn(s, u[0]), __fmul_rn(s, u[1]));
        });
        *reinterpret_cast<uint4 *>(qhat + (size_t)g * 8) = make_uint4(out[0], out[1], out[2], out[3]);
    }
}

// Work is counted in (tile, step) units: tile t owns the units [t * steps, (t + 1) * steps) and
// workgroup b (in XCD-major order) the units [b * per_block, (b + 1) * per_block).  With
// per_block = steps every workgroup computes one whole tile.  When the tiles do not fill the CUs
// evenly the launcher hands every CU the same number of units instead; a workgroup then computes
// one segment per tile its range touches, and a segment that is not a whole tile leaves its fp32
// accumulators in partial-tile slot 2 b (segment continues a tile) or 2 b + 1 (segment starts one)
// of the workspace for grad_gemm_fixup_kernel to add up.  A slot is [wave][accumulator quad 0..63][lane] float4.
//
// Workgroups that are phase_period apart in that order walk through their tiles at the same
// contraction position all the time, and with the tiles numbered along the longer side of the tile
// grid (a run of neighbours shares one operand panel, and the longer the run, the more often two
// such workgroups fall into the same one) they tend to work on tiles of one tile-row or
// tile-column, that is on the same operand rows at the same moment.  Such
// workgroups are placed on one XCD (hardware deals workgroup ids out to the eight XCDs in turn) so
// that they share the fetch through that XCD's L2.  phase_period = 0: whole tiles, all in phase.
constexpr int kSlotQuads = 4 * 64 * 64;   // float4 per partial tile (256 KiB)

__host__ __device__ __forceinline__ void tile_origin(int tile, int tile_rows, int tiles_r, int tiles_k, int phase_period,
                                                     int &r0, int &k0)
{
    if (phase_period != 0) {   // split tiles: plain order along the longer side of the tile grid
        if (tiles_k > tiles_r) {
            r0 = (tile / tiles_k) * tile_rows;
            k0 = (tile % tiles_k) * GT;
        } else {
            r0 = (tile % tiles_r) * tile_rows;
            k0 = (tile / tiles_r) * GT;
        }
        return;
    }
    // four tile-rows deep, column by column: neighbours in the order share operand rows in L2
    const int band = tile / (4 * tiles_k);
    const int band_rows = tiles_r - band * 4 < 4 ? tiles_r - band * 4 : 4;
    const int in_band = tile - band * 4 * tiles_k;
    r0 = (band * 4 + in_band % band_rows) * tile_rows;
    k0 = (in_band / band_rows) * GT;
}

// Whether two tiles of an R x K output are of one size: neither or both end at the same edge
__host__ __device__ __forceinline__ bool same_tile_size(int r0, int k0, int next_r0, int next_k0, int R, int K, int tile_rows)
{
    auto rest = [](int left, int whole) { return left < whole ? left : whole; };
    return rest(R - next_r0, tile_rows) == rest(R - r0, tile_rows) && rest(K - next_k0, GT) == rest(K - k0, GT);
}

/*
 * LDS layouts of one operand of one step (16 KiB), both free of bank conflicts for the reads below.
 *   row form  [256 rows][4 chunks of 8 contraction elements]: chunk c of row r sits at chunk
 *             c ^ ((r >> 2) & 3).  Lane l of a 128-bit fragment read takes row l % 32 and chunk
 *             2 ks + l / 32 of k-step ks.
 *   column form [32 contraction rows][32 chunks of 8 columns]: chunk c of contraction row q sits at
 *             chunk c ^ column_swz(q).  A transposing 64-bit read works on 16 lanes: lanes 4 a ..
 *             4 a + 3 point at contraction row a of a block of four, sixteen columns wide, and lane
 *             i receives column i of it (four contraction elements).  Two such reads give a lane
 *             its eight contraction elements of one matrix-instruction operand.
 * A transfer instruction moves 1 KiB (lane l to offset 16 l): sixteen rows of the row form, two
 * contraction rows of the column form; each lane fetches the chunk that belongs in its slot.
 */
/*
 * MODE 0: out[M, K] = dy[M, N] what[N, K]        left = dy rows (row form),     right = expanded [c][k]
 * MODE 1: out[N, K] = dy[M, N]^T xhat[M, K]      left = dy columns (column form), right = expanded [c][k]
 * MODE 2: out[M, N] = x[M, K] what[N, K]^T       left = x rows (row form),       right = expanded rows
 *         (row form: the weight-only forward product, contraction over the expanded matrix's columns)
 * `left` has row pitch ld_left elements, the expanded operand ld_right, `out` is [R, K] (K columns).
 * R and K need not be whole tiles: the transfers of an edge tile fetch the last rows or columns
 * that exist in place of those that do not (results of those positions are never stored).
 */
template <int EDGE>
__device__ __forceinline__ int column_swz(int crow)
{
    // rows of 512 or 256 bytes all start at the same bank: four contraction rows apart by 64 bytes; rows of
    // 384 or 128 bytes alternate between two starts 128 bytes apart: the second pair moves by 64
    static_assert(EDGE == 64 || EDGE == 128 || EDGE == 192 || EDGE == 256, "tile edge");
    return EDGE % 128 != 0 ? ((crow >> 1) & 1) << 2 : (crow & 3) << 2;
}

/*
 * RING: for workgroups that work through several whole tiles.  A tile's two ends, a prologue that waits for its first
 * transfers and an epilogue whose stores all workgroups issue at once, took 10 to 13 us with nothing to multiply meanwhile; with
 * RING the next tile's first steps are requested during the last ones of a tile, and its stores are waited for only when
 * the counter of vector-memory operations cannot tell them from transfers any more, in the next tile's third to fifth step
 * (kAhead of them are in flight) (us per call, alone, before / now: G_x 16384 x 5632 x 2048, 2 tiles of 256 rows each, 310 / 296,
 * 16384 x 2048 x 5632, 8 of 192 rows, 354 / 337, 16384 x 1024 x 4096 162 / 136; weight-only 16384 x 4096 x 1024 161 / 132).
 * Workgroups with a single tile run the loop without the two instructions per step that this costs.
 */
constexpr int kSpreadModes = 5;   // bit m: MODE m spreads its transfers over the whole step (measured, see below)

template <int MODE, int TI, bool RING>
__global__ __launch_bounds__(kGemmThreads, 1) void grad_gemm_tile_kernel(
    const uint16_t *__restrict__ dy, int64_t ld_dy, const uint16_t *__restrict__ qhat, int64_t ld_right,
    int C, int R, int K, int tiles_r, int tiles_k, int per_block, int phase_period, uint16_t *__restrict__ out,
    float4 *__restrict__ partial)
{
    constexpr bool TRANSPOSED = MODE == 1;   // left operand in column form
    constexpr bool RIGHT_ROWS = MODE == 2;   // right operand in row form
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    typedef TileSizes<TI> Sizes;
    constexpr int STAGES = Sizes::kStages, kGStage = Sizes::kStage, kLeftBytes = Sizes::kLeftBytes;
    constexpr int kTransfers = TI + 4;        // per wave and step
    constexpr int kHalf = 4 * TI;             // matrix instructions per k-step

    const int steps = C / GC;
    const int64_t total_units = (int64_t)tiles_r * tiles_k * steps;
    int block;
    if (phase_period != 0) {
        // XCD x holds the phase classes x c .. x c + c - 1 (c = phase_period / 8) of every period
        const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3, classes = phase_period >> 3;
        block = (idx / classes) * phase_period + xcd * classes + idx % classes;
    } else {
        block = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);   // one contiguous run per XCD
    }
    const int64_t unit_begin = (int64_t)block * per_block;
    if (unit_begin >= total_units)
        return;
    // wave-uniform, and 32-bit from here on: this workgroup's units, and where the first one is
    int units_left = __builtin_amdgcn_readfirstlane((int)min((int64_t)per_block, total_units - unit_begin));
    const int first_tile = __builtin_amdgcn_readfirstlane((int)(unit_begin / steps));
    const int first_step = __builtin_amdgcn_readfirstlane((int)(unit_begin - (int64_t)first_tile * steps));

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int wr = wave >> 1, wc = wave & 1;
    const int lm = lane & 31, lh = lane >> 5;
    const int l16 = lane & 15, lg = lane >> 4;
    const uint32_t smem_addr = lds_address(smem);

    // byte advance per step
    const int64_t left_step = TRANSPOSED ? (int64_t)GC * ld_dy * 2 : (int64_t)GC * 2;
    const int64_t right_step = RIGHT_ROWS ? (int64_t)GC * 2 : (int64_t)GC * ld_right * 2;

    // Fragment reads, byte offsets from the operand's place in a stage.
    //   row form, fragment i, k-step ks:      row_off[ks] + 2048 i
    //   column form, fragment j, k-step ks, half t:  col_off[j] + 512 (16 ks + 4 t)
    // (column form: lane group g = l / 16 covers columns 16 (g % 2) .. + 16 and contraction rows
    //  8 (g / 2) .. of the k-step; lane i of the group points at row i / 4, columns 4 (i % 4) ..)
    auto column_offsets = [&](auto edge, int w, auto &off) {   // wave w's fragments of 32 columns
        constexpr int kEdge = decltype(edge)::value, kFragments = kEdge / 64;
#pragma unroll
        for (int j = 0; j < kFragments; ++j) {
            const int crow = 8 * (lg >> 1) + (l16 >> 2);
            const int chunk = (4 * (kFragments * w + j) + 2 * (lg & 1) + ((l16 >> 1) & 1)) ^ column_swz<kEdge>(l16 >> 2);
            off[j] = (uint32_t)(crow * 2 * kEdge + chunk * 16 + 8 * (l16 & 1));
        }
    };
    auto row_offsets = [&](int first_row, auto &off) {
        const int x = (lm >> 2) & 3;
        off[0] = (uint32_t)((first_row + lm) * 64 + ((lh ^ x) << 4));
        off[1] = (uint32_t)((first_row + lm) * 64 + (((2 + lh) ^ x) << 4));
    };
    uint32_t left_off[4], right_off[4];
    if constexpr (RIGHT_ROWS)
        row_offsets(wc * 128, right_off);
    else
        column_offsets(std::integral_constant<int, GT>{}, wc, right_off);
    if constexpr (TRANSPOSED)
        column_offsets(std::integral_constant<int, 64 * TI>{}, wr, left_off);
    else
        row_offsets(wr * 32 * TI, left_off);

    // where a tile begins (wave-uniform)
    auto origin = [&](int tile, int &r0, int &k0) __attribute__((always_inline)) {
        int r, k;
        tile_origin(tile, Sizes::kRows, tiles_r, tiles_k, phase_period, r, k);
        r0 = __builtin_amdgcn_readfirstlane(r);
        k0 = __builtin_amdgcn_readfirstlane(k);
    };
    constexpr int kStores = 8 * TI;   // of a wave and a whole tile
    bool carried = false;             // the first steps of this tile were requested during the last ones of the tile before
    int storing = 0;                  // steps to come whose wait has a whole tile's stores behind it
    int cur_off = 0;                  // byte offset of the current stage
    int r0, k0;
    origin(first_tile, r0, k0);
    for (int tile = first_tile, s_begin = first_step; units_left > 0; ++tile, s_begin = 0) {
    const int s_end = min(steps, s_begin + units_left);
    units_left -= s_end - s_begin;
    // Transfers: piece q of an operand is the 1 KiB at offset (4 q + wave) KiB; lane l of it lands at 16 l.
    // Per-lane byte offsets from the operand's position of the step:
    //   row form:    row 16 (4 q + wave) + l / 4, chunk (l % 4) ^ ((l / 16) & 3)
    //   column form: the (64 (4 q + wave) + l)-th chunk of the step: contraction row and slot by the row length
    // with rows and columns beyond the output's edge replaced by the last ones inside it.
    uint32_t left_voff[TI], right_voff[4];
    {
        const int rows_left = R - r0, cols_left = K - k0;   // what exists of this tile: >= 64, multiples of 8
        const uint32_t row_form_chunk = (uint32_t)(((lane & 3) ^ ((lane >> 4) & 3)) << 4);
        auto column_form = [&](auto edge, int piece, int64_t ld, int exists) {
            constexpr int kEdge = decltype(edge)::value;
            const int at = 64 * piece + lane, crow = at / (kEdge / 8), slot = at % (kEdge / 8);
            const int column = (slot ^ column_swz<kEdge>(crow)) * 8;    // first of the chunk's eight columns
            return (uint32_t)crow * (uint32_t)ld * 2u + (uint32_t)min(column, exists - 8) * 2u;
        };
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int piece = 4 * q + wave, row = 16 * piece + (lane >> 2);
            right_voff[q] = RIGHT_ROWS ? (uint32_t)min(row, cols_left - 1) * (uint32_t)ld_right * 2u + row_form_chunk
                                       : column_form(std::integral_constant<int, GT>{}, piece, ld_right, cols_left);
            if (q < TI)
                left_voff[q] = TRANSPOSED ? column_form(std::integral_constant<int, 64 * TI>{}, piece, ld_dy, rows_left)
                                          : (uint32_t)min(row, rows_left - 1) * (uint32_t)ld_dy * 2u + row_form_chunk;
        }
    }
    // operand positions of contraction step 0 (wave-uniform)
    const char *left_base = reinterpret_cast<const char *>(TRANSPOSED ? dy + r0 : dy + (int64_t)r0 * ld_dy);
    const char *right_base = reinterpret_cast<const char *>(RIGHT_ROWS ? qhat + (int64_t)k0 * ld_right : qhat + k0);

    v16f acc[TI][4];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][j][r] = 0.0f;
    // TI + 4 transfers per wave fill the stage at LDS byte address `stage` with contraction step `step`
    auto transfer = [&](auto pc, uint32_t stage, int step) __attribute__((always_inline)) {
        constexpr int p = decltype(pc)::value;
        const int at = min(step, s_end - 1);   // past the end: a valid step again, never used
        if constexpr (p < TI)
            lds_dma16(left_base + at * left_step, left_voff[p], stage + (4 * p + wave_u) * 1024);
        else
            lds_dma16(right_base + at * right_step, right_voff[p - TI],
                      stage + kLeftBytes + (4 * (p - TI) + wave_u) * 1024);
    };

    // the same from operand positions that the caller keeps up to date
    // (`wave_stage`: LDS byte address of the stage plus 1024 * wave)
    auto transfer_from = [&](auto pc, uint32_t wave_stage, const char *left_at, const char *right_at) {
        constexpr int p = decltype(pc)::value;
        if constexpr (p < TI)
            lds_dma16_at<4096 * p>(left_at, left_voff[p], wave_stage);
        else
            lds_dma16_at<kLeftBytes + 4096 * (p - TI)>(right_at, right_voff[p - TI], wave_stage);
    };

    // fragments as halves of four contraction elements: [k-step][fragment][half]
    v4bf lf[2][TI][2], rf[2][4][2];
    // read number n of k-step ks out of `stage`, in the order the matrix instructions want them
    auto load_frag = [&](auto nc, const uint8_t *stage, auto ksc) {
        constexpr int ks = decltype(ksc)::value;
        constexpr ReadOp op = ReadOrder<MODE, TI>().op[decltype(nc)::value];
        if constexpr (op.half < 0) {
            const uint32_t off = (op.left ? left_off[ks] : kLeftBytes + right_off[ks]) + 2048 * op.idx;
            const v8bf v = *reinterpret_cast<const v8bf *>(stage + off);
            if constexpr (op.left) {
                lf[ks][op.idx][0] = __builtin_shufflevector(v, v, 0, 1, 2, 3);
                lf[ks][op.idx][1] = __builtin_shufflevector(v, v, 4, 5, 6, 7);
            } else {
                rf[ks][op.idx][0] = __builtin_shufflevector(v, v, 0, 1, 2, 3);
                rf[ks][op.idx][1] = __builtin_shufflevector(v, v, 4, 5, 6, 7);
            }
        } else {
            const uint32_t off = (op.left ? left_off[op.idx] : kLeftBytes + right_off[op.idx]) +
                                 2 * (op.left ? Sizes::kRows : GT) * (16 * ks + 4 * op.half);
            const v4bf v = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                (__attribute__((address_space(3))) v4bf *)(stage + off));
            if constexpr (op.left)
                lf[ks][op.idx][op.half] = v;
            else
                rf[ks][op.idx][op.half] = v;
        }
    };
    constexpr int kReads = ReadOrder<MODE, TI>::kCount;
    // read numbers [reads_before(k), reads_before(k + 1)) of a k-step go behind its k-th matrix instruction
    auto reads_before = [](int k) constexpr { return kReads <= kHalf ? (k < kReads ? k : kReads) : k * kReads / kHalf; };

    // Ring of STAGES stages: while step s is multiplied out of stage s % STAGES, the transfers of the
    // next steps are in flight or done.  Two ways to refill:
    //   late   the transfers of step s + STAGES - 1 go into the stage that step s - 1 has left, which is
    //          free once every wave has passed this step's barrier: second half of the step only;
    //   spread the transfers of step s + STAGES - 2 go into the stage that step s - 2 has left, free
    //          since the previous step's barrier: one transfer every fourth matrix instruction, all
    //          through the step, at the price of one step less of look-ahead.
    // Spreading is 1-3 % faster when the left operand is in row form (G_x: 320 instead of 328 us on
    // one box, 334 instead of 338 on another) and 0-1 % slower when both operands are in column form.
    constexpr bool kSpread = kSpreadModes & (1 << MODE);
    constexpr int kAhead = kSpread ? STAGES - 2 : STAGES - 1;   // steps in flight beyond the current one
    // the matrix instruction behind which transfer p is issued
    auto transfer_slot = [](int p) constexpr {
        return kSpread ? p * 2 * kHalf / kTransfers : kHalf + p * kHalf / kTransfers;
    };
    constexpr int kIssuedAtWait = kSpread ? (kTransfers + 1) / 2 : 0;   // transfers of this step before its wait
    static_assert(transfer_slot(kIssuedAtWait) >= kHalf && (kIssuedAtWait == 0 || transfer_slot(kIssuedAtWait - 1) < kHalf),
                  "the wait counts the transfers issued before it");
    if (!carried) {
        static_for<kAhead>([&](auto sc) {
            static_for<kTransfers>([&](auto pc) {
                transfer(pc, smem_addr + decltype(sc)::value * kGStage, s_begin + decltype(sc)::value);
            });
        });
        wait_vmcnt<kTransfers * (kAhead - 1)>();
        __builtin_amdgcn_s_barrier();
        cur_off = 0;
        static_for<kReads>([&](auto nc) { load_frag(nc, smem, std::integral_constant<int, 0>{}); });
    }
    // The ring runs on from tile to tile where the next one's transfers differ in their base addresses alone.
    // Else, and after the last tile, the look-ahead fetches the last step again.  (With 256 compute units no plan comes near
    // the fewest steps: such contractions go to the kernels of grad_gemm_mid.hip.)
    int next_r0 = 0, next_k0 = 0;
    bool carry = false;
    if (units_left > 0) {
        origin(tile + 1, next_r0, next_k0);
        carry = RING && s_end - s_begin >= 2 * kAhead && same_tile_size(r0, k0, next_r0, next_k0, R, K, Sizes::kRows);
    }

    // Scalar bookkeeping of a step is kept to additions and selects (one wave per SIMD: a chain of
    // dependent scalar instructions between two matrix instructions is time the matrix pipe idles):
    // byte offsets of the current stage and of the stage being refilled, and the operands' positions
    // at the step being fetched, min(step + kAhead, s_end - 1).
    constexpr int kRing = STAGES * kGStage;
    static_assert(kTransfers * (kAhead - 2) + kIssuedAtWait + kStores <= 63, "the six-bit counter tells them apart");
    int refill_off = cur_off + (kSpread ? kAhead : STAGES - 1) * kGStage;
    refill_off = refill_off >= kRing ? refill_off - kRing : refill_off;
    const char *left_fetch = left_base + (int64_t)min(s_begin + kAhead, s_end - 1) * left_step;
    const char *right_fetch = right_base + (int64_t)min(s_begin + kAhead, s_end - 1) * right_step;
    // RING: the steps in three runs, which differ in the wait and in what is fetched: the ones whose wait has stores behind it,
    // the ones up to the last that fetches from this tile, the ones that fetch the next tile's first.
    const int tail = carry ? kAhead : 0, head = min(storing, s_end - s_begin - tail);
    for (int run = RING ? 0 : 1, step = s_begin; run < (RING ? 3 : 2); ++run) {
    const int run_end = !RING ? s_end : run == 0 ? s_begin + head : run == 1 ? s_end - tail : s_end;
    if (RING && run == 2 && tail > 0) {
        left_fetch = reinterpret_cast<const char *>(TRANSPOSED ? dy + next_r0 : dy + (int64_t)next_r0 * ld_dy);
        right_fetch = reinterpret_cast<const char *>(RIGHT_ROWS ? qhat + (int64_t)next_k0 * ld_right : qhat + next_k0);
    }
    // (steps to go that advance the operands' positions)
    const int last_advance = RING && run == 2 ? s_end : s_end - 1 - kAhead;
    for (; step < run_end; ++step) {
        const uint8_t *cur_stage = smem + cur_off;
        const int nxt_off = cur_off + kGStage == kRing ? 0 : cur_off + kGStage;
        const uint8_t *nxt_stage = smem + nxt_off;
        const uint32_t refill = smem_addr + refill_off + wave_u * 1024;
        // 8 TI matrix instructions; each is followed by one slice of the other work, pinned in place
        // (figures for TI = 4):
        //    0..15  fragment reads of the step's second k-step
        //   15      transfers of step + 1 have landed (all but the newer groups), barrier
        //   16..31  fragment reads of the next step's first k-step
        //   16, 18, .. 30 (late) or 0, 4, .. 28 (spread)  transfers of a later step (never back to back:
        //           a wave issues in order, and a transfer that finds the memory pipeline's queue full
        //           holds up the MFMAs behind it)
        static_for<2 * kHalf>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            constexpr int ks = k / kHalf, i = (k % kHalf) >> 2, j = k & 3;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_shufflevector(rf[ks][j][0], rf[ks][j][1], 0, 1, 2, 3, 4, 5, 6, 7),
                __builtin_shufflevector(lf[ks][i][0], lf[ks][i][1], 0, 1, 2, 3, 4, 5, 6, 7), acc[i][j], 0, 0, 0);
            static_for<kTransfers>([&](auto pc) {
                if constexpr (kSpread && transfer_slot(decltype(pc)::value) == k)
                    transfer_from(pc, refill, left_fetch, right_fetch);
            });
            constexpr int first = reads_before(k % kHalf), count = reads_before(k % kHalf + 1) - first;
            static_for<count>([&](auto nc) {
                load_frag(std::integral_constant<int, first + decltype(nc)::value>{}, ks == 0 ? cur_stage : nxt_stage,
                          std::integral_constant<int, 1 - ks>{});
            });
            if constexpr (k == kHalf - 1) {
                // all transfers of step + 1 have landed: what may still be in flight are the groups of
                // the steps after it and, when spread, the transfers this step has issued so far
                constexpr int kNewer = kTransfers * (kAhead - 2) + kIssuedAtWait;
                if constexpr (RING)
                    wait_vmcnt_either<kNewer + kStores, kNewer>(run);
                else
                    wait_vmcnt<kNewer>();
                __builtin_amdgcn_s_barrier();
            }
            static_for<kTransfers>([&](auto pc) {
                if constexpr (!kSpread && transfer_slot(decltype(pc)::value) == k)
                    transfer_from(pc, refill, left_fetch, right_fetch);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        cur_off = nxt_off;
        refill_off = refill_off + kGStage == kRing ? 0 : refill_off + kGStage;
        if (step < last_advance) {
            left_fetch += left_step;
            right_fetch += right_step;
        }
    }
    }
    if (!carry)
        wait_vmcnt<0>();   // the look-ahead transfers still write into the stages

    // Epilogue.  A segment that is not a whole tile leaves its accumulators as they are, in fp32.
    const int block_row = r0 + (wave_u >> 1) * 32 * TI, block_col = k0 + (wave_u & 1) * 128;
    storing = 0;
    carried = carry;
    r0 = next_r0;
    k0 = next_k0;
    __syncthreads();
    if (TI == 4 && !RING && s_end - s_begin != steps) {   // (only tiles of 256 rows are ever split, and not with RING)
        float4 *slot = partial + ((int64_t)(2 * block + (s_begin == 0 ? 1 : 0)) * 4 + wave) * (64 * 64) + lane;
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                asm volatile("" : "+a"(acc[i][j]));   // as below
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    __builtin_nontemporal_store(
                        v4f{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]},
                        reinterpret_cast<v4f *>(slot + ((i * 4 + j) * 4 + q) * 64));
            }
        continue;   // LDS untouched since the barrier
    }
    // Each accumulator tile is a transposed output tile: lane l holds output row l % 32
    // and, in register r, output column 8 (r / 4) + 4 (l / 32) + r % 4.  A wave parks its block as bf16 in
    // pieces of 32 rows by 64 columns (chunks swizzled by row) and writes them out as 128-byte row segments.  It parks
    // in the stage that was read last, which every wave has left and which the next step does not refill (spread) or
    // only behind its barrier (late).
    uint8_t *const park = smem + (cur_off == 0 ? kRing : cur_off) - kGStage + wave * Sizes::kParkBytes;
    const uint32_t lane_offset = (uint32_t)(lane >> 3) * (uint32_t)K * 2u + 16u * (lane & 7);
    v4u out_reg[2][4];
    auto store_piece = [&](auto pc) __attribute__((always_inline)) {   // (rows and columns come in multiples of 64)
        constexpr int piece = decltype(pc)::value, i = piece / 2, half = piece % 2;
        if (block_row + 32 * i < R && block_col + 64 * half < K) {
            uint16_t *at = out + (int64_t)(block_row + 32 * i) * K + block_col + 64 * half;
#pragma unroll
            for (int pass = 0; pass < 4; ++pass)
                store_16_counted(at + (int64_t)(8 * pass) * K, lane_offset, out_reg[piece & 1][pass]);
        }
    };
    static_for<2 * TI>([&](auto pc) {
        constexpr int piece = decltype(pc)::value, i = piece / 2, half = piece % 2;
        // (in accumulation registers until then: brought over all at once they would need as many others)
        asm volatile("" : "+a"(acc[i][2 * half]), "+a"(acc[i][2 * half + 1]));
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v16f &a = acc[i][2 * half + j];
                *reinterpret_cast<uint2 *>(park + lm * 128 + (((4 * j + q) ^ (lm & 7)) << 4) + 8 * lh) =
                    make_uint2(pack_bf16(a[4 * q + 0], a[4 * q + 1]), pack_bf16(a[4 * q + 2], a[4 * q + 3]));
            }
#pragma unroll
        for (int pass = 0; pass < 4; ++pass) {
            const int row = 8 * pass + (lane >> 3), c = lane & 7;
            out_reg[piece & 1][pass] = *reinterpret_cast<const v4u *>(park + row * 128 + ((c ^ (row & 7)) << 4));
        }
        if constexpr (piece > 0)
            store_piece(std::integral_constant<int, piece - 1>{});
        __builtin_amdgcn_sched_barrier(0);
    });
    store_piece(std::integral_constant<int, 2 * TI - 1>{});
    if (!carry)
        __syncthreads();   // the next tile's first stages may be where a block is parked
    else if (block_row + 32 * TI <= R && block_col + 128 <= K)   // (fewer stores at the output's edge: waited for)
        storing = kAhead - 1;
    }
}

/*
 * Adds up the partial tiles of every tile that more than one workgroup worked on (in workgroup
 * order, so the sum does not depend on timing) and writes the bf16 result.  One wave per 32 x 32
 * accumulator tile: quadrant = the 128 x 128 block of one wave of the main kernel, (i, j) = the
 * accumulator tile in it, j = the wave of a workgroup.  (Sixty-four waves per output tile, and
 * several partial tiles in flight per lane: a small output split over many CUs has few tiles and
 * many partial tiles each, and the sum is a chain of loads.)
 */
__global__ __launch_bounds__(256) void grad_gemm_fixup_kernel(const float4 *__restrict__ partial, int steps,
                                                             int per_block, int phase_period, int R, int K,
                                                             int tiles_r, int tiles_k,
                                                             uint16_t *__restrict__ out)
{
    __shared__ __attribute__((aligned(16))) uint8_t park_all[4 * 2048];
    const int tile = blockIdx.x >> 4, quadrant = (blockIdx.x >> 2) & 3, i = blockIdx.x & 3, j = threadIdx.x >> 6;
    uint8_t *park = park_all + j * 2048;
    const int64_t first_unit = (int64_t)tile * steps, last_unit = first_unit + steps - 1;
    const int b_first = (int)(first_unit / per_block), b_last = (int)(last_unit / per_block);
    if (b_first == b_last)
        return;   // computed whole by one workgroup, already written
    const int lane = threadIdx.x & 63;
    const int lm = lane & 31, lh = lane >> 5;
    float4 sum[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        sum[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll 4
    for (int b = b_first; b <= b_last; ++b) {
        const bool continues = (int64_t)b * per_block > first_unit;
        const float4 *slot = partial + ((int64_t)(2 * b + (continues ? 0 : 1)) * 4 + quadrant) * (64 * 64) + lane;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v = slot[((i * 4 + j) * 4 + q) * 64];
            sum[q].x += v.x; sum[q].y += v.y; sum[q].z += v.z; sum[q].w += v.w;
        }
    }
    // park the 32 x 32 tile as bf16 (row lm, 64 bytes), write 16-byte chunks: 4 per row, 2 passes
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int col = 8 * q + 4 * lh;
        *reinterpret_cast<uint2 *>(park + lm * 64 + col * 2) =
            make_uint2(pack_bf16(sum[q].x, sum[q].y), pack_bf16(sum[q].z, sum[q].w));
    }
    __syncthreads();
    int r0, k0;
    tile_origin(tile, GT, tiles_r, tiles_k, phase_period, r0, k0);
    const int row0 = r0 + (quadrant >> 1) * 128 + i * 32, col0 = k0 + (quadrant & 1) * 128 + j * 32;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const int prow = pass * 16 + (lane >> 2);
        const int c = lane & 3;
        const uint4 v = *reinterpret_cast<const uint4 *>(park + prow * 64 + c * 16);
        if (row0 + prow < R && col0 + c * 8 < K)
            *reinterpret_cast<uint4 *>(out + (int64_t)(row0 + prow) * K + col0 + c * 8) = v;
    }
}

}  // namespace

namespace {

// How a call is carried out: which kernels, how the tiles are dealt out, what scratch it needs.
struct GradGemmPlan {
    bool covered;      // some kernel handles the shape
    bool tile_path;    // a shape the 256 x 256 tile kernels can do (their scratch is asked for)
    bool mid;          // the kernels of grad_gemm_mid.hip do it (always when tile_path is not set)
    bool split;        // tiles split over the CUs, partial tiles summed by the fix-up kernel
    int ti;            // tiles of 64 ti rows
    int tiles_r, tiles_k, steps, blocks, per_block, phase_period;
    int64_t out_rows, out_cols, contraction, q_rows, ld_left;
    size_t expanded_bytes, partial_bytes;
};

// grid: 1 .. 4 bits of the Eq. 1 grid, 0 E2M1; what scratch the plan needs does not depend on it
GradGemmPlan plan_grad_gemm(int which, int grid, int64_t M, int64_t N, int64_t K, int cus)
{
    GradGemmPlan p = {};
    // which = 0: out[M, K] = dy what;  1: out[N, K] = dy^T xhat;  2: out[M, N] = x what^T (weight-only)
    p.out_rows = which == 1 ? N : M;
    p.out_cols = which == 2 ? N : K;
    p.contraction = which == 0 ? N : which == 1 ? M : K;
    p.q_rows = which == 1 ? M : N;          // rows of the code-packed operand [q_rows, K]
    p.ld_left = which == 2 ? K : N;
    // the tile kernels: edge tiles may be partial (every size is a multiple of 64), offsets are 32-bit
    p.tile_path = p.out_rows >= GT / 2 && p.out_cols >= GT / 2 && (p.contraction % GC) == 0 &&
                  p.out_rows * p.out_cols < ((int64_t)1 << 31) &&
                  std::max(M, N) * std::max(K, N) < ((int64_t)1 << 30);
    p.covered = p.tile_path || !(which == 2 || grid == 0);   // these two forms: outputs of 128 x 128 or more only
    p.mid = true;
    if (!p.tile_path)
        return p;
    p.tiles_k = (int)((p.out_cols + GT - 1) / GT);
    p.steps = (int)(p.contraction / GC);
    auto tiles_of = [&](int ti) { return (int)((p.out_rows + 64 * ti - 1) / (64 * ti)) * p.tiles_k; };
    // One workgroup per CU at a time.  Two ways to deal out the work: rounds of whole tiles of 256, 192, 128 or
    // 64 rows (whichever costs least), or, when rounds would leave too many CUs idle, every CU gets
    // the same share of (tile, step) units of the largest tiles and the split tiles are summed by a
    // second, small kernel.
    const int tiles = tiles_of(4);
    const int64_t units = (int64_t)tiles * p.steps;
    // What a step of 32 contraction elements takes, us, with a share `busy` of the CUs at work (the chip is
    // power-limited: the more of them, the slower each), and what a tile's two ends take.  The weight-only
    // form reads half lines of both operands, which the smaller tiles feel, and tiles of 64 and 128 rows in many
    // rounds share fewer fetches of the right operand.  Fitted to 260 products of 128 .. 16384 tokens, each
    // timed alone in every way there is, before workgroups' rings ran on from tile to tile, and checked since on 520
    // others: the way chosen takes 1.5 % more than the best in the mean, 18 % at most but for five (21 to 35 %).  Every tile's two ends
    // are priced in full, also where RING hides them, which makes several tiles of 256 rows look dearer than they are: G_x 16384 x
    // 2048 x 5632 takes 350 us in the tiles of 192 rows that are chosen and 337 in tiles of 256, 8192 x 1280 x 11008 251 and 229.
    // Inside a training step a product takes up to 15 % more than alone, 360 tiles of
    // 192 rows in two rounds (G_w 4096 x 6912 x 2560) 25 %.
    constexpr double kStepUs[5] = {0.0, 0.212, 0.265, 0.318, 0.488}, kBusyUs[5] = {0.0, 0.085, 0.17, 0.307, 0.339};
    constexpr double kEndsUs[5] = {0.0, 5.0, 7.0, 9.5, 13.5};
    auto whole_cost = [&](int ti) {
        const int n = tiles_of(ti), rounds = (n + cus - 1) / cus;
        const double busy = (double)n / ((double)rounds * cus);
        const double step = (kStepUs[ti] + kBusyUs[ti] * busy * busy) * (which == 2 && ti < 4 ? 1.18 : 1.0);
        return rounds * (step * p.steps + kEndsUs[ti]) * (ti <= 2 && rounds >= 3 ? 1.15 : 1.0);
    };
    // split: a share of the units, partial tiles written and read back (0.08 us each), the second launch;
    // a step costs more when no other workgroup of the XCD is at the same contraction position, which those are
    // whose period divides the number of workgroups (see phase_period)
    const int share = cus >= 8 ? (int)((units + cus - 1) / cus) : 0;
    const int period = cus >= 8 ? p.steps / std::gcd(share, p.steps) : 0;
    const bool in_phase = period != 0 && cus % period == 0 && period <= 32;
    const double split_cost = cus >= 8 && units >= 4 * (int64_t)cus
                                  ? (!in_phase ? 1.12 : which == 2 ? 0.78 : 0.80) * share + 0.08 * (cus + tiles) + 8.0
                                  : 1e30;
    p.ti = 4;
    double cost = cus > 0 ? whole_cost(4) : 0.0;
    for (int ti = 3; cus > 0 && ti >= 1; --ti)
        if (whole_cost(ti) < cost) {
            cost = whole_cost(ti);
            p.ti = ti;
        }
    p.split = split_cost < cost;
    if (p.split) {
        cost = split_cost;
        p.ti = 4;
    }
    p.tiles_r = (int)((p.out_rows + 64 * p.ti - 1) / (64 * p.ti));
    const int chosen = tiles_of(p.ti);
    p.blocks = (chosen + 7) / 8 * 8;
    p.per_block = p.steps;
    p.phase_period = 0;
    if (!p.split && cus >= 8 && chosen > cus) {
        // more whole tiles than compute units: one workgroup per unit walks over several tiles, so that
        // no tile after the first waits for a workgroup to be dispatched (7 us per tile here)
        const int rounds = (chosen + cus - 1) / cus;
        p.blocks = ((chosen + rounds - 1) / rounds + 7) / 8 * 8;   // the same number on every XCD
        p.per_block = rounds * p.steps;
    }
    if (p.split) {
        p.blocks = cus;
        p.per_block = share;
        // workgroups b and b + period are at the same contraction position at all times
        p.phase_period = (period % 8 == 0 && p.blocks % period == 0) ? period : 8;
        if (p.blocks % p.phase_period != 0)
            p.phase_period = p.blocks;
    }
    // Whether the kernels that expand on the way into LDS are cheaper: theirs is their own estimate; here
    // the expansion (read 0.5, written 2 bytes per code at 4.5 TB/s) and two or three launches come on top.
    const double expand_cost = 3.0 + (double)p.q_rows * (double)K * 2.5 / 4.5e6;
    p.mid = grad_gemm_mid_cost(grid, p.contraction, p.out_rows, p.out_cols, cus >= 8 ? cus : 256) < expand_cost + cost;
    p.expanded_bytes = ((size_t)p.q_rows * K * 2 + 255) / 256 * 256;
    p.partial_bytes = p.split ? (size_t)2 * p.blocks * kSlotQuads * sizeof(float4) : 0;
    return p;
}

}  // namespace

int64_t grad_gemm_workspace_bytes(int which, bool fp4, int64_t M, int64_t N, int64_t K, int cus)
{
    if (M == 0 || N == 0 || K == 0)
        return 0;
    const GradGemmPlan p = plan_grad_gemm(which, fp4 ? 0 : 4, M, N, K, cus);
    if (!p.covered)
        return -1;
    return p.tile_path ? (int64_t)(p.expanded_bytes + p.partial_bytes) : 0;
}

namespace {

template <int MODE, int TI>
hipError_t launch_tiles(const GradGemmPlan &p, const uint16_t *left, const uint16_t *qhat, int64_t ld_right, uint16_t *out,
                        float4 *partial, hipStream_t stream)
{
    auto kernel = grad_gemm_tile_kernel<MODE, TI, false>;
    if constexpr (TI > 1) {   // (tiles of 64 rows are taken where one each is plenty)
        if (!p.split && p.per_block > p.steps)
            kernel = grad_gemm_tile_kernel<MODE, TI, true>;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)p.blocks), dim3(kGemmThreads), TileSizes<TI>::kLds,
                       stream, left, p.ld_left, qhat, ld_right, (int)p.contraction, (int)p.out_rows, (int)p.out_cols,
                       p.tiles_r, p.tiles_k, p.per_block, p.phase_period, out, partial);
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_mode(const GradGemmPlan &p, const uint16_t *left, const uint16_t *qhat, int64_t ld_right, uint16_t *out,
                       float4 *partial, hipStream_t stream)
{
    return p.ti == 4   ? launch_tiles<MODE, 4>(p, left, qhat, ld_right, out, partial, stream)
           : p.ti == 3 ? launch_tiles<MODE, 3>(p, left, qhat, ld_right, out, partial, stream)
           : p.ti == 2 ? launch_tiles<MODE, 2>(p, left, qhat, ld_right, out, partial, stream)
                       : launch_tiles<MODE, 1>(p, left, qhat, ld_right, out, partial, stream);
}

template <int MODE, int TI>
hipError_t prepare_tiles()
{
    hipError_t err =
        allow_dynamic_lds(reinterpret_cast<const void *>(grad_gemm_tile_kernel<MODE, TI, false>), TileSizes<TI>::kLds);
    if constexpr (TI > 1) {
        if (err == hipSuccess)
            err = allow_dynamic_lds(reinterpret_cast<const void *>(grad_gemm_tile_kernel<MODE, TI, true>), TileSizes<TI>::kLds);
    }
    return err;
}

template <int MODE>
hipError_t prepare_mode()
{
    hipError_t err = prepare_tiles<MODE, 4>();
    if (err == hipSuccess)
        err = prepare_tiles<MODE, 3>();
    if (err == hipSuccess)
        err = prepare_tiles<MODE, 2>();
    if (err == hipSuccess)
        err = prepare_tiles<MODE, 1>();
    return err;
}

}  // namespace

hipError_t prepare_grad_gemm_kernels()
{
    static OncePerDevice once;
    return once([] {
        hipError_t err = prepare_mode<0>();
        if (err == hipSuccess)
            err = prepare_mode<1>();
        if (err == hipSuccess)
            err = prepare_mode<2>();
        return err;
    });
}

hipError_t launch_grad_gemm(const GradGemmArgs &a, hipStream_t stream)
{
    if (a.M == 0 || a.N == 0 || a.K == 0)
        return hipSuccess;
    const auto *dy = static_cast<const uint16_t *>(a.dy);
    auto *out = static_cast<uint16_t *>(a.out);
    const GradGemmPlan p = plan_grad_gemm(a.which, a.fp4 ? 0 : a.bits, a.M, a.N, a.K, device_compute_units());
    if (!p.covered)
        return hipErrorInvalidValue;
    if (p.mid) {
        const GradMidArgs mid = {a.which, a.fp4 ? 0 : a.bits, a.dy, p.ld_left, a.q_codes, a.K * a.cb / 8, a.q_scales,
                                 p.contraction, p.out_rows, p.out_cols, a.out};
        return launch_grad_gemm_mid(mid, stream);
    }
    if (a.workspace == nullptr || (size_t)a.workspace_bytes < p.expanded_bytes + p.partial_bytes)
        return hipErrorInvalidValue;
    hipError_t err = prepare_grad_gemm_kernels();
    if (err != hipSuccess)
        return err;
    // the caller's scratch: the expanded operand, then the partial tiles
    char *memory = static_cast<char *>(a.workspace);
    auto *qhat = reinterpret_cast<uint16_t *>(memory);
    auto *partial = p.split ? reinterpret_cast<float4 *>(memory + p.expanded_bytes) : nullptr;

    const int64_t groups = p.q_rows * a.K / 8;
    if (a.fp4)   // (the tile path's operands are below 2^30 elements: 32-bit group numbers)
        hipLaunchKernelGGL(expand_fp4_codes_kernel, dim3((unsigned)((groups + 511) / 512)), dim3(256), 0, stream,
                           a.q_codes, a.q_scales, (uint32_t)(a.K / 8), (uint32_t)groups, qhat);
    else
        hipLaunchKernelGGL(expand_codes_kernel, dim3((unsigned)((groups + 1023) / 1024)), dim3(256), 0, stream,
                           a.q_codes, a.q_scales, 1 << a.bits, a.cb, (int)a.K, groups, qhat);
    err = hipGetLastError();
    if (err != hipSuccess)
        return err;
    err = a.which == 0   ? launch_mode<0>(p, dy, qhat, a.K, out, partial, stream)
          : a.which == 1 ? launch_mode<1>(p, dy, qhat, a.K, out, partial, stream)
                         : launch_mode<2>(p, dy, qhat, a.K, out, partial, stream);
    if (err == hipSuccess && p.split) {
        hipLaunchKernelGGL(grad_gemm_fixup_kernel, dim3((unsigned)(p.tiles_r * p.tiles_k * 16)), dim3(256), 0, stream,
                           partial, p.steps, p.per_block, p.phase_period, (int)p.out_rows, (int)p.out_cols, p.tiles_r,
                           p.tiles_k, out);
        err = hipGetLastError();
    }
    return err;
}

}  // namespace quest

quest_plan quest_plan_grad_gemm(int32_t form, int32_t bits, int64_t M, int64_t N, int64_t K, int32_t cus)
{
    const quest::GradGemmPlan p = quest::plan_grad_gemm(form, bits, M, N, K, cus);
    if (!p.covered)
        return {QUEST_PLAN_NONE, 0, 0, 0};
    if (p.mid)
        return quest::grad_gemm_mid_plan(bits, p.contraction, p.out_rows, p.out_cols, cus);
    return {p.split ? QUEST_PLAN_SPLIT : QUEST_PLAN_TILES, 64 * p.ti, quest::GT, p.split ? 1 : p.per_block / p.steps};
}

quest_plan_ring quest_plan_grad_gemm_ring(int32_t form, int32_t bits, int64_t M, int64_t N, int64_t K, int32_t cus)
{
    const quest::GradGemmPlan p = quest::plan_grad_gemm(form, bits, M, N, K, cus);
    quest_plan_ring ring = {0, 0, 0};
    if (!p.covered || p.mid || p.split || p.ti == 1)
        return ring;
    const int tile_rows = 64 * p.ti, tiles = p.tiles_r * p.tiles_k, each = p.per_block / p.steps;
    for (int first = 0; first < tiles; first += each) {
        int on = 0, anew = 0, r0, k0, next_r0, next_k0;
        for (int tile = first; tile + 1 < std::min(first + each, tiles); ++tile) {
            quest::tile_origin(tile, tile_rows, p.tiles_r, p.tiles_k, 0, r0, k0);
            quest::tile_origin(tile + 1, tile_rows, p.tiles_r, p.tiles_k, 0, next_r0, next_k0);
            ++(quest::same_tile_size(r0, k0, next_r0, next_k0, (int)p.out_rows, (int)p.out_cols, tile_rows) ? on : anew);
        }
        ring.on += on;
        ring.anew += anew;
        ring.mixed += on > 0 && anew > 0;
    }
    return ring;
}
