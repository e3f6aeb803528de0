// Host-side declarations shared by the QuEST translation units: one launcher per kernel family.
// Launchers assume validated arguments (the C-ABI entry points validate) and only enqueue work.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "../../include/quest.h"
#include "../../include/quest_plan.h"

namespace quest {

enum { kQuantRms = 0, kQuantAbsMax = 1, kQuantFp4 = 2 };

struct QuantizeArgs {
    const void *x;
    quest_dtype dtype;
    int64_t rows, cols, ld;
    int log2n;         // log2(had_block)
    int bits;          // b
    int cb;            // container bits
    float alpha;       // clip in RMS units
    float trust_edge;  // alpha * (1 + outer_trust / (L - 1)): trusted iff |x_h| <= trust_edge * rms
    uint8_t *codes;
    float *scales;
    uint8_t *mask;     // may be null
    float *xh_out;     // may be null
    int mode;          // kQuantRms: Eq. 1 grid, clip alpha * rms;  kQuantAbsMax: Eq. 1 grid, clip = largest
                       // |x_h| of the row (alpha, trust_edge unused);  kQuantFp4: E2M1 grid, clip alpha * rms
    // a second operand with the same dtype, cols, block, grid and clip, quantized by the same launch
    // (rows2 = 0: none); its mask is given exactly when `mask` is; it has no xh_out
    const void *x2 = nullptr;
    int64_t rows2 = 0, ld2 = 0;
    uint8_t *codes2 = nullptr;
    float *scales2 = nullptr;
    uint8_t *mask2 = nullptr;
};

hipError_t launch_hadamard_quantize(const QuantizeArgs &a, hipStream_t stream);
// Matrix-core kernel for the common bf16 / 4-bit shapes; false means "not covered, nothing launched".
bool launch_hadamard_quantize_mfma(const QuantizeArgs &a, hipStream_t stream, bool query = false);

// Matrix-core kernel for the other row lengths and blocks (run-time sizes): whether a call of `rows` rows goes there.
bool quantize_rows_preferred(const QuantizeArgs &a, int64_t rows);
hipError_t launch_hadamard_quantize_rows(const QuantizeArgs &a, hipStream_t stream);

struct GemmArgs {
    const uint8_t *a_codes;
    const float *a_scales;
    const uint8_t *b_codes;
    const float *b_scales;
    int64_t M, N, K;
    int bits, cb;
    void *y;          // bf16, may be null
    int64_t ld_y;
    int32_t *acc_out; // may be null
    void *workspace;  // caller's scratch for the re-coded operands of 1- and 2-bit products; may be null
    int64_t workspace_bytes;
};

hipError_t launch_lowbit_gemm(const GemmArgs &a, hipStream_t stream);
quest_plan plan_lowbit_gemm(int64_t M, int64_t N, int64_t K, int bits, bool with_workspace);
// Scratch the fast path of a 1- or 2-bit product needs (both operands re-coded as nibbles); 0 when the
// shape or the bit width does not take that path.
int64_t lowbit_gemm_workspace_bytes(int64_t M, int64_t N, int64_t K, int bits);

struct Fp4GemmArgs {
    const uint8_t *a_codes;
    const float *a_scales;
    const uint8_t *b_codes;
    const float *b_scales;
    int64_t M, N, K;
    void *y;          // bf16, may be null
    int64_t ld_y;
    float *acc_out;   // may be null
};

hipError_t launch_fp4_gemm(const Fp4GemmArgs &a, hipStream_t stream);
quest_plan plan_fp4_gemm(int64_t M, int64_t N, int64_t K);

// The forward product for few activation rows, on either grid.
struct SkinnyGemmArgs {
    const uint8_t *a_codes;
    const float *a_scales;
    const uint8_t *b_codes;
    const float *b_scales;
    int64_t M, N, K;
    int grid;         // 1 .. 4: bits of the Eq. 1 grid; 0: E2M1
    void *y;          // bf16, may be null
    int64_t ld_y;
    void *acc_out;    // int32 (E2M1: fp32), may be null
};

// grid as in SkinnyGemmArgs
bool skinny_gemm_preferred(int64_t M, int64_t N, int64_t K, int grid);
hipError_t launch_skinny_gemm(const SkinnyGemmArgs &a, hipStream_t stream);

struct BackwardArgs {
    const void *g;
    quest_dtype g_dtype;
    const uint8_t *mask;  // may be null
    int64_t rows, cols;
    int log2n;
    void *out;
    quest_dtype out_dtype;
    // second gradient of the same row length, dtypes and block, served by the same launch where the
    // matrix-core kernel covers the shape (rows2 = 0: none)
    const void *g2 = nullptr;
    const uint8_t *mask2 = nullptr;
    int64_t rows2 = 0;
    void *out2 = nullptr;
};

hipError_t launch_trust_backward(const BackwardArgs &a, hipStream_t stream);
// Matrix-core kernel for bf16 in / bf16 out and the common shapes; false means "not covered".
bool launch_trust_backward_mfma(const BackwardArgs &a, hipStream_t stream);

// Matrix-core kernel for the other row lengths and blocks (run-time sizes), bf16 in.
bool trust_backward_rows_covers(const BackwardArgs &a);
hipError_t launch_trust_backward_rows(const BackwardArgs &a, hipStream_t stream);

struct GradGemmArgs {
    int which;
    const void *dy;
    const uint8_t *q_codes;
    const float *q_scales;
    int bits, cb;
    bool fp4;          // the codes are E2M1 codes (bits = cb = 4)
    int64_t M, N, K;
    void *out;
    void *workspace;   // caller's scratch: the expanded operand, then the partial tiles
    int64_t workspace_bytes;
};

// The same products for outputs of few tiles (grad_gemm_mid.hip); needs no scratch.
struct GradMidArgs {
    int mode;            // as GradGemmArgs::which
    int grid;            // 1 .. 4: bits of the Eq. 1 grid; 0: E2M1
    const void *left;    // bf16: dy, or x for the weight-only product
    int64_t ld_left;
    const uint8_t *q_codes;
    int64_t q_row_bytes;
    const float *q_scales;
    int64_t C, R, K;     // contraction length, output rows and columns
    void *out;
};

// every shape of multiples of 64; E2M1 codes for modes 0 and 1 only
hipError_t launch_grad_gemm_mid(const GradMidArgs &a, hipStream_t stream);
// the block of the kernel the call gets (kernel, block_rows, block_cols, count)
quest_plan grad_gemm_mid_plan(int grid, int64_t C, int64_t R, int64_t K, int cus);
// what the call is expected to take, us
double grad_gemm_mid_cost(int grid, int64_t C, int64_t R, int64_t K, int cus);

// hipErrorInvalidValue: the shape is not one the kernels cover, or the workspace is too small
// (the entry points check both beforehand with grad_gemm_workspace_bytes).
hipError_t launch_grad_gemm(const GradGemmArgs &a, hipStream_t stream);
// Scratch bytes a call with these arguments needs on a device with `cus` compute units (0 for the
// small-shape kernel, which dequantizes in place); -1 when no kernel covers the shape.
int64_t grad_gemm_workspace_bytes(int which, bool fp4, int64_t M, int64_t N, int64_t K, int cus);

// Compute units of the current device, rounded down to a multiple of eight (one per XCD); 256, the
// MI355X's count, when no device can be asked (host-only use of the size queries).
int device_compute_units();

// Each family's kernels get their dynamic LDS limits on the current device, and the code objects of
// the files without such kernels are loaded (what quest_init does, so that no enqueue call has to
// change a kernel attribute or load code later).
hipError_t prepare_quantize_kernels();
hipError_t prepare_quantize_mfma_kernels();
hipError_t prepare_quantize_rows_kernels();
hipError_t prepare_trust_backward_rows_kernels();
hipError_t prepare_trust_backward_mfma_kernels();
hipError_t prepare_lowbit_gemm_kernels();
hipError_t prepare_skinny_gemm_kernels();
hipError_t prepare_fp4_gemm_kernels();
hipError_t prepare_trust_backward_kernels();
hipError_t prepare_grad_gemm_kernels();
hipError_t prepare_grad_gemm_mid_kernels();

// Runs a set-up step until it has succeeded once on the current device; afterwards the cost is the question
// which device that is (a call's path through the locks and look-ups of six limits was 0.5 us).  Safe
// from several threads: a step may run more than once, they are all idempotent.
class OncePerDevice {
public:
    template <typename Step>
    hipError_t operator()(Step &&step)
    {
        int device = 0;
        hipError_t err = hipGetDevice(&device);
        if (err != hipSuccess)
            return err;
        const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;
        if (done_.load(std::memory_order_acquire) & bit)
            return hipSuccess;
        err = step();
        if (err == hipSuccess)
            done_.fetch_or(bit, std::memory_order_release);
        return err;
    }

private:
    std::atomic<uint64_t> done_{0};
};

// Raise the dynamic LDS limit of `kernel` to `bytes` on the current device.  The attribute is set
// once per (kernel, device, size) and remembered; safe to call from several host threads.
hipError_t allow_dynamic_lds(const void *kernel, int bytes);

}  // namespace quest
