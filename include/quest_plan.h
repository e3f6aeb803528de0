/*
 * quest_plan.h - which kernel an entry point of quest.h runs for a shape, without running it.  Host functions for
 * tests (that they reach the kernel they are about) and profiles (which name to look for); not part of the
 * operations' interface: the answers change with the library's dispatch rules.
 */
#ifndef QUEST_PLAN_H
#define QUEST_PLAN_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

typedef enum {
    QUEST_PLAN_NONE = -1,      /* the shape is not covered */
    QUEST_PLAN_GENERAL = 0,    /* hq_generic_kernel, lowbit_gemm_kernel */
    QUEST_PLAN_INSTANCE = 1,   /* quantizer: hq_mfma_kernel */
    QUEST_PLAN_ROWS = 2,       /* quantizer: hq_rows_kernel */
    QUEST_PLAN_FEW = 3,        /* forward product: skinny_gemm_kernel */
    QUEST_PLAN_TILES = 4,      /* products: tile kernels (whole tiles) */
    QUEST_PLAN_SPLIT = 5,      /* 16-bit products: tiles split over the compute units, then the fix-up kernel */
    QUEST_PLAN_MID = 6         /* 16-bit products: grad_gemm_mid_kernel */
} quest_plan_kernel;

typedef struct {
    int32_t kernel;            /* quest_plan_kernel */
    int32_t block_rows;        /* of a workgroup's output block, 0 where that says nothing */
    int32_t block_cols;
    int32_t count;             /* TILES (16-bit products): tiles per workgroup; MID: groups of waves; forward: re-coding launches */
} quest_plan;

/* form 0, 1: quest_grad_gemm (bits 1 .. 4) or quest_grad_gemm_fp4 (bits = 0), 2: quest_weight_only_gemm; on a device of `cus`
 * compute units */
quest_plan quest_plan_grad_gemm(int32_t form, int32_t bits, int64_t M, int64_t N, int64_t K, int32_t cus);

/* Of a launch with several whole tiles per workgroup: from how many tiles its ring of stages runs on to the workgroup's next
 * one, after how many it begins anew (the next one ends at another edge of the output), and workgroups that do both */
typedef struct {
    int32_t on, anew, mixed;
} quest_plan_ring;
quest_plan_ring quest_plan_grad_gemm_ring(int32_t form, int32_t bits, int64_t M, int64_t N, int64_t K, int32_t cus);

/* quest_lowbit_gemm (bits 1 .. 4; with_workspace: scratch given) and quest_lowbit_gemm_fp4 (bits = 0) */
quest_plan quest_plan_forward(int32_t bits, int64_t M, int64_t N, int64_t K, int32_t with_workspace);

/* The block of a product that FEW takes: of the output, units of 128 contraction elements that a wave has in flight, waves */
typedef struct {
    int32_t block_rows, block_cols, in_flight, waves;
} quest_plan_few;
quest_plan_few quest_plan_forward_few(int32_t bits, int64_t M, int64_t N, int64_t K);

/* quest_hadamard_quantize (mode 0), _absmax (1) and _fp4 (2); rows: of both operands; f32: fp32 rows */
quest_plan quest_plan_quantize(int32_t mode, int32_t f32, int64_t rows, int64_t cols, int32_t had_block, int32_t bits);

#ifdef __cplusplus
}
#endif
#endif /* QUEST_PLAN_H */
