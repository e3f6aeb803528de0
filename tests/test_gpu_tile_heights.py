"""The gradient and weight-only products at sizes where the dispatch takes tiles of 64, 128, 192 or 256 rows,
several tiles per workgroup and split tiles included (csrc/grad_gemm.hip): outputs ending inside a tile
both ways, sampled rows around the tile edges against the product of the same 16-bit operands in double.
(tests/test_plans.py holds the cases to the paths they are listed under.)"""
import numpy as np
import pytest
import torch

from oracle import quest_oracle as qo
from paper_2502_05003_amd import binding as q
from paper_2502_05003_amd import synth

import plan
from gpu_util import BF16_HALF_ULP, DEV, grad_ws, to_device, to_host_f64, weight_only_ws

pytestmark = pytest.mark.gpu

# kernel, rows of a tile, several tiles per workgroup?, then form, contraction, output rows, output columns
CASES = [(plan.TILES, 64, False, 0, 2048, 1600, 2496), (plan.TILES, 64, False, 1, 2816, 1600, 2496),
         (plan.TILES, 128, False, 0, 5632, 4032, 1984), (plan.TILES, 128, False, 0, 11008, 1088, 5568),
         (plan.TILES, 128, True, 0, 1536, 1088, 12224), (plan.TILES, 128, True, 1, 1536, 3200, 4928),
         (plan.TILES, 128, False, 2, 1024, 1472, 2880), (plan.TILES, 128, True, 2, 2816, 3200, 4928),
         (plan.TILES, 192, False, 1, 2048, 5568, 1984), (plan.TILES, 192, False, 2, 1024, 3392, 2368),
         (plan.TILES, 192, False, 0, 6912, 4032, 2496), (plan.TILES, 192, True, 1, 4096, 6848, 2496),
         (plan.TILES, 192, True, 2, 1024, 4160, 4928),
         (plan.TILES, 256, False, 1, 2048, 4032, 4032), (plan.TILES, 256, True, 0, 1024, 4544, 5440),
         (plan.TILES, 256, True, 1, 1024, 5312, 4672), (plan.TILES, 256, False, 2, 1024, 2240, 5440),
         (plan.TILES, 256, True, 2, 1024, 5696, 4416),
         # split: one tile row, one tile column, a grid of tiles
         (plan.SPLIT, 256, False, 0, 11008, 128, 640), (plan.SPLIT, 256, False, 0, 12288, 576, 128),
         (plan.SPLIT, 256, False, 1, 16384, 2048, 1216), (plan.SPLIT, 256, False, 1, 12288, 448, 832),
         (plan.SPLIT, 256, False, 2, 14336, 256, 1280), (plan.SPLIT, 256, False, 2, 10752, 1856, 4096)]


def layer(form, C, R, cols):
    """M, N, K of the call"""
    return ((R, C, cols), (C, R, cols), (R, cols, C))[form]


# E2M1 codes (their own expansion): each kind of tile once in both forms there are; 1 bit: where weight-only outputs take
# tiles of 64 rows
RUNS = [(*case, 4) for case in CASES] + [(*case, "fp4") for case in CASES if case[3] != 2 and case[4] * case[5] < 1 << 25] + \
       [(plan.TILES, 64, False, 2, 1088, 1600, 2496, 1), (plan.TILES, 64, False, 0, 576, 1600, 2496, 1)]


@pytest.mark.parametrize("kernel,tile_rows,several,form,C,R,cols,grid", RUNS)
def test_sampled_rows(kernel, tile_rows, several, form, C, R, cols, grid):
    rng = np.random.default_rng(C + R + cols + form)
    q_shape = (cols, C) if form == 2 else (C, cols)
    fp4, bits = grid == "fp4", 4 if grid == "fp4" else grid
    codes = rng.integers(0, 256, size=(q_shape[0], q_shape[1] * qo.container_bits(bits) // 8), dtype=np.uint8)
    scales = ((rng.random(q_shape[0]) + 0.5) * 0.01).astype(np.float32)
    left = synth.gaussian(*((C, R) if form == 1 else (R, C)), 0.03, 5, "bf16")
    out = torch.full((R, cols), float("nan"), dtype=torch.bfloat16, device=DEV)
    M, N, K = layer(form, C, R, cols)
    if form == 2:
        q.quest_weight_only_gemm(to_device(left), to_device(codes), to_device(scales), bits, y=out,
                                 workspace=weight_only_ws(M, N, K))
    elif fp4:
        q.quest_grad_gemm_fp4(form, to_device(left), to_device(codes), to_device(scales), M, N, K, out=out,
                              workspace=grad_ws(form, M, N, K, fp4=True))
    else:
        q.quest_grad_gemm(form, to_device(left), to_device(codes), to_device(scales), bits, M, N, K, out=out,
                          workspace=grad_ws(form, M, N, K))
    torch.cuda.synchronize()
    assert not torch.isnan(out.float()).any()
    rows = np.unique(np.concatenate([np.arange(0, R, 64), np.arange(63, R, 64), rng.integers(0, R, 30), [R - 1]]))
    value = qo.unpack_fp4(codes, q_shape[1]) if fp4 else qo.unpack_odd(codes, q_shape[1], bits)
    q16 = qo.widen(synth.to_bf16_bits(scales[:, None] * value.astype(np.float32)))
    l64 = qo.widen(np.ascontiguousarray(left[:, rows].T if form == 1 else left[rows]))
    r64 = q16.T if form == 2 else q16
    mirror, spread = l64 @ r64, np.sqrt((l64 ** 2) @ (r64 ** 2))
    got = to_host_f64(out[torch.from_numpy(rows).to(DEV)])
    # fp32 accumulation order and one bf16 rounding (the bound of the other tests of these products)
    assert np.all(np.abs(got - mirror) <= BF16_HALF_ULP * 1.001 * np.abs(mirror) + 2e-5 * spread)
