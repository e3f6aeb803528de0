"""The 16-bit products of outputs of few tiles (csrc/grad_gemm_mid.hip) against the product of the same
16-bit operands in double: every block shape the dispatch chooses from, tiles and step counts that end
inside a block or a round, all three forms, every grid."""
import numpy as np
import pytest
import torch

from oracle import quest_oracle as qo
from paper_2502_05003_amd import binding as q
from paper_2502_05003_amd import synth

from gpu_util import BF16_HALF_ULP, DEV, grad_ws, to_device, to_host_f64, weight_only_ws

pytestmark = pytest.mark.gpu

# contraction, output rows, output columns: one step; 3 steps for four groups; 9 for two; 28; 11 of 128 x 128
# blocks for two groups, rows ending inside one; 3 of 128 x 128 blocks, both edges inside one
SHAPES = [(64, 64, 64), (192, 64, 64), (576, 64, 128), (1792, 2048, 640), (704, 576, 5632), (192, 4160, 2112),
          # the smaller blocks at outputs that every form and grid takes
          (128, 128, 128), (192, 192, 192), (128, 320, 11008), (192, 640, 1664)]


# (E2M1 codes and the weight-only product: outputs of at least 128 x 128; no weight-only product on E2M1)
CASES = [(*shape, form, grid) for shape in SHAPES for form in (0, 1, 2) for grid in (1, 2, 3, 4, "fp4")
         if not ((grid == "fp4" or form == 2) and min(shape[1:]) < 128) and not (grid == "fp4" and form == 2)]


@pytest.mark.parametrize("C,R,cols,form,grid", CASES)
def test_product_of_the_16_bit_operands(C, R, cols, form, grid):
    fp4, bits = grid == "fp4", 4 if grid == "fp4" else grid
    rng = np.random.default_rng(C + R + cols + form)
    q_shape = (cols, C) if form == 2 else (C, cols)          # the packed operand
    cb = qo.container_bits(bits)
    codes = rng.integers(0, 256, size=(q_shape[0], q_shape[1] * cb // 8), dtype=np.uint8)
    if grid == 3:
        codes &= 0x77
    scales = ((rng.random(q_shape[0]) + 0.5) * 0.01).astype(np.float32)
    value = qo.unpack_fp4(codes, q_shape[1]) if fp4 else qo.unpack_odd(codes, q_shape[1], bits)
    q16 = qo.widen(synth.to_bf16_bits(scales[:, None] * value.astype(np.float32)))
    left = synth.gaussian(*((C, R) if form == 1 else (R, C)), 0.03, 5, "bf16")
    l64 = qo.widen(left).T if form == 1 else qo.widen(left)
    r64 = q16.T if form == 2 else q16
    out = torch.full((R, cols), float("nan"), dtype=torch.bfloat16, device=DEV)
    if form == 2:
        q.quest_weight_only_gemm(to_device(left), to_device(codes), to_device(scales), bits, y=out,
                                 workspace=weight_only_ws(R, cols, C))
    else:
        M, N = (R, C) if form == 0 else (C, R)
        ws = grad_ws(form, M, N, cols, fp4=fp4)
        if fp4:
            q.quest_grad_gemm_fp4(form, to_device(left), to_device(codes), to_device(scales), M, N, cols, out=out,
                                  workspace=ws)
        else:
            q.quest_grad_gemm(form, to_device(left), to_device(codes), to_device(scales), bits, M, N, cols, out=out,
                              workspace=ws)
    torch.cuda.synchronize()
    # fp32 accumulation order and one bf16 rounding (the bound of the other tests of these products)
    mirror, spread = l64 @ r64, np.sqrt((l64 ** 2) @ (r64 ** 2))
    assert np.all(np.abs(to_host_f64(out) - mirror) <= BF16_HALF_ULP * 1.001 * np.abs(mirror) + 2e-5 * spread)
