"""The gradient and weight-only products at sizes where the dispatch takes tiles of 64, 128, 192 or 256 rows,
several tiles per workgroup included (csrc/grad_gemm.hip): outputs ending inside a tile both ways,
sampled rows around the tile edges against the product of the same 16-bit operands in double."""
import numpy as np
import pytest
import torch

from oracle import quest_oracle as qo
from paper_2502_05003_amd import binding as q
from paper_2502_05003_amd import synth

from gpu_util import BF16_HALF_ULP, DEV, grad_ws, to_device, to_host_f64, weight_only_ws

pytestmark = pytest.mark.gpu

# form, contraction, output rows, output columns
CASES = [(1, 16384, 1600, 1664), (0, 8192, 4032, 960),          # rows of 64: about a round of the chip
         (0, 5632, 4032, 1984), (0, 11008, 1088, 5568),         # 128
         (1, 2048, 5568, 1984), (2, 2048, 1984, 5568), (0, 6912, 4032, 2496), (1, 4096, 6848, 2496),   # 192, one and two rounds
         (0, 2048, 8128, 4544), (2, 1024, 4032, 4160), (1, 2048, 4032, 4032)]   # 256 and several rounds


@pytest.mark.parametrize("form,C,R,cols", CASES)
def test_sampled_rows(form, C, R, cols):
    rng = np.random.default_rng(C + R + cols + form)
    q_shape = (cols, C) if form == 2 else (C, cols)
    codes = rng.integers(0, 256, size=(q_shape[0], q_shape[1] // 2), dtype=np.uint8)
    scales = ((rng.random(q_shape[0]) + 0.5) * 0.01).astype(np.float32)
    left = synth.gaussian(*((C, R) if form == 1 else (R, C)), 0.03, 5, "bf16")
    out = torch.full((R, cols), float("nan"), dtype=torch.bfloat16, device=DEV)
    if form == 2:
        q.quest_weight_only_gemm(to_device(left), to_device(codes), to_device(scales), 4, y=out,
                                 workspace=weight_only_ws(R, cols, C))
    else:
        M, N = (R, C) if form == 0 else (C, R)
        q.quest_grad_gemm(form, to_device(left), to_device(codes), to_device(scales), 4, M, N, cols, out=out,
                          workspace=grad_ws(form, M, N, cols))
    torch.cuda.synchronize()
    assert not torch.isnan(out.float()).any()
    rows = np.unique(np.concatenate([np.arange(0, R, 64), np.arange(63, R, 64), rng.integers(0, R, 30), [R - 1]]))
    q16 = qo.widen(synth.to_bf16_bits(scales[:, None] * qo.unpack_odd(codes, q_shape[1], 4).astype(np.float32)))
    l64 = qo.widen(np.ascontiguousarray(left[:, rows].T if form == 1 else left[rows]))
    r64 = q16.T if form == 2 else q16
    mirror, spread = l64 @ r64, np.sqrt((l64 ** 2) @ (r64 ** 2))
    got = to_host_f64(out[torch.from_numpy(rows).to(DEV)])
    # fp32 accumulation order and one bf16 rounding (the bound of the other tests of these products)
    assert np.all(np.abs(got - mirror) <= BF16_HALF_ULP * 1.001 * np.abs(mirror) + 2e-5 * spread)
