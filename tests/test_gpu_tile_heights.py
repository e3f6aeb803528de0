"""The gradient and weight-only products at sizes where the dispatch takes tiles of 64, 128, 192 or 256 rows,
several tiles per workgroup and split tiles included (csrc/grad_gemm.hip): outputs ending inside a tile
both ways, sampled rows around the tile edges against the product of the same 16-bit operands in double.
Where workgroups have several tiles, whole outputs: the ring of stages runs on from a tile to the next, or begins anew.
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


# rows of a tile, form, contraction, output rows, output columns; what a workgroup's ring does at the ends of its tiles: it
# always runs on; or it begins anew at an edge of the output in some workgroups, in some of which it also runs on.  Three tiles
# or four to a workgroup, two of 128 rows, which never have more; columns beyond the last whole tile: none, 64, 128 or 192
RINGS = [(128, 0, 1280, 3136, 5120, "on"), (128, 1, 1088, 4992, 3328, "on"), (128, 2, 2880, 4992, 3328, "on"),
         (192, 0, 640, 19008, 1792, "on"), (192, 1, 704, 19008, 1792, "on"), (192, 2, 1024, 2112, 17408, "on"),
         (256, 0, 1024, 2560, 18688, "on"), (256, 1, 768, 15552, 4096, "on"), (256, 2, 768, 18944, 2560, "on"),
         (192, 0, 640, 12096, 2752, "mixed"), (192, 1, 640, 11136, 3008, "mixed"), (192, 2, 960, 6912, 4800, "mixed"),
         (256, 0, 896, 10240, 4672, "mixed"), (256, 1, 960, 15104, 3136, "mixed"), (256, 2, 896, 15168, 2816, "mixed")]


@pytest.mark.parametrize("tile_rows,form,C,R,cols,ends", RINGS)
def test_whole_output_where_workgroups_have_several_tiles(tile_rows, form, C, R, cols, ends):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(C + R + cols + form)
    q_shape = (cols, C) if form == 2 else (C, cols)
    codes = torch.randint(0, 256, (q_shape[0], q_shape[1] // 2), dtype=torch.uint8, device=DEV, generator=gen)
    scales = (torch.rand(q_shape[0], device=DEV, generator=gen) + 0.5) * 0.01
    lefts = [(torch.randn(*((C, R) if form == 1 else (R, C)), device=DEV, generator=gen) * 0.03).bfloat16() for _ in range(2)]
    M, N, K = layer(form, C, R, cols)
    workspace = weight_only_ws(M, N, K) if form == 2 else grad_ws(form, M, N, K)
    outs = [torch.full((R, cols), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(3)]
    for left, out in zip(lefts + lefts[:1], outs):
        if form == 2:
            q.quest_weight_only_gemm(left, codes, scales, 4, y=out, workspace=workspace)
        else:
            q.quest_grad_gemm(form, left, codes, scales, 4, M, N, K, out=out, workspace=workspace)
    torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.int16), outs[2].view(torch.int16))
    odd = 2 * torch.stack([codes & 15, codes >> 4], dim=2).reshape(q_shape).float() - 15
    q64 = (scales[:, None] * odd).bfloat16().double()
    r64 = q64.t().contiguous() if form == 2 else q64
    for left, out in zip(lefts, outs):
        l64 = (left.t().contiguous() if form == 1 else left).double()
        mirror, spread = l64 @ r64, torch.sqrt((l64 ** 2) @ (r64 ** 2))
        # fp32 accumulation order and one bf16 rounding, as above (a NaN fails)
        assert bool(((out.double() - mirror).abs() <= BF16_HALF_ULP * 1.001 * mirror.abs() + 2e-5 * spread).all())
