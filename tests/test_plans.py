"""The GPU tests' cases against the dispatch rules, on the CPU: each kernel and block shape of the products that a
rule can choose is run by a case that is listed for it.  A change of a rule that takes a case elsewhere fails here."""
import math
import random

import pytest

import plan
import test_gpu_forward_edges as edges
import test_gpu_mid_products as mid
import test_gpu_parity as parity
import test_gpu_tile_heights as tiles

from paper_2502_05003_amd import binding as q


@pytest.mark.parametrize("kernel,rows,several,form,C,R,cols,grid", tiles.RUNS)
def test_tile_cases_are_where_they_are_listed(kernel, rows, several, form, C, R, cols, grid):
    p = plan.grad_gemm(form, *tiles.layer(form, C, R, cols), bits=0 if grid == "fp4" else grid)
    assert (p.kernel, p.rows, p.count > 1) == (kernel, rows, several)


@pytest.mark.parametrize("rows,form,C,R,cols,ends", tiles.RINGS)
def test_ring_cases_do_what_they_are_listed_for(rows, form, C, R, cols, ends):
    p, ring = plan.grad_gemm(form, *tiles.layer(form, C, R, cols)), plan.ring(form, *tiles.layer(form, C, R, cols))
    assert (p.kernel, p.rows) == (plan.TILES, rows) and p.count >= (2 if rows == 128 else 3)
    assert ring.on > 0 and (ring.anew, ring.mixed) == (0, 0) if ends == "on" else ring.mixed > 0


def test_tile_cases_with_several_have_workgroups_that_begin_anew():
    """(two tiles each: in one workgroup the ring either runs on or begins anew)"""
    for kernel, rows, several, form, C, R, cols, grid in tiles.RUNS:
        ring = plan.ring(form, *tiles.layer(form, C, R, cols), bits=0 if grid == "fp4" else grid)
        assert (ring.on > 0) == several and ring.mixed == 0


def test_tile_cases_have_every_height_in_every_form():
    heights = {(case[3], case[0], case[1]) for case in tiles.RUNS if case[-1] != "fp4"}
    assert heights == {(form, plan.TILES, rows) for form in (0, 1, 2) for rows in (64, 128, 192, 256)} | \
        {(form, plan.SPLIT, 256) for form in (0, 1, 2)}
    assert {(case[0], case[1]) for case in tiles.RUNS if case[-1] == "fp4"} == {k[1:] for k in heights}


def test_tiles_of_64_rows_are_one_to_a_workgroup():
    """There is no form of theirs that runs on from tile to tile: sizes of every magnitude, every form and grid."""
    rng = random.Random(1)
    size = lambda: 64 * round(math.exp(rng.uniform(0, math.log(rng.choice((256, 1024, 65536))))))
    found = set()
    for _ in range(30000):
        form = rng.choice((0, 1, 2))
        p = plan.grad_gemm(form, size(), size(), size(), bits=rng.choice((1, 2, 3, 4) if form == 2 else (0, 1, 2, 3, 4)))
        if p.kernel == plan.TILES:
            found.add((p.rows, p.count > 1))
    assert found == {(64, False)} | {(rows, several) for rows in (128, 192, 256) for several in (False, True)}


def test_mid_cases_have_every_block_in_every_form_and_grid():
    found = {}
    for C, R, cols, form, grid in mid.CASES:
        p = plan.grad_gemm(form, *tiles.layer(form, C, R, cols), bits=0 if grid == "fp4" else grid)
        assert p.kernel == plan.MID
        found.setdefault((form, grid), set()).add(p[1:])
    blocks = {(64, 64, 2), (64, 64, 4), (64, 128, 1), (64, 128, 2), (128, 128, 1), (128, 128, 2)}
    assert len(found) == 14
    for (form, grid), b in found.items():   # (one bit: no blocks of 64 x 128 with two groups)
        assert b == (blocks - {(64, 128, 2)} if grid == 1 else blocks), (form, grid)


def test_forward_cases_reach_the_tile_kernels():
    for M, N, K, _ in edges.SHAPES:
        assert plan.forward(M, N, K, 0).kernel == plan.TILES
    assert {plan.forward(M, N, K, 0).rows for M, N, K, _ in edges.SHAPES} == {128, 256}
    for M, N, K, _, bits in edges.INTEGER_CASES:
        assert plan.forward(M, N, K, bits)[::3] == (plan.TILES, 2 if bits == 2 else 0)


def test_forward_cases_reach_every_kernel():
    found = {}
    for M, N, K, bits, scratch in parity.GEMM_RUNS:
        p = plan.forward(M, N, K, bits, scratch and q.quest_lowbit_gemm_workspace_bytes(M, N, K, bits) > 0)
        found.setdefault(bits, set()).add((p.kernel, p.rows, p.cols))
    general, few = (plan.GENERAL, 128, 128), (plan.FEW, 0, 0)
    assert found[1] >= {few, general} and found[2] >= {few, general}
    assert {k[0] for k in found[1]} >= {plan.TILES} and {k[0] for k in found[2]} >= {plan.TILES}
    assert found[3] >= {few, general, (plan.TILES, 256, 128)} and found[4] >= {few, general, (plan.TILES, 256, 128)}


# the block each of these products runs fastest with (of 16 rows and 16 columns: 1, of 64 and 32: 4x2), us there and with the
# block in brackets
@pytest.mark.parametrize("M,N,K,bits,rows,cols,in_flight,waves", [
    (460, 3552, 1792, 1, 64, 64, 1, 4),       # 10.9 (4x2, two units in flight, 14.8)
    (972, 1664, 1664, 2, 64, 64, 1, 4),       # 8.7 (so 10.8, one unit 9.5)
    (763, 4096, 1280, 1, 64, 64, 1, 4),       # 13.6 (18.2, 16.5)
    (3937, 422, 1600, 4, 64, 64, 1, 4),       # 12.0 (14.0, 12.9)
    (97, 11008, 1664, 2, 64, 32, 1, 4),       # 7.7 (8.6; 4x4 8.2)
    (333, 4096, 1024, 2, 64, 32, 2, 4),       # 7.7 (one unit 7.8, 4x4 8.1)
    (1600, 1024, 1024, 2, 64, 64, 1, 4),      # 8.2 (9.1)
    (573, 5225, 1088, 3, 64, 32, 2, 4),       # 14.2 (4x4 16.2)
    (2346, 256, 1792, 0, 64, 64, 1, 4),       # 7.6 (4x2 8.5)
    (512, 2048, 1664, 4, 64, 32, 1, 8),       # 6.3 (four waves 6.6, 4x4 7.1)
    (512, 1664, 2048, 4, 64, 64, 1, 4),       # 8.6 (4x2 9.1)
    (10, 11008, 11008, 0, 16, 16, 2, 4),      # 18.0 (eight waves 20.3)
    (13, 11008, 11008, 3, 16, 16, 1, 8),      # 20.0
    (1, 2048, 5632, 4, 16, 16, 2, 8), (1, 5632, 2048, 4, 16, 16, 1, 8), (24, 2048, 5632, 4, 16, 16, 1, 8)])
def test_blocks_of_few_rows(M, N, K, bits, rows, cols, in_flight, waves):
    assert plan.forward(M, N, K, bits).kernel == plan.FEW
    assert plan.few(M, N, K, bits) == (rows, cols, in_flight, waves)


def test_few_rows_cases_have_every_block():
    import test_gpu_few_rows as few
    shapes = few.SHAPES + [shape for test in (few.test_integer_grids_many_blocks, few.test_integer_grids_many_blocks_of_few_units)
                           for mark in test.pytestmark if mark.args[0] == "M,N,K" for shape in mark.args[1]]
    every = {(16, 16, 1, 8), (16, 16, 2, 8), (16, 32, 2, 4), (32, 32, 2, 4), (64, 32, 1, 8), (64, 32, 1, 4), (64, 32, 2, 4),
             (64, 64, 1, 4)}
    for bits in (1, 2, 3, 4):
        assert {tuple(plan.few(M, N, K, bits)) for M, N, K in shapes if plan.forward(M, N, K, bits).kernel == plan.FEW} == every
    fp4 = [s for s in few.SHAPES if s[2] % 128 == 0] + [(30, 96, 640)] + few.FP4_MANY
    assert {tuple(plan.few(M, N, K, 0)) for M, N, K in fp4 if plan.forward(M, N, K, 0).kernel == plan.FEW} == \
        every | {(16, 16, 2, 4)}


def test_quantizer_kernels():
    assert plan.quantize(24, 2560, 512, 4, "bf16") == plan.quantize(8192, 2560, 512, 4, "bf16") == plan.ROWS
    assert plan.quantize(24, 2048, 2048, 4, "bf16") == plan.quantize(8192, 2048, 2048, 4, "bf16") == plan.INSTANCE
    assert plan.quantize(24, 2048, 2048, 4, "f32") == plan.INSTANCE
    assert plan.quantize(8192, 2048, 2048, 4, "f32") == plan.ROWS
    # blocks of 8 or less: bf16 rows only
    assert plan.quantize(24, 1344, 8, 4, "bf16") == plan.ROWS and plan.quantize(8192, 1344, 8, 4, "f32") == plan.GENERAL
    import test_gpu_stage_isolated as stages
    assert all(plan.quantize(rows, cols, n, bits, dtype) == plan.GENERAL for rows, cols, n, bits, dtype in stages.CASES)
    assert all(plan.quantize(rows, cols, n, bits, dtype) == plan.ROWS for rows, cols, n, bits, dtype in stages.TILE_CASES)


def test_fp4_one_large_tile_per_unit():
    """Long contractions: tiles of 128 rows only where they come out in no more rounds than those of 256."""
    rows = {(tiles, K): plan.forward(256 * tiles // 8, 1024, K, 0).rows
            for tiles in (128, 136, 256, 264, 376, 384) for K in (2048, 2560, 11008)}
    assert all((h == 256) == (tiles == 384 or (tiles in (136, 256) and K > 2048)) for (tiles, K), h in rows.items()), rows
