"""The quantizer and the masked inverse transform at row lengths and blocks without an instantiation of
their own (csrc/hadamard_quantize_rows.hip, csrc/trust_backward_rows.hip) against the CPU oracle: rows that
end anywhere in a tile, every kind of block, one and several rows per wave, rows shared by a workgroup.  (The
blocks of 8 or less among them run the general kernels for fp32 rows and for the inverse transform.)"""
import numpy as np
import pytest
import torch

from oracle import quest_oracle as qo
from paper_2502_05003_amd import binding as q
from paper_2502_05003_amd import synth

from gpu_util import BF16_HALF_ULP, DEV, compare_quantizer, compare_quantizer_fp4, gpu_quantize, to_device, to_host_f64

pytestmark = pytest.mark.gpu

#        rows, row length, block: one tile or less, an odd multiple of 64; ends in a tile; two and four tiles
#        per block; more rows than resident waves (4096) or row-sharing workgroups (1024)
SHAPES = [(256, 64, 64), (300, 192, 2), (257, 960, 64), (261, 1088, 16), (333, 2560, 512), (259, 6144, 2048),
          (256, 8192, 4096), (1031, 3136, 64), (4201, 1536, 512), (1100, 5760, 128)]


CASES = [(*shape, dtype, grid) for shape in SHAPES for dtype in ("bf16", "f32") for grid in (1, 2, 3, 4, 8, "fp4")]


@pytest.mark.parametrize("rows,cols,n,dtype,grid", CASES)
def test_quantizer(rows, cols, n, dtype, grid):
    x = synth.outlier_activations(rows, cols, 0.01, 20.0, seed=rows + cols, dtype=dtype)
    x[rows // 2] = 0
    if grid == "fp4":
        got = gpu_quantize(x, n, 4, fp4=True, want_xh=False)
        compare_quantizer_fp4(got, qo.hadamard_quantize_fp4(x, n), cols)
    else:
        got = gpu_quantize(x, n, grid, want_xh=(grid == 3))
        compare_quantizer(got, qo.hadamard_quantize(x, n, grid), cols, grid)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_8_bit_codes_are_decided_by_the_rounded_product(dtype):
    """A code differs from the 64-bit one where a cell boundary lies between x_h / step and its fp32 value.  With
    the fp32 roundings of scale and product, 6e-8 each, and |x_h| / step = 26 on average that is about 2e-6 of the
    elements; deciding on the sum with 127.5 (spacing 1.5e-5) makes it 6e-6."""
    rows, cols, n = 4096, 2560, 512
    x = synth.outlier_activations(rows, cols, 0.01, 20.0, seed=5, dtype=dtype)
    got, ref = gpu_quantize(x, n, 8, want_xh=False), qo.hadamard_quantize(x, n, 8)
    assert compare_quantizer(got, ref, cols, 8)[0] < 3.5e-6 * x.size


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("grid", [1, 2, 3, 4, 8, "fp4"])
def test_rows_whose_squares_underflow_are_zero_rows(grid, dtype):
    """Entries of about 2^-80 of both signs: the row's sum of squares is 0 in fp32, so the row is quantized like
    an all-zero one, scale 0, code k = 0 (E2M1: +0) and every element trusted."""
    rows, cols = 300, 1536
    x = synth.gaussian(rows, cols, 1.0, 3, "f32") * np.float32(2.0 ** -80)
    x = synth.to_bf16_bits(x) if dtype == "bf16" else x
    got = gpu_quantize(x, 512, 4 if grid == "fp4" else grid, fp4=grid == "fp4", want_xh=False)
    assert np.all(got["scales"] == 0.0) and np.all(got["mask"] == 0xFF)
    if grid == "fp4":
        assert np.all(got["codes"] == 0)
    else:
        assert np.all(qo.unpack_odd(got["codes"], cols, grid) == 1)


# a shape without an instantiation, each grid; one wave per row and shared rows (up to 1024) on the larger side
COUNTS = [(1100, 2560, 512, "bf16", grid) for grid in (1, 2, 3, 4, 8, "fp4")] + \
         [(300, 1088, 16, "f32", 4), (1100, 2560, 512, "f32", 3), (300, 8192, 4096, "bf16", 4)] + \
         [(2100, cols, n, "f32", 4) for cols, n in ((1024, 1024), (1280, 256), (1664, 128), (1792, 256), (2048, 2048),
                                                    (2816, 256), (3584, 512), (4096, 4096), (4608, 512), (5632, 512))] + \
         [(300, 11008, 256, "bf16", 4), (300, 5632, 512, "bf16", 4)]


@pytest.mark.parametrize("rows,cols,n,dtype,grid", COUNTS)
def test_a_row_does_not_depend_on_the_number_of_rows(rows, cols, n, dtype, grid):
    """A token quantized alone, in a short call and in a long one gets the same bytes, whatever kernel takes the call."""
    x = synth.outlier_activations(rows, cols, 0.01, 20.0, seed=cols, dtype=dtype)
    args = dict(bits=4, fp4=True) if grid == "fp4" else dict(bits=grid)
    whole = gpu_quantize(x, n, want_xh=False, **args)
    for rows_of_call in (slice(0, 1), slice(7, 31), slice(0, 255), slice(1, 299)):
        part = gpu_quantize(x[rows_of_call], n, want_xh=False, **args)
        for name in ("codes", "scales", "mask"):
            assert np.array_equal(part[name].view(np.uint8), whole[name][rows_of_call].view(np.uint8)), (name, rows_of_call)


# every block size has stages of its own, in whole groups of tiles and in the one that the row ends in; rows of 2048 and
# 2816 fp32 elements change kernels between 40 and 1100 of them
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("cols,n", [(2112, 1), (3136, 4), (2112, 32), (3136, 64), (2432, 128), (2304, 256), (2560, 512),
                                    (5120, 1024), (6144, 2048), (12288, 4096), (2048, 2048), (2816, 256)])
def test_quantizer_block_sizes(cols, n, dtype):
    x = synth.outlier_activations(1100, cols, 0.01, 20.0, seed=n, dtype=dtype)
    whole, few = (gpu_quantize(x[:rows], n, 4, want_xh=False) for rows in (1100, 40))
    compare_quantizer(whole, qo.hadamard_quantize(x, n, 4), cols, 4)
    for name in ("codes", "scales", "mask"):
        assert np.array_equal(few[name].view(np.uint8), whole[name][:40].view(np.uint8)), name


def test_quantizer_strided_rows_and_no_mask():
    """A row pitch above the row length; the codes do not depend on whether the mask is asked for."""
    x = synth.outlier_activations(270, 2560, 0.01, 20.0, seed=1, dtype="bf16")
    with_mask, without = gpu_quantize(x, 512, 4, want_xh=False), gpu_quantize(x, 512, 4, want_xh=False, want_mask=False, ld=2568)
    assert np.array_equal(with_mask["codes"], without["codes"])
    assert np.array_equal(with_mask["scales"], without["scales"])


@pytest.mark.parametrize("rows_x,rows_w", [(400, 300), (3000, 500), (3000, 40), (0, 300)])
def test_pairs_equal_single_calls(rows_x, rows_w):
    cols, n = 2560, 512
    x, w = (torch.randn(r, cols, device=DEV).bfloat16() for r in (rows_x + 1, rows_w))
    x = x[:rows_x]
    def buffers(r):
        return dict(codes=torch.full((r, cols // 2), 0xAA, dtype=torch.uint8, device=DEV),
                    scales=torch.full((r,), -1.0, device=DEV), mask=torch.full((r, cols // 8), 0x55, dtype=torch.uint8, device=DEV))
    pair, single = (buffers(rows_x), buffers(rows_w)), (buffers(rows_x), buffers(rows_w))
    q.quest_hadamard_quantize_pair(x, w, n, 4, **{f"x_{k}": v for k, v in pair[0].items()},
                                   **{f"w_{k}": v for k, v in pair[1].items()})
    for t, out in ((x, single[0]), (w, single[1])):
        if t.shape[0]:
            q.quest_hadamard_quantize(t, n, 4, **out)
    dx = [torch.full((r, cols), 7.0, dtype=torch.bfloat16, device=DEV) for r in (rows_x, rows_w, rows_x, rows_w)]
    q.quest_trust_backward_pair(x, pair[0]["mask"], w, pair[1]["mask"], n, out_x=dx[0], out_w=dx[1])
    for t, m, out in ((x, pair[0]["mask"], dx[2]), (w, pair[1]["mask"], dx[3])):
        if t.shape[0]:
            q.quest_trust_backward(t, m, n, out=out)
    torch.cuda.synchronize()
    for a, b in zip(pair, single):     # the same bits, whether a row is one wave's or shared by a workgroup
        assert all(torch.equal(a[k], b[k]) for k in a)
    assert torch.equal(dx[0], dx[2]) and torch.equal(dx[1], dx[3])


@pytest.mark.parametrize("od", ["bf16", "f32"])
@pytest.mark.parametrize("masked", [True, False])
@pytest.mark.parametrize("rows,cols,n", SHAPES + [(3, 5632, 512), (9, 11008, 256), (5, 3584, 4), (3, 12288, 4096), (1, 64, 1)])
def test_inverse_transform(rows, cols, n, masked, od):
    g = synth.gaussian(rows, cols, 0.03, seed=rows + cols, dtype="bf16")
    trust = (np.random.default_rng(cols).random((rows, cols)) < 0.9).astype(np.uint8)
    packed = np.packbits(trust, axis=1, bitorder="little")
    out = torch.full((rows, cols), float("nan"), dtype=torch.bfloat16 if od == "bf16" else torch.float32, device=DEV)
    q.quest_trust_backward(to_device(g), to_device(packed) if masked else None, n, out=out)
    torch.cuda.synchronize()
    ref = qo.trust_backward(qo.widen(g), trust if masked else np.ones_like(trust), n)
    scale = np.sqrt(np.mean(ref * ref, axis=1, keepdims=True))
    rounding = BF16_HALF_ULP if od == "bf16" else 0.0
    assert np.all(np.abs(to_host_f64(out) - ref) <= rounding * np.abs(ref) + 1e-5 * scale + 1e-30)


# row lengths that have an instantiation for few elements (512, 640, 1280), none (2560: units end inside a row; 64), blocks of
# 2048 and 4096; the second gradient starts a unit of its own
@pytest.mark.parametrize("od", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,cols,n", [(7001, 512, 512), (5503, 640, 128), (2611, 1280, 256), (1601, 2560, 512),
                                         (4097, 64, 64), (701, 6144, 2048), (401, 12288, 4096)])
def test_inverse_transform_of_a_row_does_not_depend_on_the_others(rows, cols, n, od):
    """A row alone, in a short call, in a long one and as the second gradient gets the same bits; an infinity and a
    NaN stay in their rows."""
    g = torch.randn(rows, cols, device=DEV).bfloat16()
    mask = torch.randint(0, 256, (rows, cols // 8), dtype=torch.uint8, device=DEV)
    g[rows // 2, 3], g[rows - 2, cols - 1] = float("inf"), float("nan")
    clean = torch.ones(rows, dtype=torch.bool, device=DEV)
    clean[rows // 2] = clean[rows - 2] = False

    def transform(*parts):
        out = [torch.full((p.stop - p.start, cols), 7.0, dtype=od, device=DEV) for p in parts]
        if len(parts) == 1:
            q.quest_trust_backward(*(t[parts[0]].clone() for t in (g, mask)), n, out=out[0])
        else:
            q.quest_trust_backward_pair(*(t[p].clone() for p in parts for t in (g, mask)), n, out_x=out[0], out_w=out[1])
        return out

    whole, = transform(slice(0, rows))
    for parts in ([slice(0, 2)], [slice(rows - 16, rows)], [slice(0, 304)], [slice(0, 32), slice(rows - 2, rows)],
                  [slice(0, rows - 1), slice(16, 32)]):
        for part, out in zip(parts, transform(*parts)):
            keep = clean[part]
            assert torch.equal(out[keep], whole[part][keep])
    assert torch.isfinite(whole[clean].float()).all()


# more units than the 4096 resident waves: of the second on, the stores of the one before are on their way while it is awaited
@pytest.mark.parametrize("od", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("masked", [True, False])
@pytest.mark.parametrize("rows,cols,n", [(8201, 2560, 512), (140001, 64, 64), (4100, 6144, 2048), (4201, 12288, 4096)])
def test_inverse_transform_where_waves_have_several_units(rows, cols, n, masked, od):
    """The same bits as from calls in which no wave has more than one."""
    g = torch.randn(rows, cols, device=DEV).bfloat16()
    mask = torch.randint(0, 256, (rows, cols // 8), dtype=torch.uint8, device=DEV)
    whole = torch.full((rows, cols), 7.0, dtype=od, device=DEV)
    q.quest_trust_backward(g, mask if masked else None, n, out=whole)
    part_rows = (2 << 20) // cols // 2 * 2   # (an even number: 16 bytes of mask bits)
    for at in range(0, rows, part_rows):
        part = slice(at, min(at + part_rows, rows))
        out = torch.full((part.stop - at, cols), 7.0, dtype=od, device=DEV)
        q.quest_trust_backward(g[part], mask[part] if masked else None, n, out=out)
        assert torch.equal(out, whole[part]), at


# rows of three groups of tiles and more, which a workgroup shares up to 128 rows: 5632 and 4608 through LDS, 11008 not
@pytest.mark.parametrize("cols,n,grid", [(5632, 512, 4), (5632, 32, 4), (5632, 512, 1), (5632, 512, 2), (5632, 512, 3), (5632, 512, 8),
                                         (5632, 512, "fp4"), (4608, 512, 4), (11008, 256, 4), (11008, 1, 4)])
def test_a_row_that_a_workgroup_shares_has_the_same_bytes(cols, n, grid):
    """One row, the most that are shared, and more; with and without mask; with an infinity and a zero row among them."""
    x = synth.outlier_activations(130, cols, 0.01, 20.0, seed=cols, dtype="bf16")
    x[5], x[9] = 0, 0
    x[9, 17] = 0x7F80   # infinity: this row's codes are unspecified
    args = dict(bits=4, fp4=True) if grid == "fp4" else dict(bits=grid)
    whole = gpu_quantize(x, n, want_xh=False, **args)
    for rows in (1, 9, 128):
        for want_mask in (True, False):
            part = gpu_quantize(x[:rows], n, want_xh=False, want_mask=want_mask, **args)
            keep = np.arange(rows) != 9
            for name in ("codes", "scales") + (("mask",) if want_mask else ()):
                assert np.array_equal(part[name][keep].view(np.uint8), whole[name][:rows][keep].view(np.uint8)), (name, rows)


# both operands' rows count: 128 are shared by workgroups, 129 are not; the first operand's rows end before, at and after a workgroup's
@pytest.mark.parametrize("rows_x,rows_w", [(1, 1), (100, 28), (100, 29), (0, 7), (7, 0)])
@pytest.mark.parametrize("cols,fp4", [(5632, False), (5632, True), (11008, False)])
def test_pairs_that_workgroups_share_equal_single_calls(rows_x, rows_w, cols, fp4):
    operands = [torch.randn(r, cols, device=DEV).bfloat16() for r in (rows_x, rows_w)]
    def buffers(r):
        return dict(codes=torch.full((r, cols // 2), 0xAA, dtype=torch.uint8, device=DEV),
                    scales=torch.full((r,), -1.0, device=DEV), mask=torch.full((r, cols // 8), 0x55, dtype=torch.uint8, device=DEV))
    pair, single = ([buffers(r) for r in (rows_x, rows_w)] for _ in range(2))
    block = cols & -cols
    named = {f"{operand}_{k}": v for operand, out in zip("xw", pair) for k, v in out.items()}
    if fp4:
        q.quest_hadamard_quantize_fp4_pair(*operands, block, **named)
    else:
        q.quest_hadamard_quantize_pair(*operands, block, 4, **named)
    for t, out in zip(operands, single):
        if t.shape[0] and fp4:
            q.quest_hadamard_quantize_fp4(t, block, **out)
        elif t.shape[0]:
            q.quest_hadamard_quantize(t, block, 4, **out)
    torch.cuda.synchronize()
    for a, b in zip(pair, single):
        assert all(torch.equal(a[k], b[k]) for k in a)
