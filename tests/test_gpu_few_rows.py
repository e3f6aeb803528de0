"""The forward product with few activation rows (csrc/skinny_gemm.hip) against the CPU oracle: every
block size of the kernel, ragged last blocks, contractions that end in half a unit or are one, every grid."""
import numpy as np
import pytest
import torch

from oracle import quest_oracle as qo
from oracle.quest_oracle import _load, _ptr
from paper_2502_05003_amd import binding as q

from gpu_util import DEV, check_gemm_output, to_device

pytestmark = pytest.mark.gpu

#        M, N, K: blocks of 1x1, 1x2, 2x2, 4x2 and 4x4 sixteens
# (One rounding is up to 2^-8 = 3.9e-3 of an element and 1.7e-3 norm-wise over many; check_gemm_output's
# norm-wise bound of 2e-3 needs the many: a few hundred outputs of comparable size at least.)
SHAPES = [(1, 1057, 64), (16, 4100, 192), (5, 130, 4096), (17, 4097, 320), (33, 2561, 128), (40, 5632, 256),
          (65, 2050, 576), (129, 1030, 1088)]


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_integer_grids(M, N, K, bits):
    rng = np.random.default_rng(M + N + K + bits)
    L, cb = 1 << bits, qo.container_bits(bits)
    ka = rng.integers(-L // 2, L // 2, size=(M, K), dtype=np.int32)
    kb = rng.integers(-L // 2, L // 2, size=(N, K), dtype=np.int32)
    ka[M // 2], kb[0], kb[-1] = L // 2 - 1, L // 2 - 1, -L // 2      # largest |acc|
    if M == 1:   # one row of two huge outputs and small ones would round like two elements
        ka[0, ::2] = rng.integers(-L // 2, L // 2, size=K // 2)
    a, b = (np.empty((r, K * cb // 8), dtype=np.uint8) for r in (M, N))
    _load().qo_pack_codes(_ptr(ka), M, K, bits, _ptr(a))
    _load().qo_pack_codes(_ptr(kb), N, K, bits, _ptr(b))
    sa = (rng.random(M) + 0.5).astype(np.float32)
    sb = ((rng.random(N) + 0.5) * 0.01).astype(np.float32)
    y = torch.full((M, N + 3), 7.0, dtype=torch.bfloat16, device=DEV)
    acc = torch.empty(M, N, dtype=torch.int32, device=DEV)
    q.quest_lowbit_gemm(to_device(a), to_device(sa), to_device(b), to_device(sb), K, bits, y=y[:, :N], acc_out=acc)
    torch.cuda.synchronize()
    ref = qo.gemm_odd(2 * ka + 1, 2 * kb + 1)
    assert np.array_equal(acc.cpu().numpy().astype(np.int64), ref)
    check_gemm_output(y[:, :N], ref, sa, sb)
    assert torch.all(y[:, N:] == 7.0)


@pytest.mark.parametrize("M,N,K", [s for s in SHAPES if s[2] % 128 == 0] + [(30, 96, 640)])
def test_fp4_grid(M, N, K):
    rng = np.random.default_rng(M + N + K)
    a = rng.integers(0, 256, size=(M, K // 2), dtype=np.uint8)
    b = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
    sa = (rng.random(M) + 0.5).astype(np.float32)
    sb = ((rng.random(N) + 0.5) * 0.01).astype(np.float32)
    y = torch.full((M, N), 7.0, dtype=torch.bfloat16, device=DEV)
    acc = torch.empty(M, N, dtype=torch.float32, device=DEV)
    q.quest_lowbit_gemm_fp4(to_device(a), to_device(sa), to_device(b), to_device(sb), K, y=y, acc_out=acc)
    torch.cuda.synchronize()
    ref = qo.unpack_fp4(a, K).astype(np.float64) @ qo.unpack_fp4(b, K).astype(np.float64).T
    assert np.array_equal(acc.cpu().numpy().astype(np.float64), ref)
    check_gemm_output(y, ref, sa, sb)


def test_a_captured_decode_step_replays_on_new_inputs():
    """Quantizer and product of a decode step captured with no call of either before it in this stream (only
    quest_init): every replay gives the bytes of eager calls on the same inputs."""
    M, N, K, n, bits = 24, 2048, 2560, 512, 4
    q.quest_init()
    x = torch.empty(M, K, dtype=torch.bfloat16, device=DEV)
    w_codes = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device=DEV)
    w_scales = torch.rand(N, device=DEV) * 0.01 + 0.005

    def step():
        codes = torch.empty(M, K // 2, dtype=torch.uint8, device=DEV)
        scales = torch.empty(M, device=DEV)
        y = torch.empty(M, N, dtype=torch.bfloat16, device=DEV)
        q.quest_hadamard_quantize(x, n, bits, codes=codes, scales=scales)
        q.quest_lowbit_gemm(codes, scales, w_codes, w_scales, K, bits, y=y)
        return codes, scales, y

    torch.cuda.synchronize()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            captured = step()
    for seed in range(3):
        x.copy_(torch.randn(M, K, generator=torch.Generator().manual_seed(seed)).bfloat16())
        eager = step()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(captured, eager):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), seed


def test_calls_go_to_the_current_stream():
    """The stream handle the binding passes on is that of torch's current stream, default and others."""
    streams = [torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    for stream in streams:
        with torch.cuda.stream(stream):
            assert q._stream() == torch.cuda.current_stream().cuda_stream == stream.cuda_stream
    assert len({stream.cuda_stream for stream in streams}) == 3


# many blocks: 4x2 sixteens by four waves, one and two units of a wave in flight; 4x4
@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("M,N,K", [(65, 8200, 192), (70, 8200, 1088), (66, 8200, 2112)])
def test_integer_grids_many_blocks(M, N, K, bits):
    test_integer_grids(M, N, K, bits)


# the other blocks of many: 4x4 of 8 and 12 units, in one round; 4x2 by eight waves, 4x4 of 14 E2M1 units
@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("M,N,K", [(130, 8200, 1088), (130, 8200, 1600), (66, 6200, 1792)])
def test_integer_grids_many_blocks_of_few_units(M, N, K, bits):
    test_integer_grids(M, N, K, bits)


# the other blocks that E2M1 codes can get: two sixteens square, 4x2 by four and by eight waves, 4x4 of 14 and 16 units, and one for
# few rows of large weights
FP4_MANY = [(33, 3000, 128), (40, 16500, 256), (40, 16500, 1024), (66, 6200, 1664), (66, 6200, 1792), (66, 8100, 2048),
            (10, 8300, 8192)]


@pytest.mark.parametrize("M,N,K", FP4_MANY)
def test_fp4_grid_many_blocks(M, N, K):
    test_fp4_grid(M, N, K)
