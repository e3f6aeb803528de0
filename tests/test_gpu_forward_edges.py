"""Edges of the forward product's tile kernels against the CPU oracle: the E2M1 kernel's tiles of 128 rows
(csrc/fp4_gemm.hip) and output rows that 16-byte stores do not fit (csrc/gemm_tile.h), on every grid that uses them."""
import numpy as np
import pytest
import torch

from oracle import quest_oracle as qo
from oracle.quest_oracle import _load, _ptr
from paper_2502_05003_amd import binding as q

from gpu_util import DEV, check_gemm_output, to_device

pytestmark = pytest.mark.gpu

# M, N, K, extra output pitch.  All beyond the few-rows kernel (more than 256 blocks of 64 x 64 at 3 and 4 bits and
# E2M1).  Row pitches of every kind (odd, even, multiple of 8), last tiles of 1, 3, 4 and 128 rows and of 1, 2, 6, 8
# and 72 columns, one to nine contraction steps, one tile row that is not full; (6145, 2050) has enough tiles of
# 256 rows for those.
SHAPES = [(1025, 1153, 128, 0), (1027, 1154, 256, 0), (1280, 1032, 384, 0), (1092, 1224, 1152, 3),
          (1025, 1158, 128, 2), (2049, 520, 384, 1), (6145, 2050, 128, 0), (65, 8321, 128, 0), (127, 8200, 384, 2)]
# 2 bits, re-coded: more than 768 blocks
RECODED = [(2049, 1601, 128, 0), (1793, 1858, 256, 0), (3073, 1032, 384, 1)]
INTEGER_CASES = [(*shape, bits) for shape in SHAPES for bits in (3, 4)] + [(*shape, 2) for shape in RECODED]


def _scales(rng, M, N):
    return (rng.random(M) + 0.5).astype(np.float32), ((rng.random(N) + 0.5) * 0.01).astype(np.float32)


@pytest.mark.parametrize("M,N,K,pad", SHAPES)
def test_fp4_grid(M, N, K, pad):
    rng = np.random.default_rng(M + N + K)
    a = rng.integers(0, 256, size=(M, K // 2), dtype=np.uint8)
    b = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
    sa, sb = _scales(rng, M, N)
    y = torch.full((M, N + pad), 7.0, dtype=torch.bfloat16, device=DEV)
    acc = torch.empty(M, N, dtype=torch.float32, device=DEV)
    q.quest_lowbit_gemm_fp4(to_device(a), to_device(sa), to_device(b), to_device(sb), K, y=y[:, :N], acc_out=acc)
    torch.cuda.synchronize()
    ref = qo.unpack_fp4(a, K).astype(np.float64) @ qo.unpack_fp4(b, K).astype(np.float64).T
    assert np.array_equal(acc.cpu().numpy().astype(np.float64), ref)
    check_gemm_output(y[:, :N], ref, sa, sb)
    assert torch.all(y[:, N:] == 7.0)


@pytest.mark.parametrize("M,N,K,pad,bits", INTEGER_CASES)
def test_integer_grids(M, N, K, pad, bits):
    rng = np.random.default_rng(M + N + K + bits)
    L, cb = 1 << bits, qo.container_bits(bits)
    ka = rng.integers(-L // 2, L // 2, size=(M, K), dtype=np.int32)
    kb = rng.integers(-L // 2, L // 2, size=(N, K), dtype=np.int32)
    a, b = (np.empty((r, K * cb // 8), dtype=np.uint8) for r in (M, N))
    _load().qo_pack_codes(_ptr(ka), M, K, bits, _ptr(a))
    _load().qo_pack_codes(_ptr(kb), N, K, bits, _ptr(b))
    sa, sb = _scales(rng, M, N)
    y = torch.full((M, N + pad), 7.0, dtype=torch.bfloat16, device=DEV)
    acc = torch.empty(M, N, dtype=torch.int32, device=DEV)
    nbytes = q.quest_lowbit_gemm_workspace_bytes(M, N, K, bits)
    scratch = torch.empty(nbytes, dtype=torch.uint8, device=DEV) if nbytes > 0 else None
    q.quest_lowbit_gemm(to_device(a), to_device(sa), to_device(b), to_device(sb), K, bits, y=y[:, :N], acc_out=acc,
                        workspace=scratch)
    torch.cuda.synchronize()
    ref = (2.0 * ka + 1) @ (2.0 * kb + 1).T      # whole numbers below 2^53
    assert np.array_equal(acc.cpu().numpy().astype(np.float64), ref)
    check_gemm_output(y[:, :N], ref, sa, sb)
    assert torch.all(y[:, N:] == 7.0)
