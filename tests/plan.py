"""Which kernel a call runs, asked of the library (include/quest_plan.h): for tests that must reach a certain one.
No GPU needed."""
import ctypes
from collections import namedtuple

from paper_2502_05003_amd import binding as q

CUS = 256                                                      # compute units of an MI355X
GENERAL, INSTANCE, ROWS, FEW, TILES, SPLIT, MID = range(7)     # quest_plan_kernel
Plan = namedtuple("Plan", "kernel rows cols count")


class _Plan(ctypes.Structure):
    _fields_ = [(name, ctypes.c_int32) for name in ("kernel", "block_rows", "block_cols", "count")]


Ring = namedtuple("Ring", "on anew mixed")


Few = namedtuple("Few", "rows cols in_flight waves")


class _Ring(ctypes.Structure):
    _fields_ = [(name, ctypes.c_int32) for name in Ring._fields]


class _Few(ctypes.Structure):
    _fields_ = [(name, ctypes.c_int32) for name in ("block_rows", "block_cols", "in_flight", "waves")]


def _ask(name, *args, result=_Plan):
    function = getattr(q.load(), name)
    function.restype = result
    p = function(*args)
    return {_Plan: Plan, _Ring: Ring, _Few: Few}[result](*(getattr(p, field) for field, _ in result._fields_))


def _i64(*values):
    return [ctypes.c_int64(v) for v in values]


def grad_gemm(form, M, N, K, bits=4):
    """bits = 0: E2M1 codes"""
    return _ask("quest_plan_grad_gemm", form, bits, *_i64(M, N, K), CUS)


def ring(form, M, N, K, bits=4):
    return _ask("quest_plan_grad_gemm_ring", form, bits, *_i64(M, N, K), CUS, result=_Ring)


def forward(M, N, K, bits, workspace=True):
    """bits = 0: E2M1 codes"""
    return _ask("quest_plan_forward", bits, *_i64(M, N, K), int(workspace))


def few(M, N, K, bits):
    """The block where forward() says FEW; bits = 0: E2M1 codes"""
    return _ask("quest_plan_forward_few", bits, *_i64(M, N, K), result=_Few)


def quantize(rows, cols, block, bits, dtype, absmax=False, fp4=False):
    return _ask("quest_plan_quantize", 1 if absmax else 2 if fp4 else 0, int(dtype == "f32"), *_i64(rows, cols), block,
                bits).kernel
