"""The binding's two ways to an entry point, native code and ctypes, pass it the same arguments; what is not a plain call
takes the second.  (No GPU: the entry points are stand-ins that record what they are given.)"""
import ctypes
import gc
import inspect
import sys
import sysconfig
import types

import numpy as np
import pytest
import torch

import paper_2502_05003_amd as package
from paper_2502_05003_amd import binding as q
from paper_2502_05003_amd import build


class Subclass(torch.Tensor):
    pass


def tensors(dtype=torch.bfloat16):
    wide = torch.zeros(9, 160, dtype=dtype)
    return types.SimpleNamespace(
        x=wide[:5, :128], w=torch.zeros(7, 128, dtype=dtype), none=torch.zeros(0, 128, dtype=dtype),
        codes=torch.zeros(5, 64, dtype=torch.uint8), w_codes=torch.zeros(7, 64, dtype=torch.uint8), scales=torch.zeros(5),
        w_scales=torch.zeros(7), mask=torch.zeros(5, 16, dtype=torch.uint8), w_mask=torch.zeros(7, 16, dtype=torch.uint8),
        xh=torch.zeros(5, 128), y=torch.zeros(5, 24, dtype=torch.bfloat16)[:, :7], acc=torch.zeros(5, 7, dtype=torch.int32),
        scratch=torch.zeros(33, dtype=torch.int16), out=torch.zeros(5, 128), out_w=torch.zeros(7, 128),
        dy=torch.zeros(64, 128, dtype=torch.bfloat16))


def calls(t):
    """name, positional, keyword arguments; forms and options of every call"""
    pair = dict(x_codes=t.codes, x_scales=t.scales, w_codes=t.w_codes, w_scales=t.w_scales)
    masks = dict(x_mask=t.mask, w_mask=t.w_mask)
    yield "quest_hadamard_quantize", (t.x, 64, 4), dict(codes=t.codes, scales=t.scales)
    yield "quest_hadamard_quantize", (t.x, 128, 3, 2.5, 0.75), dict(codes=t.codes, scales=t.scales, mask=t.mask, xh_out=t.xh)
    yield "quest_hadamard_quantize", (t.none, 1, 8), dict(codes=t.codes, scales=t.scales)
    yield "quest_hadamard_quantize_pair", (t.x, t.w, 64, 2, 1.5, 0.5), pair | masks
    yield "quest_hadamard_quantize_pair", (t.none, t.w, 64, 4), pair
    yield "quest_hadamard_quantize_fp4", (t.x, 16), dict(codes=t.codes, scales=t.scales, mask=t.mask)
    yield "quest_hadamard_quantize_fp4", (t.x, 16, 2.0), dict(codes=t.codes, scales=t.scales, xh_out=t.xh)
    yield "quest_hadamard_quantize_fp4_pair", (t.x, t.w, 16, 1.25), pair | masks
    yield "quest_lowbit_gemm", (t.codes, t.scales, t.w_codes, t.w_scales, 128, 4), dict(y=t.y)
    yield "quest_lowbit_gemm", (t.codes, t.scales, t.w_codes, t.w_scales, 128, 2), dict(y=None, acc_out=t.acc, workspace=t.scratch)
    yield "quest_lowbit_gemm_fp4", (t.codes, t.scales, t.w_codes, t.w_scales, 128), dict(y=t.y)
    yield "quest_lowbit_gemm_fp4", (t.codes, t.scales, t.w_codes, t.w_scales, 128), dict(y=None, acc_out=t.out)
    yield "quest_trust_backward", (t.w, t.w_mask, 64), dict(out=t.out_w)
    yield "quest_trust_backward", (t.w, None, 64), dict(out=t.w)
    yield "quest_trust_backward_pair", (t.x, t.mask, t.w, t.w_mask, 32), dict(out_x=t.out, out_w=t.out_w)
    yield "quest_trust_backward_pair", (t.x, None, t.w, None, 32), dict(out_x=t.out, out_w=t.out_w)
    for which in (0, 1):
        yield "quest_grad_gemm", (which, t.dy, t.codes, t.scales, 3, 64, 128, 192), dict(out=t.out, workspace=t.scratch)
        yield "quest_grad_gemm_fp4", (which, t.dy, t.codes, t.scales, 64, 128, 192), dict(out=t.out)
    yield "quest_weight_only_gemm", (t.x, t.w_codes, t.w_scales, 4), dict(y=t.y, workspace=t.scratch)
    yield "quest_weight_only_gemm", (t.x, t.w_codes, t.w_scales, 1), dict(y=t.y)


@pytest.fixture
def record(monkeypatch):
    """The library replaced by stand-ins for the entry points; what they were called with, in order."""
    seen, keep = [], {}
    real = q.load()
    def entry(name):
        of = getattr(real, name)
        def called(*args):
            seen.append((name, args))
            return record.status
        return ctypes.CFUNCTYPE(ctypes.c_int, *of.argtypes)(called)
    keep.update({name: entry(name) for name in q._NATIVE})
    from paper_2502_05003_amd import quest_python
    native = quest_python.Calls(*(ctypes.cast(f, ctypes.c_void_p).value for f in keep.values()))
    refuses = types.SimpleNamespace(**{name: lambda *args: None for name in dir(native) if not name.startswith("_")})
    # (keep: `native` holds addresses only, the stand-ins have to outlive what a test takes out of the library)
    record = types.SimpleNamespace(seen=seen, status=0, native=native, refuses=refuses, keep=keep)
    library = types.SimpleNamespace(calls=native, quest_status_string=real.quest_status_string, **keep)
    record.library = library
    monkeypatch.setattr(q, "_lib", library)
    monkeypatch.setattr(q, "_stream", lambda: 0x7fff_1234_5678)
    return record


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_both_ways_pass_the_same_arguments(record, dtype):
    named = set()
    for name, args, kwargs in calls(tensors(dtype)):
        record.library.calls = record.native
        assert getattr(q, name)(*args, **kwargs) is None
        record.library.calls = record.refuses
        getattr(q, name)(*args, **kwargs)
        native, general = record.seen[-2:]
        assert native[0] == general[0] == name and native[1] == general[1], name
        assert len(record.seen) % 2 == 0
        named.add(name)
    assert named == set(q._NATIVE)


def test_plain_calls_are_native_ones(record):
    """Nothing of the general way is reached."""
    for name in q._NATIVE:
        setattr(record.library, name, None)
    gc.collect()
    for name, args, kwargs in calls(tensors()):
        getattr(q, name)(*args, **kwargs)
    assert record.seen


def test_other_arguments_take_the_general_way(record):
    """Subclasses, an active torch-function mode, numbers of other types or sizes: the native method returns None."""
    t = tensors()
    native = record.native.hadamard_quantize
    plain = [t.x, 64, 4, 0.0, -1.0, t.codes, t.scales, None, None, lambda: 0]
    assert native(*plain) == 0 and len(record.seen) == 1
    for at, value in ((0, t.x.as_subclass(Subclass)), (0, t.x[0]), (0, t.x.half()), (0, None), (0, 3),
                      (1, 64.0), (1, True), (1, 1 << 31), (1, np.int64(64)), (1, 1 << 70), (3, 1), (3, np.float32(1)),
                      (5, None), (5, t.codes.numpy()), (7, t.mask.as_subclass(Subclass))):
        assert native(*plain[:at], value, *plain[at + 1:]) is None, (at, value)
    assert native(*plain[:-1]) is None
    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))
    with Mode():
        assert native(*plain) is None
    assert len(record.seen) == 1
    q.quest_hadamard_quantize(t.x.as_subclass(Subclass), 64, 4, 1, codes=t.codes, scales=t.scales)   # alpha: an int
    assert record.seen[-1][1][7] == 1.0 and record.seen[-1][1][0] == t.x.data_ptr()


def test_errors_are_those_of_the_general_way(record):
    t = tensors()
    with pytest.raises(TypeError):
        q.quest_hadamard_quantize(t.x.half(), 64, 4, codes=t.codes, scales=t.scales)
    with pytest.raises(TypeError):
        q.quest_trust_backward(t.w, None, 64, out=t.w.half())
    with pytest.raises(ValueError):
        q.quest_hadamard_quantize(t.x[0], 64, 4, codes=t.codes, scales=t.scales)
    outputs = dict(x_codes=t.codes, x_scales=t.scales, w_codes=t.w_codes, w_scales=t.w_scales)
    for w in (t.w.float(), t.w[:, :64]):
        with pytest.raises(ValueError):
            q.quest_hadamard_quantize_pair(t.x, w, 64, 4, **outputs)
    with pytest.raises(ValueError):
        q.quest_trust_backward_pair(t.x, None, t.w, None, 64, out_x=t.out, out_w=t.w)
    assert not record.seen
    record.status = 4
    with pytest.raises(q.QuestError) as error:
        q.quest_hadamard_quantize(t.x, 64, 4, codes=t.codes, scales=t.scales)
    assert error.value.status == 4


def test_a_stream_that_cannot_be_asked_for_raises(record, monkeypatch):
    def fails():
        raise RuntimeError("no device")
    monkeypatch.setattr(q, "_stream", fails)
    t = tensors()
    with pytest.raises(RuntimeError, match="no device"):
        q.quest_hadamard_quantize(t.x, 64, 4, codes=t.codes, scales=t.scales)
    assert not record.seen


@pytest.mark.parametrize("module", [None, types.SimpleNamespace(Calls=None),
                                    types.SimpleNamespace(Calls=None, TORCH_BUILD="2.0.0 0123abc")])
def test_without_a_native_module_that_fits_calls_take_the_general_way(module, record, monkeypatch):
    """None at all, one that does not say what it was built for, and one for another torch."""
    if module is None:
        monkeypatch.delattr(package, "quest_python", raising=False)
    else:
        monkeypatch.setattr(package, "quest_python", module, raising=False)
    monkeypatch.setitem(sys.modules, package.__name__ + ".quest_python", module)
    monkeypatch.setattr(q, "_lib", None)
    with pytest.warns(RuntimeWarning, match="g.build()"):
        assert q.quest_alpha_star(4) > 2
    record.library.calls = q.load().calls
    monkeypatch.setattr(q, "_lib", record.library)
    for name, args, kwargs in calls(tensors()):
        getattr(q, name)(*args, **kwargs)
        assert record.seen[-1][0] == name


def test_the_native_module_says_what_it_was_built_for():
    from paper_2502_05003_amd import quest_python
    assert quest_python.__file__ == build.PYTHON_LIB and build.PYTHON_LIB.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    assert quest_python.TORCH_BUILD == q.torch_build() and torch.__version__ in q.torch_build()


@pytest.mark.parametrize("compiler", ["false", "/nowhere/g++"])
def test_a_build_without_a_host_compiler_goes_on_without_the_native_module(compiler, tmp_path, monkeypatch, capsys):
    old = tmp_path / "quest_python.so"
    old.write_bytes(b"of another build")
    monkeypatch.setattr(build, "PYTHON_LIB", str(old))
    monkeypatch.setenv("CXX", compiler)
    assert not build.build_python_calls() and not old.exists()
    assert "was not built" in capsys.readouterr().out


# positional parameters; keyword-only ones; "name=value": with a default
SIGNATURES = {
    "quest_hadamard_quantize": ("x had_block bits alpha=0.0 outer_trust=-1.0", "codes scales mask=None xh_out=None"),
    "quest_hadamard_quantize_pair": ("x w had_block bits alpha=0.0 outer_trust=-1.0",
                                     "x_codes x_scales w_codes w_scales x_mask=None w_mask=None"),
    "quest_hadamard_quantize_absmax": ("x had_block bits", "codes scales mask=None xh_out=None"),
    "quest_hadamard_quantize_fp4": ("x had_block alpha=0.0", "codes scales mask=None xh_out=None"),
    "quest_hadamard_quantize_fp4_pair": ("x w had_block alpha=0.0",
                                         "x_codes x_scales w_codes w_scales x_mask=None w_mask=None"),
    "quest_lowbit_gemm": ("a_codes a_scales b_codes b_scales K bits", "y acc_out=None workspace=None"),
    "quest_lowbit_gemm_static": ("a_codes a_scales b_codes b_scales K bits", "y acc_out=None"),
    "quest_lowbit_gemm_fp4": ("a_codes a_scales b_codes b_scales K", "y acc_out=None"),
    "quest_trust_backward": ("g mask had_block", "out"),
    "quest_trust_backward_pair": ("g_x mask_x g_w mask_w had_block", "out_x out_w"),
    "quest_grad_gemm": ("which dy q_codes q_scales bits M N K", "out workspace=None"),
    "quest_grad_gemm_fp4": ("which dy q_codes q_scales M N K", "out workspace=None"),
    "quest_weight_only_gemm": ("x w_codes w_scales bits", "y workspace=None"),
}


def test_signatures():
    """Names, kinds and defaults that callers use, of every call of the path."""
    assert set(q._NATIVE) < set(SIGNATURES)
    for name, expected in SIGNATURES.items():
        kinds = {inspect.Parameter.POSITIONAL_OR_KEYWORD: [], inspect.Parameter.KEYWORD_ONLY: []}
        for p in inspect.signature(getattr(q, name)).parameters.values():
            kinds[p.kind].append(p.name if p.default is p.empty else f"{p.name}={p.default}")
        assert tuple(" ".join(names) for names in kinds.values()) == expected, name


def test_defaults_that_reach_the_library(record):
    """alpha 0: the built-in clip; outer trust -1: the paper's mask."""
    t = tensors()
    pair = dict(x_codes=t.codes, x_scales=t.scales, w_codes=t.w_codes, w_scales=t.w_scales)
    for library_calls in (record.native, record.refuses):
        record.library.calls = library_calls
        q.quest_hadamard_quantize(t.x, 64, 4, codes=t.codes, scales=t.scales)
        assert record.seen[-1][1][7:9] == (0.0, -1.0)
        q.quest_hadamard_quantize_pair(t.x, t.w, 64, 4, **pair)
        assert record.seen[-1][1][16:18] == (0.0, -1.0)
        q.quest_hadamard_quantize_fp4(t.x, 64, codes=t.codes, scales=t.scales)
        assert record.seen[-1][1][6] == 0.0
        q.quest_hadamard_quantize_fp4_pair(t.x, t.w, 64, **pair)
        assert record.seen[-1][1][15] == 0.0
