"""The extension module of the Python calls: what reaches the C ABI, by position and by name, and what is refused."""
import ctypes
import inspect
import os
import shutil
import subprocess
import sys
import sysconfig
import types

import numpy as np
import pytest

pytest.importorskip("torch")                               # (before the library: both then use one HIP runtime)

from paper_2411_00915_amd import _calls, calls_ctypes
from paper_2411_00915_amd import binding as B

P, I32, I64, F, Z = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_float, ctypes.c_size_t
ABI = {"lora_plan_upload": [P, P], "lora_shrink": [P, P, I64, P, P, P], "lora_expand": [P, P, P, P, I64, F, P],
       "lora_delta": [P, P, I64, P, P, P, P, I64, F, P], "lora_delta_static": [P, P, I64, P, P, P, I64, F, P],
       "lora_base_gemm": [I32, I32, I32, I32, P, I64, P, I64, P, I64, P],
       "lora_fused_forward": [P, P, I64, P, I64, P, P, P, I64, P, Z, P],
       "lora_merge": [I32, I32, I32, I32, F, I32, I32, P, I64, P, P, P]}


class Buffer:
    def data_ptr(self):
        return 0xfedcba9876543210


@pytest.fixture
def seen():
    """(name, arguments) of the last call that reached a stand-in for the library"""
    last, keep = [], []
    for name, arguments in ABI.items():
        keep.append(ctypes.CFUNCTYPE(ctypes.c_int, *arguments)(lambda *a, name=name: (last.__setitem__(slice(None), [name, a]), last_status[0])[1]))
    last_status = [0]
    _calls.bind(B._check, B._first_stream, *(B._address(f) for f in keep))
    yield last, last_status
    _calls.bind(B._check, B._first_stream, *(B._address(getattr(B._lib, name)) for name in ABI))


@pytest.mark.parametrize("name", list(ABI))
def test_arguments_reach_the_abi_by_position_and_by_name(name, seen):
    last, status = seen
    function = getattr(B, name)
    parameters = inspect.signature(function).parameters
    plan = types.SimpleNamespace(handle=0x1000)
    values, expected = {}, []
    for i, (p, info) in enumerate(parameters.items()):
        if p == "plan":
            values[p], e = plan, 0x1000
        elif p == "beta" or p == "scale":
            values[p], e = np.float64(0.25), 0.25
        elif p == "stream":
            values[p], e = 0x77, 0x77
        elif p in ("x", "v", "y", "Wt", "workspace") or p.startswith("d_"):
            values[p], e = (Buffer(), 0xfedcba9876543210) if i % 2 else (4096 * i, 4096 * i)
        else:
            values[p], e = np.int64(40 + i), 40 + i
        expected.append(e)
    if name == "lora_merge":                                # (variant comes before the addresses in the C call)
        expected.insert(6, expected.pop(10))
    function(*values.values())
    assert last[0] == name and list(last[1]) == expected
    last[:] = []
    function(**dict(reversed(values.items())))
    assert last[0] == name and list(last[1]) == expected
    # what has a default may be left out, nothing else
    required = [p for p, info in parameters.items() if info.default is inspect.Parameter.empty]
    function(**{p: values[p] for p in required}, stream=5)
    for default, i in ((1.0, "beta"), (B.LORA_VARIANT_AUTO, "variant")):
        if i in parameters:
            assert last[1][ABI[name].index(F) if i == "beta" else 6] == default == parameters[i].default
    last[:] = []
    for wrong in ([values[p] for p in required][:-1], [*values.values(), 0]):
        with pytest.raises(TypeError):
            function(*wrong)
    with pytest.raises(TypeError):
        function(*values.values(), stream=0)
    with pytest.raises(TypeError):
        function(**values, other=0)
    for p in required:                                      # neither an address nor a number nor a plan
        with pytest.raises((AttributeError, TypeError)):
            function(**{**values, p: object()})
    assert not last
    status[0] = B.LORA_ERR_WORKSPACE
    with pytest.raises(B.LoraError, match=f"{name}: workspace") as e:
        function(**values)
    assert e.value.status == B.LORA_ERR_WORKSPACE


def test_no_address_and_no_plan_are_null(seen):
    last, _ = seen
    B.lora_shrink(B.Plan(None, None), None, 8, None, None, 0)
    assert last[1] == (None, None, 8, None, None, None)


@pytest.mark.parametrize("private", [True, False])
def test_no_stream_is_the_current_one_with_and_without_torchs_private_functions(private, seen, monkeypatch):
    import torch
    current = {0: 0x50, 1: 0x60}
    device = [0]
    monkeypatch.setattr(torch.cuda, "current_device", lambda: device[0])
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d=None: types.SimpleNamespace(cuda_stream=current[device[0] if d is None else d]))
    for name, stand_in in (("_cuda_getDevice", lambda: device[0]), ("_cuda_getCurrentRawStream", lambda d: current[d])):
        if private:
            monkeypatch.setattr(torch._C, name, stand_in, raising=False)
        else:
            monkeypatch.delattr(torch._C, name, raising=False)
    last, _ = seen
    plan = types.SimpleNamespace(handle=0x1000)
    for device[0], want in ((0, 0x50), (0, 0x50), (1, 0x60), (0, 0x50)):       # (the first call initialises torch's side)
        B.lora_plan_upload(plan)
        assert last[1] == (0x1000, want)
        B.lora_plan_upload(plan, stream=None)
        assert last[1] == (0x1000, want)
    current[0] = 0x70
    B.lora_plan_upload(plan)
    assert last[1] == (0x1000, 0x70)


def _import_binding(tmp_path, calls, library, code):
    """Runs `code` after the import of binding from a copy of the package's Python files, with the extension module or without"""
    here = os.path.dirname(B.__file__)
    copy = tmp_path / "paper_2411_00915_amd"
    copy.mkdir()
    for name in os.listdir(here):
        if name.endswith(".py") or (calls and name.startswith("_calls.")):
            shutil.copy(os.path.join(here, name), copy / name)
    if not library:
        os.symlink(B.LIB_PATH, copy / "liblora_amd.so")
    env = {k: v for k, v in os.environ.items() if k != "LORA_AMD_LIBRARY"}
    if library:
        env["LORA_AMD_LIBRARY"] = B.LIB_PATH
    return subprocess.run([sys.executable, "-c", "import torch\nfrom paper_2411_00915_amd import binding as B\n" + code], cwd=tmp_path, env=env,
                          capture_output=True, text=True)


def test_a_library_built_elsewhere_needs_no_extension_module(tmp_path):
    """LORA_AMD_LIBRARY in a tree that has not been built: the same functions, by ctypes"""
    out = _import_binding(tmp_path, False, True, """
import inspect
plan = B.lora_plan(4, [0, 4], [0], [8], [1.0], 8, 8, B.LORA_F32)
assert B.lora_plan_query(plan)[0] == 8
for name, call in (("lora_shrink", lambda: B.lora_shrink(B.Plan(None, None), None, 8, None, None, 0)),
                   ("lora_delta", lambda: B.lora_delta(plan, None, 8, None, None, None, None, 8, 1.0, stream=0)),
                   ("lora_base_gemm", lambda: B.lora_base_gemm(-1, 8, 8, B.LORA_F32, None, 8, None, 8, None, 8, stream=0))):
    try:
        call()
    except B.LoraError as e:
        assert e.status == B.LORA_ERR_INVALID_ARG and str(e).startswith(name), e
    else:
        raise AssertionError(name)
for name in %r:
    print(name, inspect.signature(getattr(B, name)))
""" % (list(ABI),))
    assert out.returncode == 0, out.stderr
    assert out.stdout.split("\n")[:-1] == [f"{name} {inspect.signature(getattr(B, name))}" for name in ABI]


def test_a_missing_extension_module_says_how_to_build(tmp_path):
    out = _import_binding(tmp_path, False, False, "")
    assert out.returncode and "python -m paper_2411_00915_amd.build" in out.stderr.strip().split("\n")[-1]


def test_extension_module_is_named_for_its_interpreter(tmp_path):
    assert os.path.basename(_calls.__file__) == "_calls" + sysconfig.get_config_var("EXT_SUFFIX")
    out = _import_binding(tmp_path, True, False, "from paper_2411_00915_amd import _calls\nassert B.lora_delta is _calls.lora_delta")
    assert out.returncode == 0, out.stderr


@pytest.mark.parametrize("name", list(ABI))
def test_arguments_reach_the_abi_by_ctypes_too(name):
    """The stand-in for the extension module: every argument of every function, in place"""
    seen = []
    keep = [ctypes.CFUNCTYPE(ctypes.c_int, *arguments)(lambda *a, n=n: (seen.append((n, list(a))), 0)[1]) for n, arguments in ABI.items()]
    order = ["lora_plan_upload", "lora_shrink", "lora_expand", "lora_delta", "lora_delta_static", "lora_base_gemm", "lora_fused_forward", "lora_merge"]
    calls_ctypes.bind(B._check, None, *(B._address(keep[list(ABI).index(n)]) for n in order))
    parameters = list(inspect.signature(getattr(B, name)).parameters)
    values = [types.SimpleNamespace(handle=0x1000) if p == "plan" else 0.25 if p in ("beta", "scale") else Buffer() if p in ("x", "y") else 64 + i
              for i, p in enumerate(parameters)]
    expected = [0x1000 if p == "plan" else 0xfedcba9876543210 if p in ("x", "y") else v for p, v in zip(parameters, values)]
    if name == "lora_merge":
        expected.insert(6, expected.pop(10))
    getattr(calls_ctypes, name)(*values)
    getattr(calls_ctypes, name)(**dict(zip(parameters, values)))
    assert seen == [(name, expected)] * 2
