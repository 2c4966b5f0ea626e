"""The native forms of the binding's calls against the Python functions they stand for, without a GPU: the same refusals and the same
library errors for the same arguments, whatever way they are given.  Every call below fails on the host, before a launch."""
import ctypes
import inspect
import os
import pickle
import shutil
import subprocess
import sys
import weakref

import numpy as np
import pytest
import torch

import paper_2412_00876_amd.binding as b
from paper_2412_00876_amd import _calls

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="calls with host pointers: only where nothing can be launched")
NAMES = [n for n in b.EXPORTS if hasattr(b, n) and "stream" in inspect.signature(getattr(b, n)).parameters]


@pytest.fixture(autouse=True)
def no_device(monkeypatch):
    """Both forms believe that stream 0 is current."""
    monkeypatch.setattr(b, "_stream", lambda stream: None if stream is None else getattr(stream, "cuda_stream", stream) or None)
    _calls.init(b.KVCache, b.Predictor, b._check, lambda: 0, lambda: 0, lambda device: 0)
    yield
    _calls.init(b.KVCache, b.Predictor, b._check, torch.cuda.current_device, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)


def _outcome(f, *args, **kw):
    try:
        return "returned", f(*args, **kw)
    except Exception as e:  # noqa: BLE001
        return type(e), getattr(e, "status", None), str(e)


def _both(name, *args, **kw):
    f = getattr(b, name)
    native, python = _outcome(f, *args, **kw), _outcome(f.__wrapped__, *args, **kw)
    assert native == python, (name, native, python)
    return native


def _cache(Dh=64, H=2, dtype=torch.bfloat16):
    return b.KVCache(torch.zeros(4, 2, H, 16, Dh, dtype=dtype), torch.zeros(2, 2, dtype=torch.int32), torch.zeros(2, dtype=torch.int32))


def _valid(name):
    """Arguments of every kind in their places, and a dtype or head size that the library refuses."""
    t = torch.zeros(64)
    special = dict(cache=_cache(), p=b.Predictor(64, {}, []), workspace=torch.zeros(512, dtype=torch.uint8), dtype=9, scale=0.1, threshold=0.0,
                   keep_ratio=0.5, rope_base=1e4, eps=1e-5, mode=0, act=0, B=1, M=1, H=2, Dh=64, d=64, dh=16, K=64, N=64, F=64, rows=1, sumN=1,
                   ldx=64, ldy=64)
    out = []
    for q in inspect.signature(getattr(b, name)).parameters:
        if q == "stream":
            continue
        out.append(t if name.endswith(("_attn", "_compact")) and q in ("K", "V") else special.get(q, t))
    if name.startswith("dllava_decode"):
        out[[q for q in inspect.signature(getattr(b, name)).parameters].index("threshold")] = float("nan")
    return out


def test_every_call_with_a_stream_is_native():
    assert len(NAMES) == 19
    for n in NAMES:
        f = getattr(b, n)
        assert type(f).__name__ == "Call" and f.__name__ == n and inspect.isfunction(f.__wrapped__)
        assert inspect.signature(f) == inspect.signature(f.__wrapped__)
        assert list(inspect.signature(f).parameters)[-1] == "stream"
        assert pickle.loads(pickle.dumps(f)) is f


@pytest.mark.parametrize("name", NAMES)
def test_the_library_sees_the_same_arguments(name):
    """The library's own refusal, with the offending value in its message: positional, by keyword, mixed, with an explicit stream."""
    args = _valid(name)
    names = list(inspect.signature(getattr(b, name)).parameters)
    first = _both(name, *args)
    assert first[0] is b.DllavaError, first
    for i in range(len(args)):                    # a library check that names the value, wherever one does
        if isinstance(args[i], int):
            for v in (-3, 7, 1 << 33, True, np.int64(5)):
                _both(name, *args[:i], v, *args[i + 1:])
        if isinstance(args[i], float):
            for v in (-1.0, 2, float("inf"), np.float64(0.25), np.float32(-2.0), 10 ** 400):
                _both(name, *args[:i], v, *args[i + 1:])
        if isinstance(args[i], (torch.Tensor, b.KVCache)):
            for v in (None, args[i][1:] if isinstance(args[i], torch.Tensor) and len(args[i]) > 1 else None):
                _both(name, *args[:i], v, *args[i + 1:])
    assert _both(name, **dict(zip(names, args))) == first
    assert _both(name, *args[:2], **dict(zip(names[2:], args[2:]))) == first
    for stream in (None, 0, type("S", (), {"cuda_stream": 0})()):
        assert _both(name, *args, stream) == first and _both(name, *args, stream=stream) == first


@pytest.mark.parametrize("name", NAMES)
def test_what_is_refused_is_refused_alike(name):
    args = _valid(name)
    names = list(inspect.signature(getattr(b, name)).parameters)
    assert _both(name)[0] is TypeError and _both(name, *args[:-1])[0] is TypeError
    assert _both(name, *args, None, None)[0] is TypeError and _both(name, *args, nothing=1)[0] is TypeError
    assert _both(name, *args, **{names[0]: args[0]})[0] is TypeError
    for i, a in enumerate(args):
        for v in ("text", 1.5, object(), torch.zeros(4, device="meta"), torch.nn.Parameter(torch.zeros(64)), type("T", (torch.Tensor,), {})(64), [1]):
            if isinstance(a, float) and isinstance(v, float):
                continue
            _both(name, *args[:i], v, *args[i + 1:])
        if isinstance(a, int):
            assert _both(name, *args[:i], 1.0, *args[i + 1:])[0] is ctypes.ArgumentError


def test_without_a_device_the_python_function_says_so(monkeypatch):
    monkeypatch.undo()  # the binding's own _stream
    _calls.init(b.KVCache, b.Predictor, b._check, torch.cuda.current_device, torch.cuda.current_device, torch._C._cuda_getCurrentRawStream)
    with pytest.raises((RuntimeError, AssertionError)) as e:
        b.dllava_rope(torch.zeros(64), torch.zeros(1, dtype=torch.int32), 1, 1, 64, 1e4, b.BF16)
    assert not isinstance(e.value, b.DllavaError) and any(f.name == "_stream" for f in e.traceback)


_TWO = """
import importlib, sys
sys.path.insert(0, sys.argv[1])
a, b = importlib.import_module("one.binding"), importlib.import_module("two.binding")
import torch
for m in (a, b):
    for f in (m.dllava_rope, m.dllava_rope.__wrapped__):
        try:
            f(torch.zeros(64), torch.zeros(1, dtype=torch.int32), 1, 1, 63, 1e4, m.BF16)
        except m.DllavaError as e:
            print(e)
"""


def _copy_package(to, name, calls=True):
    pkg = os.path.dirname(os.path.abspath(b.__file__))
    os.makedirs(to / name / "lib")
    for f in ("__init__.py", "binding.py", "lib/libdllava.so") + (("_calls.so",) if calls else ()):
        shutil.copy(os.path.join(pkg, f), to / name / f)


def _python(program, *args):
    r = subprocess.run([sys.executable, "-c", program, *map(str, args)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
    return r.stdout.splitlines(), r.stderr


def test_two_copies_of_the_library_in_one_process(tmp_path):
    """Each copy of the package calls the library beside it: the refusal's text comes from the library that refused.  (The stream is
    read before the call: without a device the Python form's own refusal would come first, so a stream-less stand-in is used.)"""
    for name in ("one", "two"):
        _copy_package(tmp_path, name)
    program = _TWO.replace("import torch\n", "import torch\nfor m in (a, b):\n    m._calls = importlib.import_module(m.__package__ + '._calls')\n"
                           "    m._calls.init(m.KVCache, m.Predictor, m._check, lambda: 0, lambda: 0, lambda device: 0)\n"
                           "    torch.cuda.current_device = lambda: 0\n    torch._C._cuda_getCurrentRawStream = lambda device: 0\n")
    lines, _ = _python(program, tmp_path)
    assert len(lines) == 4 and len(set(lines)) == 1 and "63" in lines[0], lines


def test_another_library_or_stream_is_used(monkeypatch):
    """The binding's _lib, one of its functions or its _stream replaced: the native form follows, as the Python form does."""
    args = _valid("dllava_rope")
    seen = []

    class Lib:
        def dllava_rope(self, *a):
            seen.append(a)
            return 0

    real = b._lib
    for replace in (lambda: monkeypatch.setattr(b, "_lib", Lib()), lambda: monkeypatch.setattr(b._lib, "dllava_rope", Lib().dllava_rope)):
        replace()
        b.dllava_rope(*args), b.dllava_rope.__wrapped__(*args)
        assert len(seen) == 2 and seen[0] == seen[1]
        seen.clear()
        monkeypatch.setattr(b, "_lib", real)
    monkeypatch.undo()
    for stream, outcome in ((lambda s: 1 // 0, ZeroDivisionError), (lambda s: None, b.DllavaError), (lambda s: object(), ctypes.ArgumentError)):
        monkeypatch.setattr(b, "_stream", stream)
        assert _both("dllava_rope", *args)[0] is outcome


@pytest.mark.parametrize("state", ["missing", "broken", "another torch", "an older one"])
def test_the_package_does_without_the_native_forms(tmp_path, state):
    """Only libdllava.so is needed: the calls are then the ctypes forms, and the import says so."""
    _copy_package(tmp_path, "one", calls=state == "another torch")
    if state == "broken":
        (tmp_path / "one" / "_calls.so").write_bytes(b"not a library")
    if state == "an older one":             # without the name of its torch, and with other functions
        (tmp_path / "one" / "_calls.py").write_text("def init(): pass\n")
    other = "torch.version.git_version = 'another'\n" if state == "another torch" else ""
    lines, err = _python("import sys, torch\n" + other + "sys.path.insert(0, sys.argv[1])\nimport one.binding as m\nimport inspect\n"
                         "print(inspect.isfunction(m.dllava_rope), m.dllava_version())\n"
                         "try:\n    m.dllava_rope(torch.zeros(64), torch.zeros(1, dtype=torch.int32), 1, 1, 63, 1e4, m.BF16, 0)\n"
                         "except m.DllavaError as e:\n    print(e)\n", tmp_path)
    assert lines[0].startswith("True ") and "63" in lines[1] and "RuntimeWarning" in err, (lines, err)


def test_the_library_is_built_without_a_host_compiler(tmp_path, monkeypatch):
    from paper_2412_00876_amd import build
    stale = tmp_path / "_calls.so"
    stale.write_bytes(b"an older one")
    monkeypatch.setattr(build, "CALLS", str(stale))
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    for compiler in ("false", "no-such-compiler"):
        monkeypatch.setenv("CXX", compiler)
        assert compiler in build.build_calls() and not stale.exists()


def test_used_as_functions_are():
    """Weak references and methods."""
    f = b.dllava_rope
    assert weakref.ref(f)() is f and weakref.WeakKeyDictionary({f: 1})[f] == 1

    class Layer:
        run = f
        plain = f.__wrapped__

    x = Layer()
    assert Layer.run is f and x.run.__self__ is x and x.run.__func__ is f
    args = _valid("dllava_rope")[1:]
    assert _outcome(x.run, *args) == _outcome(x.plain, *args)
