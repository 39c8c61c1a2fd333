"""The native short way of the binding's calls without a GPU: it serves nothing that is not on the device, and the checks written out
in Python answer as they do without it."""
import copy
import ctypes
import functools
import gc
import weakref

import pytest

import paper_2311_09550_amd as w4a8


@pytest.fixture(scope="module")
def short():
    pytest.importorskip("torch")
    w4a8.lib()
    return w4a8._short


def _calls(t):
    x, xq, s = t.zeros((2, 64), dtype=t.float16), t.zeros((2, 64), dtype=t.int8), t.zeros(2)
    wp, wt, wt8, sw = t.zeros((32, 32), dtype=t.uint8), t.zeros(2048, dtype=t.uint8), t.zeros(4096, dtype=t.uint8), t.zeros(32)
    return [("quantize_act", w4a8.w4a8_quantize_act, (x,), (x, None, None)),
            ("quantize_act_strided", w4a8.w4a8_quantize_act_strided, (x,), (x, None, None)),
            ("gemm", w4a8.w4a8_gemm, (xq, s, wp, sw, None, wt), (xq, s, wp, sw, None)),
            ("gemm_tiled", w4a8.w4a8_gemm_tiled, (xq, s, wt, sw), (xq, s, wt, sw, None)),
            ("gemm_tiled_splitk", w4a8.w4a8_gemm_tiled_splitk, (xq, s, wt, sw, 0, 0, wt), (xq, s, wt, sw, wt, None)),
            ("w8a8_gemm_tiled", w4a8.w8a8_gemm_tiled, (xq, s, wt8, sw), (xq, s, wt8, sw, None)),
            ("linear_tiled_fp16", w4a8.w4a8_linear_tiled_fp16, (x, wt, sw), (x, wt, sw, None, None))]


@pytest.mark.parametrize("i", range(7))
def test_host_tensors_are_refused_by_the_checks_in_python(short, i, monkeypatch):
    import torch
    name, function, args, short_args = _calls(torch)[i]
    assert getattr(short, name)(*short_args) is None
    with pytest.raises(TypeError) as with_short:
        function(*args)
    monkeypatch.setattr(w4a8, "_short", w4a8._NothingLoaded())
    with pytest.raises(TypeError) as without:
        function(*args)
    assert str(with_short.value) == str(without.value)


@pytest.mark.parametrize("args", [(), (None,), (1, 2, 3), ("a", None, None), (None,) * 3, (None,) * 5, (object(),) * 6])
def test_what_is_no_tensor_is_not_served(short, args):
    for name in ("quantize_act", "quantize_act_strided", "gemm", "gemm_tiled", "gemm_tiled_splitk", "w8a8_gemm_tiled", "linear_tiled_fp16"):
        assert getattr(short, name)(*args) is None


@pytest.mark.parametrize("how", ["missing", "unreadable", "another torch"])
def test_without_the_short_way_calls_go_by_ctypes(short, monkeypatch, tmp_path, how):
    """A missing, broken or foreign _binding.so takes no call away: the library loads, says so once, and bound_call still binds."""
    import torch
    if how != "another torch":
        path = tmp_path / "_binding.so"
        if how == "unreadable":
            path.write_bytes(b"no library")
        monkeypatch.setattr(w4a8, "BINDING_PATH", str(path))
    else:
        monkeypatch.setattr(torch, "__version__", "1.0")
    monkeypatch.setattr(w4a8, "_lib", None)
    monkeypatch.setattr(w4a8, "_short", w4a8._NothingLoaded())
    with pytest.warns(RuntimeWarning, match="_binding.so"):
        assert w4a8.lib().w4a8_version() > 0
    assert isinstance(w4a8._short, w4a8._NothingLoaded) and w4a8._short.quantize_act(None, None, None) is None
    with pytest.raises(TypeError):
        w4a8.w4a8_quantize_act(torch.zeros((2, 64), dtype=torch.float16))
    assert w4a8.w4a8_tiled_weight_bytes(32, 128) == 2048


def test_the_library_is_built_without_torch(monkeypatch, tmp_path):
    """hipcc is all that the C interface needs: no torch, no C++ compiler of the host, no CPython headers."""
    import subprocess
    import sys

    from paper_2311_09550_amd import build
    ran = []

    class Done:
        returncode = 0

        def communicate(self):
            return "", None
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libw4a8.so"))
    monkeypatch.setattr(build, "BINDING", str(tmp_path / "_binding.so"))
    monkeypatch.setattr(subprocess, "Popen", lambda cmd, **kw: ran.append(cmd) or Done())
    monkeypatch.setattr(subprocess, "run", lambda cmd, **kw: ran.append(cmd))
    build.build_library()
    assert any("binding.cpp" in part for cmd in ran for part in cmd) and len(ran) == len(build.SOURCES) + 2
    ran.clear()
    monkeypatch.setitem(sys.modules, "torch", None)  # as where it is not installed
    build.build_library()
    assert len(ran) == len(build.SOURCES) + 1 and all("hipcc" in cmd[0] for cmd in ran)


def test_bind_wants_every_address(short):
    with pytest.raises(KeyError):
        short.bind(w4a8._check, {})
    with pytest.raises(TypeError):
        short.bind(w4a8._check, None)


def test_a_bound_call_has_what_a_function_has(short):
    """Weak references, attributes, a name, and copies that are itself: what bound_call returned before it was native, and still returns
    where its arguments are left to ctypes."""
    class Tensor:  # stands for what is kept alive
        pass
    kept = Tensor()
    alive = weakref.ref(kept)
    address = ctypes.cast(w4a8.lib().w4a8_quantize_act, ctypes.c_void_p).value
    bound = short.bound("w4a8_quantize_act", address, (0, 0, 0, 1, 64), 0, [kept])
    assert bound is not None and callable(bound)
    assert (bound.__name__, bound.__qualname__, bound.__module__) == ("call", "bound_call.<locals>.call", "paper_2311_09550_amd")
    bound.note = "down projection"
    assert vars(bound)["note"] == bound.note
    assert copy.copy(bound) is bound and copy.deepcopy([bound])[0] is bound
    wrapped = functools.wraps(bound)(lambda: bound())
    assert wrapped.__name__ == "call" and wrapped.note == bound.note and wrapped.__wrapped__ is bound
    assert {weakref.ref(bound)} and weakref.WeakSet([bound])
    with pytest.raises(TypeError):
        type(bound)()
    bound.me = bound  # a cycle through its attributes is collected
    gone = weakref.ref(bound)
    del bound, wrapped, kept
    gc.collect()
    assert gone() is None and alive() is None
