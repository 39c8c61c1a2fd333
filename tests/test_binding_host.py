"""The native short way of the binding on host tensors, built with tests/binding_on_host.cpp: which entry point it calls, with what, how
often, and what it does where something fails around the call."""
import ctypes
import importlib.machinery
import importlib.util
import os
import subprocess

import pytest

import paper_2311_09550_amd as w4a8

HERE = os.path.dirname(os.path.abspath(__file__))
M, N, K = 3, 96, 256
ENTRIES = {"w4a8_quantize_act": 6, "w4a8_quantize_act_strided": 7, "w4a8_gemm": 11, "w4a8_gemm_tiled": 9, "w4a8_gemm_tiled_splitk": 13,
           "w8a8_gemm_tiled": 11, "w4a8_linear_tiled_fp16": 10, "w4a8_quantize_weights": 6, "w4a8_tile_weights": 5}


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    pytest.importorskip("torch")
    from paper_2311_09550_amd import build
    path = str(tmp_path_factory.mktemp("binding") / "binding_on_host.so")
    command = build.binding_command()
    command[command.index(build.BINDING)] = path
    command[command.index(os.path.join(build.CSRC, "binding.cpp"))] = os.path.join(HERE, "binding_on_host.cpp")
    subprocess.run([c for c in command if c != "-O2"] + ["-O1"], check=True)
    loader = importlib.machinery.ExtensionFileLoader("binding_on_host", path)
    module = importlib.util.module_from_spec(importlib.util.spec_from_loader("binding_on_host", loader))
    loader.exec_module(module)
    return module, ctypes.c_int.in_dll(ctypes.CDLL(path), "wraps_until_failure")


class Refused(Exception):
    pass


@pytest.fixture
def short(built):
    """(the short way, the launches it made, a switch: the code that entry points return)"""
    module, failure = built
    launches, code, lib = [], [0], w4a8.lib()

    def entry(name, nargs):
        def called(*args):
            launches.append((name, args))
            return code[0]
        return ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_ssize_t] * nargs)(called)
    kept = {name: entry(name, n) for name, n in ENTRIES.items()}
    address = {name: ctypes.cast(f, ctypes.c_void_p).value for name, f in kept.items()}
    for name in ("w4a8_tiled_weight_bytes", "w8a8_tiled_weight_bytes"):
        address[name] = ctypes.cast(getattr(lib, name), ctypes.c_void_p).value

    def check(c):
        raise Refused(c)
    module.bind(check, address)
    failure.value = 0
    yield module, launches, code, failure
    failure.value = 0
    del kept


def _calls():
    """name -> (entry point, arguments without outputs, number of outputs, sizes that the entry is told, in its order)"""
    import torch as t
    x, xq, s_a, s_w = t.zeros((M, K), dtype=t.float16), t.zeros((M, K), dtype=t.int8), t.zeros(M), t.zeros(N)
    wp, wt, wt8, ws = (t.zeros(n, dtype=t.uint8) for n in ((N, K // 2), N * K // 2, N * K, 1 << 12))
    w = t.zeros((N, K), dtype=t.float16)
    return {"quantize_act": ("w4a8_quantize_act", (x,), 2, (M, K)),
            "quantize_act_strided": ("w4a8_quantize_act_strided", (t.zeros((M, K + 32), dtype=t.float16)[:, 32:],), 2, (M, K)),
            "gemm": ("w4a8_gemm", (xq, s_a, wp, s_w), 1, (M, N, K)),
            "gemm_tiled": ("w4a8_gemm_tiled", (xq, s_a, wt, s_w), 1, (M, N, K)),
            "gemm_tiled_splitk": ("w4a8_gemm_tiled_splitk", (xq, s_a, wt, s_w, ws), 1, (M, N, K)),
            "w8a8_gemm_tiled": ("w8a8_gemm_tiled", (xq, s_a, wt8, s_w), 1, (M, N, K)),
            "linear_tiled_fp16": ("w4a8_linear_tiled_fp16", (x, wt, s_w), 2, (M, N, K)),
            "quantize_weights": ("w4a8_quantize_weights", (w,), 2, (N, K)),
            "tile_weights": ("w4a8_tile_weights", (wp,), 1, (N, K))}


NAMES = ["quantize_act", "quantize_act_strided", "gemm", "gemm_tiled", "gemm_tiled_splitk", "w8a8_gemm_tiled", "linear_tiled_fp16",
         "quantize_weights", "tile_weights"]


@pytest.mark.parametrize("name", NAMES)
def test_one_launch_with_the_sizes_and_pointers_of_its_tensors(short, name):
    module, launches, _, _ = short
    entry, args, outs, sizes = _calls()[name]
    result = getattr(module, name)(*args, *[None] * outs)
    results = result if isinstance(result, tuple) else (result,)
    (called, values), = launches
    assert called == entry
    at = [i for i in range(len(values) - len(sizes) + 1) if values[i:i + len(sizes)] == sizes]
    assert at, (values, sizes)
    for t in (*args, *results):
        assert t.data_ptr() in values
    again = getattr(module, name)(*args, *results, *[None] * (outs - len(results)))
    assert all(a is b for a, b in zip(again if isinstance(again, tuple) else (again,), results)) and len(launches) == 2


@pytest.mark.parametrize("name", NAMES)
def test_an_output_that_cannot_be_wrapped_is_found_out_before_the_launch(short, name):
    module, launches, _, failure = short
    _, args, outs, _ = _calls()[name]
    wrapped = 1 if name == "linear_tiled_fp16" else outs  # its scales are written only on request
    for nth in range(1, wrapped + 1):
        failure.value = nth
        assert getattr(module, name)(*args, *[None] * outs) is None
        assert failure.value == 0 and not launches, "None says that nothing was launched"


@pytest.mark.parametrize("name", NAMES)
def test_an_error_code_raises_once(short, name):
    module, launches, code, _ = short
    _, args, outs, _ = _calls()[name]
    code[0] = -4
    with pytest.raises(Refused) as e:
        getattr(module, name)(*args, *[None] * outs)
    assert e.value.args == (-4,) and len(launches) == 1


@pytest.mark.parametrize("name", NAMES)
def test_what_is_too_small_is_not_served(short, name):
    module, launches, _, _ = short
    _, args, outs, _ = _calls()[name]
    given = getattr(module, name)(*args, *[None] * outs)
    given = list(given if isinstance(given, tuple) else (given,))
    launches.clear()
    for i, t in enumerate(given):
        outputs = [None] * outs
        outputs[i] = t[:-1]
        assert getattr(module, name)(*args, *outputs) is None
    for i, t in enumerate(args):
        if i > 0 and name != "linear_tiled_fp16" and not (name == "gemm_tiled_splitk" and i == 4):
            assert getattr(module, name)(*(t[:-40] if i == j else u for j, u in enumerate(args)), *[None] * outs) is None
    assert not launches
