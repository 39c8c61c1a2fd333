"""Tensors that are too small for a call raise before anything is launched.  Without a GPU: the tensors claim to be on the device, and
the library is one that counts what would have been launched."""
import pytest

import paper_2311_09550_amd as w4a8

M, N, K = 3, 96, 256


@pytest.fixture
def launches(monkeypatch):
    torch = pytest.importorskip("torch")
    real = w4a8.lib()
    seen = []

    class Counting:
        def __getattr__(self, name):
            if name.endswith("_bytes") or name == "w4a8_strerror":
                return getattr(real, name)
            return lambda *args: seen.append(name) or 0

    class OnDevice(torch.Tensor):
        __torch_function__ = torch._C._disabled_torch_function_impl
        is_cuda = True

        def get_device(self):
            return 0

    w4a8._torch()
    counting = Counting()
    monkeypatch.setattr(w4a8, "lib", lambda: counting)
    monkeypatch.setattr(w4a8, "_current_device", lambda: 0)
    monkeypatch.setattr(w4a8, "_raw_stream", lambda index: 0)
    return seen, lambda dtype, *shape: torch.zeros(shape, dtype=dtype).as_subclass(OnDevice)


def _calls(e):
    """name -> (function, arguments, those whose size follows from the others)"""
    import torch as t
    half, i8, u8, f32 = t.float16, t.int8, t.uint8, t.float32
    xq, s_a, s_w, out = e(i8, M, K), e(f32, M), e(f32, N), e(half, M, N)
    x, wt, wp, ws = e(half, M, K), e(u8, N * K // 2), e(u8, N, K // 2), e(u8, 1 << 16)
    tiled = dict(xq=xq, s_a=s_a, wt=wt, s_w=s_w, out=out)
    w, gate_up = e(half, N, K), e(half, M, 2 * N)
    rows = dict(xq=e(i8, M, K), s_a=e(f32, M))
    return {
        "quantize_act": (w4a8.w4a8_quantize_act, dict(x=x, **rows), ("xq", "s_a")),
        "quantize_act_strided": (w4a8.w4a8_quantize_act_strided, dict(x=x, **rows), ("xq", "s_a")),
        "gemm": (w4a8.w4a8_gemm, dict(xq=xq, s_a=s_a, wp=wp, s_w=s_w, out=out, ws=ws), ("s_a", "s_w", "wp", "out")),
        "gemm_acc_i32": (w4a8.w4a8_gemm_acc_i32, dict(xq=xq, wp=wp, acc=e(t.int32, M, N), ws=ws), ("acc",)),
        "gemm_tuned": (w4a8.w4a8_gemm_tuned, dict(xq=xq, s_a=s_a, wp=wp, s_w=s_w, tiling=0, out=out, ws=ws), ("s_a", "s_w", "out")),
        "gemm_tuned_tiled": (w4a8.w4a8_gemm_tuned, dict(xq=xq, s_a=s_a, wp=wt, s_w=s_w, tiling=w4a8.TILING_AUTO_TILED, out=out, ws=ws, N=N),
                             ("s_a", "s_w", "wp", "out")),
        "tile_weights": (w4a8.w4a8_tile_weights, dict(wp=wp, wt=wt), ("wt",)),
        "gemm_tiled": (w4a8.w4a8_gemm_tiled, tiled, ("s_a", "wt", "out")),
        "gemm_tiled_splitk": (w4a8.w4a8_gemm_tiled_splitk, dict(tiled, ws=ws), ("s_a", "wt", "out")),
        "gemm_tiled_splitk_static": (w4a8.w4a8_gemm_tiled_splitk_static, tiled, ("s_a", "wt", "out")),
        "gemm_tiled_unsigned": (w4a8.w4a8_gemm_tiled_unsigned, dict(xq=xq, s_a=s_a, ut=wt, s_w=s_w, N=N, out=out), ("s_a", "ut", "s_w", "out")),
        "gemm_tiled_swiglu": (w4a8.w4a8_gemm_tiled_swiglu, dict(xq=xq, s_a=s_a, wt_gu=wt, s_w_gu=s_w, h=e(half, M, N // 2)), ("s_a", "wt_gu", "h")),
        "w8a8_tile_weights": (w4a8.w8a8_tile_weights, dict(w8=e(i8, N, K), wt=e(u8, N * K)), ("wt",)),
        "w8a8_gemm_tiled": (w4a8.w8a8_gemm_tiled, dict(xq=xq, s_a=s_a, wt=e(u8, N * K), s_w=s_w, N=N, out=out), ("s_a", "wt", "s_w", "out")),
        "linear_tiled_fp16": (w4a8.w4a8_linear_tiled_fp16, dict(x=x, wt=wt, s_w=s_w, out=out, s_a_out=s_a), ("wt", "out", "s_a_out")),
        "linear_tiled_swiglu_fp16": (w4a8.w4a8_linear_tiled_swiglu_fp16, dict(x=x, wt_gu=wt, s_w_gu=s_w, h=e(half, M, N // 2), s_a_out=s_a),
                                     ("wt_gu", "h", "s_a_out")),
        "linear_tiled_norm_fp16": (w4a8.w4a8_linear_tiled_norm_fp16,
                                   dict(x=x, res=e(half, M, K), gamma=e(half, K), eps=1e-5, wt=wt, s_w=s_w, out=out, r_out=e(half, M, K),
                                        y_out=e(half, M, K), s_a_out=s_a), ("res", "gamma", "wt", "out", "r_out", "y_out", "s_a_out")),
        "add_rmsnorm_quantize": (w4a8.w4a8_add_rmsnorm_quantize,
                                 dict(x=x, res=e(half, M, K), gamma=e(half, K), eps=1e-5, r_out=e(half, M, K), y_out=e(half, M, K), **rows),
                                 ("res", "gamma", "r_out", "y_out", "xq", "s_a")),
        "gemm_fine_grained": (w4a8.w4a8_gemm_fine_grained, dict(xq=xq, s_a=s_a, wt=wt, s_g=e(f32, K // 128, N), out=out), ("s_a", "wt", "s_g", "out")),
        "quantize_weights": (w4a8.w4a8_quantize_weights, dict(w=w, wp=wp, s_w=s_w), ("wp", "s_w")),
        "quantize_weights_clipped": (w4a8.w4a8_quantize_weights_clipped, dict(w=w, gamma=e(f32, N), beta=e(f32, N), wp=wp, s_w=s_w),
                                     ("gamma", "beta", "wp", "s_w")),
        "silu_mul": (w4a8.w4a8_silu_mul, dict(gate_up=gate_up, h=e(half, M, N)), ("h",)),
        "silu_mul_quantize": (w4a8.w4a8_silu_mul_quantize, dict(gate_up=gate_up, xq=e(i8, M, N), s_a=e(f32, M)), ("xq", "s_a")),
    }


NAMES = ["quantize_act", "quantize_act_strided", "gemm", "gemm_acc_i32", "gemm_tuned", "gemm_tuned_tiled", "tile_weights", "gemm_tiled",
         "gemm_tiled_splitk", "gemm_tiled_splitk_static", "gemm_tiled_unsigned", "gemm_tiled_swiglu", "w8a8_tile_weights", "w8a8_gemm_tiled",
         "linear_tiled_fp16", "linear_tiled_swiglu_fp16", "linear_tiled_norm_fp16", "add_rmsnorm_quantize", "gemm_fine_grained",
         "quantize_weights", "quantize_weights_clipped", "silu_mul", "silu_mul_quantize"]


@pytest.mark.parametrize("name", NAMES)
def test_a_tensor_that_is_too_small_launches_nothing(launches, name):
    seen, e = launches
    calls = _calls(e)
    assert sorted(calls) == sorted(NAMES)
    function, args, sized = calls[name]
    function(**args)
    assert len(seen) == 1, "the whole call is launched"
    for key in sized:
        short = args[key][:-1].as_subclass(type(args[key]))
        with pytest.raises((TypeError, ValueError)):
            function(**dict(args, **{key: short}))
        assert len(seen) == 1, key


@pytest.mark.parametrize("name", ["gemm_tiled", "gemm_tiled_splitk", "gemm_tiled_splitk_static", "gemm_tiled_unsigned", "w8a8_gemm_tiled",
                                  "gemm_fine_grained", "silu_mul_quantize", "quantize_weights"])
def test_a_longer_buffer_of_scales_is_enough(launches, name):
    seen, e = launches
    function, args, _ = _calls(e)[name]
    key = "s_w" if name == "quantize_weights" else "s_a"
    function(**dict(args, **{key: e(args[key].dtype, args[key].numel() + 5)}))
    assert len(seen) == 1


def test_a_residual_on_another_device_launches_nothing(launches):
    seen, e = launches
    function, args, _ = _calls(e)["linear_tiled_norm_fp16"]

    class Elsewhere(type(args["res"])):
        def get_device(self):
            return 1
    with pytest.raises(ValueError):
        function(**dict(args, res=args["res"].as_subclass(Elsewhere)))
    assert not seen
