"""The native short way of the binding's calls on a GPU: the results, objects and errors of the checks written out in Python."""
import pytest

import paper_2311_09550_amd as w4a8

pytestmark = pytest.mark.gpu

M, N, K = 3, 96, 160


@pytest.fixture
def operands(gpu):
    t = gpu
    g = t.Generator(device="cuda").manual_seed(5)
    x = t.randn((M, K), generator=g, device="cuda").half()
    w = (t.randn((N, K), generator=g, device="cuda") * 0.02).half()
    wp, sw = w4a8.w4a8_quantize_weights(w)
    w8, sw8 = w4a8.w4a8_quantize_act(w)
    xq, sa = w4a8.w4a8_quantize_act(x)
    return dict(x=x, xq=xq, sa=sa, wp=wp, wt=w4a8.w4a8_tile_weights(wp), sw=sw, wt8=w4a8.w8a8_tile_weights(w8), sw8=sw8,
                ws=t.empty(1 << 16, dtype=t.uint8, device="cuda"), wide=t.randn((M, K + 32), generator=g, device="cuda").half())


def _calls(o):
    """name -> (function, its arguments, names of its outputs, the short way's arguments but for them)"""
    return {"quantize_act": (w4a8.w4a8_quantize_act, dict(x=o["x"]), ("xq", "s_a"), ("x",)),
            "quantize_act_strided": (w4a8.w4a8_quantize_act_strided, dict(x=o["wide"][:, 32:]), ("xq", "s_a"), ("x",)),
            "gemm": (w4a8.w4a8_gemm, dict(xq=o["xq"], s_a=o["sa"], wp=o["wp"], s_w=o["sw"]), ("out",), ("xq", "s_a", "wp", "s_w")),
            "gemm_tiled": (w4a8.w4a8_gemm_tiled, dict(xq=o["xq"], s_a=o["sa"], wt=o["wt"], s_w=o["sw"]), ("out",), ("xq", "s_a", "wt", "s_w")),
            "gemm_tiled_splitk": (w4a8.w4a8_gemm_tiled_splitk, dict(xq=o["xq"], s_a=o["sa"], wt=o["wt"], s_w=o["sw"], ws=o["ws"]), ("out",),
                                  ("xq", "s_a", "wt", "s_w", "ws")),
            "w8a8_gemm_tiled": (w4a8.w8a8_gemm_tiled, dict(xq=o["xq"], s_a=o["sa"], wt=o["wt8"], s_w=o["sw8"]), ("out",), ("xq", "s_a", "wt", "s_w")),
            "linear_tiled_fp16": (w4a8.w4a8_linear_tiled_fp16, dict(x=o["wide"][:, :K], wt=o["wt"], s_w=o["sw"]), ("out", "s_a_out"), ("x", "wt", "s_w")),
            "quantize_weights": (w4a8.w4a8_quantize_weights, dict(w=o["x"]), ("wp", "s_w"), ("w",)),
            "tile_weights": (w4a8.w4a8_tile_weights, dict(wp=o["wp"]), ("wt",), ("wp",))}


NAMES = ["quantize_act", "quantize_act_strided", "gemm", "gemm_tiled", "gemm_tiled_splitk", "w8a8_gemm_tiled", "linear_tiled_fp16",
         "quantize_weights", "tile_weights"]


def _tuple(r):
    return r if isinstance(r, tuple) else (r,)


@pytest.mark.parametrize("name", NAMES)
def test_same_results_and_objects_with_and_without(gpu, operands, monkeypatch, name):
    t = gpu
    function, args, outs, order = _calls(operands)[name]
    assert getattr(w4a8._short, name)(*(args[k] for k in order), *(None for _ in outs)) is not None, "the plain case is served"
    fast = _tuple(function(**args))
    given = {k: t.empty_like(r) for k, r in zip(outs, fast)}
    back = _tuple(function(**args, **given))
    assert all(b is given[k] for k, b in zip(outs, back))
    stream = t.cuda.Stream()
    with t.cuda.stream(stream):
        elsewhere = _tuple(function(**args))
    stream.synchronize()
    monkeypatch.setattr(w4a8, "_short", w4a8._NothingLoaded())
    slow = _tuple(function(**args))
    t.cuda.synchronize()
    for a, b, c, d in zip(slow, fast, back, elsewhere):
        assert a.shape == b.shape and a.dtype == b.dtype and a.device == b.device and b.is_contiguous() and not b.requires_grad
        assert t.equal(a, b) and t.equal(a, c) and t.equal(a, d)


@pytest.mark.parametrize("name", NAMES)
def test_what_is_not_plain_is_left_to_the_checks_in_python(gpu, operands, monkeypatch, name):
    """Another type, shape, order or class of each tensor, an output that does not fit: not served, and the same answer (an error, or
    a result) with the short way and without."""
    t = gpu
    function, args, outs, order = _calls(operands)[name]

    class Sub(t.Tensor):
        pass

    def forms(v):
        yield v.double()
        yield v[:-40] if v.dim() == 1 else v[:, :-1]  # 40 channels fewer are a block fewer
        yield v.cpu()
        yield t.zeros((*v.shape[:-1], 2 * v.shape[-1]), dtype=v.dtype, device=v.device)[..., ::2]
        yield v.as_subclass(Sub)
        yield v.reshape(1, *v.shape)
    tried = 0
    for key in order:
        for form in forms(args[key]):
            changed = dict(args, **{key: form})
            if key == "ws" and form.dtype == t.uint8 and form.is_cuda and form.is_contiguous() and type(form) is t.Tensor:
                continue  # a workspace of another shape is a workspace
            if form.dim() == 2 and form.stride(1) == 1 and form.dtype == t.float16 and form.is_cuda and key == "x" and type(form) is t.Tensor:
                continue  # a narrower view of x: a call in its own right, for the C side to answer
            assert getattr(w4a8._short, name)(*(changed[k] for k in order), *(None for _ in outs)) is None, (key, tuple(form.shape))
            answers = []
            for short in (w4a8._short, w4a8._NothingLoaded()):
                with monkeypatch.context() as m:
                    m.setattr(w4a8, "_short", short)
                    try:
                        answers.append([r.shape for r in _tuple(function(**changed))])
                    except Exception as e:  # noqa: BLE001 - whatever it says, it says twice
                        answers.append((type(e), str(e)))
            assert answers[0] == answers[1], key
            tried += 1
    counted = ("quantize_weights", "tile_weights")  # whose outputs are held to a size in Python, not to a shape
    for key, r in zip(outs, _tuple(function(**args))):
        for shape, dtype in ((r.shape, t.float64), ((r.shape[0] - 1, *r.shape[1:]), r.dtype), ((*r.shape, 1), r.dtype)):
            if name in counted and len(shape) > r.dim():
                continue
            form = t.empty(shape, dtype=dtype, device="cuda")
            assert getattr(w4a8._short, name)(*(args[k] for k in order), *(form if k == key else None for k in outs)) is None
            with pytest.raises((TypeError, ValueError)):
                function(**args, **{key: form})
            tried += 1
    assert tried >= 7, tried
    t.cuda.synchronize()


def test_error_codes_raise(gpu, operands):
    t, o = gpu, operands
    x5 = t.zeros((5, K), dtype=t.float16, device="cuda")  # more tokens than the linear that quantises takes
    with pytest.raises(w4a8.W4A8Error) as e:
        w4a8.w4a8_linear_tiled_fp16(x5, o["wt"], o["sw"])
    assert e.value.code == -7 or e.value.code == -4, e.value.code
    odd = t.zeros(M * K + 8, dtype=t.float16, device="cuda")[1:M * K + 1].view(M, K)
    with pytest.raises(w4a8.W4A8Error) as e:
        w4a8.w4a8_quantize_act(odd)
    assert e.value.code == -3


def test_a_mode_that_watches_allocations_sees_them(gpu, operands):
    from torch.overrides import TorchFunctionMode

    seen = []

    class Watch(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))
    with Watch():
        w4a8.w4a8_quantize_act(operands["x"])
    assert gpu.empty in seen


def _bound_args(t, o):
    import ctypes
    e = lambda dtype, *shape: t.empty(shape, dtype=dtype, device="cuda")  # noqa: E731
    half, codes, scales, one = e(t.float16, M, N), e(t.int8, M, K), e(t.float32, M), ctypes.c_float(1e-5)
    gamma = t.ones(K, dtype=t.float16, device="cuda")
    return [("w4a8_quantize_act", (o["x"], codes, scales, M, K), (codes, scales)),
            ("w4a8_quantize_act_strided", (o["wide"], K + 32, codes, scales, M, K), (codes, scales)),
            ("w4a8_add_rmsnorm_quantize", (o["x"], None, gamma, one, None, None, codes, scales, M, K), (codes, scales)),
            ("w4a8_gemm_tiled_splitk", (o["xq"], o["sa"], o["wt"], o["sw"], half, M, N, K, 0, 0, o["ws"], o["ws"].numel()), (half,)),
            ("w4a8_linear_tiled_norm_fp16", (o["wide"], K + 32, None, 0, gamma, one, None, None, o["wt"], o["sw"], half, None, M, N, K, 0), (half,)),
            ("w8a8_gemm_tiled", (o["xq"], o["sa"], o["wt8"], o["sw8"], half, None, M, N, K, 0), (half,))]


@pytest.mark.parametrize("i", range(6))
def test_bound_calls_are_those_of_ctypes(gpu, operands, monkeypatch, i):
    import gc
    t = gpu
    name, args, outs = _bound_args(t, operands)[i]
    native = w4a8.bound_call(name, *args)
    with monkeypatch.context() as m:
        m.setattr(w4a8, "_short", w4a8._NothingLoaded())
        by_ctypes = w4a8.bound_call(name, *args)
    assert type(native) is not type(by_ctypes)
    results = []
    for call in (by_ctypes, native):
        for r in outs:
            r.zero_()
        assert call() is None
        results.append([r.clone() for r in outs])
    assert all(t.equal(a, b) and bool(a.any()) for a, b in zip(*results))
    stream = t.cuda.Stream()
    for r in outs:
        r.zero_()
    stream.wait_stream(t.cuda.current_stream())
    with t.cuda.stream(stream):
        native()
    stream.synchronize()
    assert all(t.equal(a, b) for a, b in zip(results[0], outs))
    with pytest.raises(TypeError):
        native(1)
    # the tensors live as long as the call does
    def refs(r):
        return sum(x is r for x in gc.get_referents(native)[0])
    assert all(refs(r) == 1 for r in outs)


def test_bound_calls_raise_error_codes_and_leave_odd_arguments_to_ctypes(gpu, operands):
    o = operands
    codes, scales = gpu.empty((M, K), dtype=gpu.int8, device="cuda"), gpu.empty(M, device="cuda")
    with pytest.raises(w4a8.W4A8Error) as e:
        w4a8.bound_call("w4a8_quantize_act", o["x"], codes, scales, M, 100)()
    assert e.value.code == -2
    with pytest.raises(Exception):
        w4a8.bound_call("w4a8_quantize_act", o["x"], codes, scales, "three", K)()
    with pytest.raises(Exception):
        w4a8.bound_call("w4a8_quantize_act", o["x"], codes, scales, M)()
