"""GPU parity of the per-token quantiser fused behind the residual addition and RMSNorm (w4a8_add_rmsnorm_quantize),
stage by stage against the CPU oracle: r bit-exact, y within an fp16 rounding of the fp64 value, codes and scales
bit-exact on the y the GPU computed (the decision that makes integers is taken on the same fp16 values on both sides),
through the C ABI."""
import numpy as np
import pytest

import paper_2311_09550_amd as w4a8
from paper_2311_09550_amd import synth

from parity import assert_equal_bits

pytestmark = pytest.mark.gpu


def _gain(K, seed):
    rng = np.random.default_rng(seed)
    return rng.uniform(0.25, 2.0, K).astype(np.float16)


def _check(t, oracle, x, res, g, eps, what):
    M, K = x.shape
    dx, dg = t.from_numpy(x).cuda(), t.from_numpy(g).cuda()
    dres = None if res is None else t.from_numpy(res).cuda()
    r_out = t.empty((M, K), dtype=t.float16, device="cuda")
    y_out = t.empty((M, K), dtype=t.float16, device="cuda")
    xq, s_a = w4a8.w4a8_add_rmsnorm_quantize(dx, dres, dg, eps, r_out=r_out, y_out=y_out)
    xq2, s_a2 = w4a8.w4a8_add_rmsnorm_quantize(dx, dres, dg, eps)      # production form: neither r nor y written
    t.cuda.synchronize()
    r_o, y64, _ = oracle.add_rmsnorm(x, res, g, eps)
    assert_equal_bits(r_out.cpu().numpy().view(np.uint16), r_o.view(np.uint16), what + " r")
    y = y_out.cpu().numpy()
    big = np.abs(y64) >= 2.0 ** -14
    assert np.all(np.abs(y.astype(np.float64) - y64)[big] <= 2.0 ** -10 * np.abs(y64)[big]), what + " y"
    assert np.all(np.abs(y.astype(np.float64) - y64)[~big] <= 2.0 ** -24), what + " y (subnormal range)"
    xq_o, s_a_o = oracle.quantize_act(y)                                # the oracle's quantiser on the GPU's y
    assert_equal_bits(s_a.cpu().numpy().view(np.uint32), s_a_o.view(np.uint32), what + " s_a")
    assert_equal_bits(xq.cpu().numpy(), xq_o, what + " xq")
    assert_equal_bits(xq2.cpu().numpy(), xq_o, what + " xq without r / y outputs")
    assert_equal_bits(s_a2.cpu().numpy().view(np.uint32), s_a_o.view(np.uint32), what + " s_a without r / y outputs")
    return dx, dres, dg, r_out, xq, s_a


@pytest.mark.parametrize("with_res", [False, True])
@pytest.mark.parametrize("M,K", [(1, 32), (3, 96), (1, 4096), (16, 5120), (5, 8192), (2, 16384), (2, 16416), (3, 28672),
                                 (1, 65536), (130, 1024), (1024, 5120)])
def test_add_rmsnorm_quantize_stage_wise(gpu, oracle, M, K, with_res):
    x = synth.activations_fp16(M, K, config_id=2, tag=95)
    res = synth.activations_fp16(M, K, config_id=2, tag=96) if with_res else None
    _check(gpu, oracle, x, res, _gain(K, K), 1e-5, f"M={M} K={K} res={with_res}")


def test_add_rmsnorm_quantize_special_rows_and_in_place_residual(gpu, oracle):
    t = gpu
    M, K = 6, 16416                    # longer than what a thread keeps in registers: the later passes read r back
    x = synth.activations_fp16(M, K, config_id=2, tag=97)
    res = synth.activations_fp16(M, K, config_id=2, tag=98)
    x[0, :] = 0
    res[0, :] = 0                      # an all-zero row: y = 0, scale 0, codes 0 (eps > 0)
    res[1, :] = -x[1, :]               # cancels to a zero row
    x[2, :] = np.float16(2048)
    res[2, :] = np.float16(3)          # every sum is a tie in fp16 (2051 -> 2052)
    x[3, :] = np.float16(6e-8)
    res[3, :] = 0                      # fp16 subnormals: the mean square is far below eps
    x[4, :] = np.float16(60000)
    res[4, :] = np.float16(5000)       # sums near the top of the fp16 range (65000 rounds to 64992)
    g = _gain(K, 7)
    dx, dres, dg, r_ref, xq_ref, sa_ref = _check(t, oracle, x, res, g, 1e-5, "special rows")
    # the residual stream updated in place: r_out is the residual buffer itself
    res_buf = dres.clone()
    xq, s_a = w4a8.w4a8_add_rmsnorm_quantize(dx, res_buf, dg, 1e-5, r_out=res_buf)
    t.cuda.synchronize()
    assert bool((res_buf.view(t.int16) == r_ref.view(t.int16)).all()), "in-place residual differs"
    assert bool((xq == xq_ref).all()) and bool((s_a.view(t.int32) == sa_ref.view(t.int32)).all()), "in-place: codes differ"


def test_add_rmsnorm_quantize_refuses_bad_arguments(gpu):
    t = gpu
    x = t.zeros((2, 64), dtype=t.float16, device="cuda")
    g = t.ones((64,), dtype=t.float16, device="cuda")
    for eps in (-1.0, float("nan"), float("inf")):
        with pytest.raises(w4a8.W4A8Error) as e:
            w4a8.w4a8_add_rmsnorm_quantize(x, None, g, eps)
        assert e.value.code == -7
    with pytest.raises(w4a8.W4A8Error) as e:
        w4a8.w4a8_add_rmsnorm_quantize(t.zeros((2, 40), dtype=t.float16, device="cuda"), None,
                                       t.ones((40,), dtype=t.float16, device="cuda"), 1e-5)
    assert e.value.code == -2


@pytest.mark.parametrize("swiglu", [False, True])
@pytest.mark.parametrize("with_res", [False, True])
@pytest.mark.parametrize("M,N,K", [(1, 64, 32), (2, 192, 160), (3, 1024, 1056), (1, 2560, 5120), (4, 512, 4096), (2, 320, 8192),
                                   (1, 15360, 5120)])
def test_norm_linear_stage_wise(gpu, oracle, M, N, K, with_res, swiglu):
    """w4a8_linear_tiled_norm_fp16: r bit-exact and y within an fp16 rounding of the oracle; the output, bit for bit,
    what the linear without the norm gives on the y this call computed (which is itself checked against the oracle's
    quantiser and GEMM in test_gpu_fused_linear.py / test_gpu_swiglu.py)."""
    t = gpu
    if M * K > 27000:
        pytest.skip("the rows do not fit in LDS three times over: refused")
    x = synth.activations_fp16(M, K, config_id=2, tag=101)
    res = synth.activations_fp16(M, K, config_id=2, tag=102) if with_res else None
    g = _gain(K, K + 1)
    w = t.from_numpy(synth.weights_fp16(N, K, config_id=101)).cuda()
    wp, s_w = w4a8.w4a8_quantize_weights(w4a8.interleave_gate_up(w) if swiglu else w)
    wt = w4a8.w4a8_tile_weights(wp)
    dx, dg = t.from_numpy(x).cuda(), t.from_numpy(g).cuda()
    dres = None if res is None else t.from_numpy(res).cuda()
    r_out = t.empty((M, K), dtype=t.float16, device="cuda")
    y_out = t.empty((M, K), dtype=t.float16, device="cuda")
    s_a = t.empty((M,), dtype=t.float32, device="cuda")
    out = w4a8.w4a8_linear_tiled_norm_fp16(dx, dres, dg, 1e-5, wt, s_w, swiglu=swiglu, r_out=r_out, y_out=y_out, s_a_out=s_a)
    out2 = w4a8.w4a8_linear_tiled_norm_fp16(dx, dres, dg, 1e-5, wt, s_w, swiglu=swiglu)   # nothing but the output written
    ref = w4a8.w4a8_linear_tiled_swiglu_fp16(y_out, wt, s_w) if swiglu else w4a8.w4a8_linear_tiled_fp16(y_out, wt, s_w)
    t.cuda.synchronize()
    what = f"M={M} N={N} K={K} res={with_res} swiglu={swiglu}"
    r_o, y64, _ = oracle.add_rmsnorm(x, res, g, 1e-5)
    assert_equal_bits(r_out.cpu().numpy().view(np.uint16), r_o.view(np.uint16), what + " r")
    y = y_out.cpu().numpy()
    big = np.abs(y64) >= 2.0 ** -14
    assert np.all(np.abs(y.astype(np.float64) - y64)[big] <= 2.0 ** -10 * np.abs(y64)[big]), what + " y"
    assert np.all(np.abs(y.astype(np.float64) - y64)[~big] <= 2.0 ** -24), what + " y (subnormal range)"
    _, s_a_o = oracle.quantize_act(y)
    assert_equal_bits(s_a.cpu().numpy().view(np.uint32), s_a_o.view(np.uint32), what + " s_a")
    assert_equal_bits(out.cpu().numpy().view(np.uint16), ref.cpu().numpy().view(np.uint16), what + " out vs the linear on y")
    assert_equal_bits(out2.cpu().numpy().view(np.uint16), ref.cpu().numpy().view(np.uint16), what + " out without r / y outputs")


def test_norm_linear_strided_inputs_zero_rows_and_refusals(gpu, oracle):
    t = gpu
    M, N, K = 3, 264, 2080
    x = synth.activations_fp16(M, K, config_id=2, tag=103)
    res = synth.activations_fp16(M, K, config_id=2, tag=104)
    x[1, :] = 0
    res[1, :] = 0                                     # a zero row: y = 0, scale 0, output 0
    g = _gain(K, 3)
    w = t.from_numpy(synth.weights_fp16(N, K, config_id=103)).cuda()
    wp, s_w = w4a8.w4a8_quantize_weights(w)
    wt = w4a8.w4a8_tile_weights(wp)
    dg = t.from_numpy(g).cuda()
    dense = w4a8.w4a8_linear_tiled_norm_fp16(t.from_numpy(x).cuda(), t.from_numpy(res).cuda(), dg, 1e-5, wt, s_w)
    wide_x = t.zeros((M, 3 * K), dtype=t.float16, device="cuda")
    wide_r = t.zeros((M, 2 * K + 8), dtype=t.float16, device="cuda")
    wide_x[:, K:2 * K] = t.from_numpy(x).cuda()
    wide_r[:, 8:8 + K] = t.from_numpy(res).cuda()
    strided = w4a8.w4a8_linear_tiled_norm_fp16(wide_x[:, K:2 * K], wide_r[:, 8:8 + K], dg, 1e-5, wt, s_w)
    t.cuda.synchronize()
    assert_equal_bits(strided.cpu().numpy().view(np.uint16), dense.cpu().numpy().view(np.uint16), "strided inputs")
    assert bool((dense[1] == 0).all()), "zero row"
    for bad in (dict(M=5, K=1024), dict(M=1, K=8224)):            # beyond four tokens; beyond the hidden sizes it serves
        xb = t.zeros((bad["M"], bad["K"]), dtype=t.float16, device="cuda")
        wtb = t.zeros((w4a8.w4a8_tiled_weight_bytes(64, bad["K"]),), dtype=t.uint8, device="cuda")
        with pytest.raises(w4a8.W4A8Error) as e:
            w4a8.w4a8_linear_tiled_norm_fp16(xb, None, t.ones((bad["K"],), dtype=t.float16, device="cuda"), 1e-5, wtb,
                                             t.ones((64,), dtype=t.float32, device="cuda"))
        assert e.value.code == -7


@pytest.mark.parametrize("K", [64, 1056, 4096])
def test_scales_of_rows_whose_maximum_is_near_an_fp16_rounding_boundary(gpu, K):
    """The row's largest |y| follows from the largest |r g| unless that falls near a boundary between two fp16 values, about once
    in two thousand rows: over enough rows that many do, codes and scales are the quantiser's on the very y that comes out."""
    t = gpu
    gen = t.Generator(device="cuda").manual_seed(K)
    M = 20000 if K < 4096 else 6000
    x = t.randn((M, K), generator=gen, device="cuda").half()
    res = t.randn((M, K), generator=gen, device="cuda").half()
    g = (1 + 0.1 * t.randn((K,), generator=gen, device="cuda")).half()
    for m in (100, 200, M):                               # 1024, 512 and 256 threads a row
        y = t.empty((m, K), dtype=t.float16, device="cuda")
        xq, s_a = w4a8.w4a8_add_rmsnorm_quantize(x[:m], res[:m], g, 1e-5, y_out=y)
        xq_ref, s_ref = w4a8.w4a8_quantize_act(y)
        t.cuda.synchronize()
        assert t.equal(xq, xq_ref) and t.equal(s_a.view(t.int32), s_ref.view(t.int32)), m
    if K > 64:
        return
    # the same inside the linear, where the rows of a launch are up to four
    wt, s_w = t.zeros((w4a8.w4a8_tiled_weight_bytes(64, K),), dtype=t.uint8, device="cuda"), t.ones((64,), dtype=t.float32, device="cuda")
    y, s_a = t.empty((M, K), dtype=t.float16, device="cuda"), t.empty((M,), dtype=t.float32, device="cuda")
    for m in range(0, M, 4):
        w4a8.w4a8_linear_tiled_norm_fp16(x[m:m + 4], res[m:m + 4], g, 1e-5, wt, s_w, y_out=y[m:m + 4], s_a_out=s_a[m:m + 4])
    s_ref = w4a8.w4a8_quantize_act(y)[1]
    t.cuda.synchronize()
    assert t.equal(s_a.view(t.int32), s_ref.view(t.int32))


def _rows_whose_maximum_lies_at_a_boundary(t, K, want):
    """(x, res, gain) of `want` rows whose largest |r g| / rms, in fp64, lies within 2^-22 of a value halfway between two fp16
    neighbours: well inside the 2^-21 within which the kernel has to look at its values, whatever it rounds on the way."""
    gen = t.Generator(device="cuda").manual_seed(K)
    gain = (1 + 0.1 * t.randn((K,), generator=gen, device="cuda")).half()
    found = []
    for _ in range(400):
        x, res = (t.randn((500, K), generator=gen, device="cuda").half() for _ in range(2))
        r = (x.float() + res.float()).half().double()
        v = (r * gain.double()).abs().amax(1) / (r.square().mean(1) + 1e-5).sqrt()
        h = v.half()
        low = t.where(h.double() > v, (h.view(t.int16) - 1).view(t.float16), h)
        edge = (low.double() + (low.view(t.int16) + 1).view(t.float16).double()) / 2
        found += [(x[i], res[i]) for i in t.nonzero((v / edge - 1).abs() < 2.0 ** -22).flatten().tolist()]
        if len(found) >= want:
            break
    assert len(found) >= want
    return t.stack([f[0] for f in found[:want]]), t.stack([f[1] for f in found[:want]]), gain


@pytest.mark.parametrize("swiglu", [False, True])
@pytest.mark.parametrize("K", [64, 2080, 4096, 5120])
def test_linear_over_rows_whose_maximum_lies_at_a_boundary(gpu, K, swiglu):
    """Here the linear finds its maxima in y after all.  The scales and the output are those of the plain linear on the y that this
    call wrote, with chunks of the row in every wave and several k steps a wave, for all rows of a launch and for one among others,
    with and without r and y written."""
    t = gpu
    N, most = 320, 4 if K <= 4096 else 3
    x, res, gain = _rows_whose_maximum_lies_at_a_boundary(t, K, 8)
    gen = t.Generator(device="cuda").manual_seed(N)
    plain = t.randn((2, 2, 8, K), generator=gen, device="cuda").half()
    w = (0.02 * t.randn((N, K), generator=gen, device="cuda")).half()
    wp, s_w = w4a8.w4a8_quantize_weights(w)
    wt = w4a8.w4a8_tile_weights(wp)
    linear = w4a8.w4a8_linear_tiled_swiglu_fp16 if swiglu else w4a8.w4a8_linear_tiled_fp16
    for i in range(8):
        M = 1 + i % most
        dx, dres = plain[0, 0, :M].clone(), plain[0, 1, :M].clone()
        rows = range(M) if i < 4 else [i % M]
        for j in rows:
            dx[j], dres[j] = x[(i + j) % 8], res[(i + j) % 8]
        r, y, s_a = t.empty_like(dx), t.empty_like(dx), t.empty((M,), dtype=t.float32, device="cuda")
        out = w4a8.w4a8_linear_tiled_norm_fp16(dx, dres, gain, 1e-5, wt, s_w, swiglu=swiglu, r_out=r, y_out=y, s_a_out=s_a)
        bare = w4a8.w4a8_linear_tiled_norm_fp16(dx, dres, gain, 1e-5, wt, s_w, swiglu=swiglu)
        ref, s_ref = linear(y, wt, s_w), w4a8.w4a8_quantize_act(y)[1]
        t.cuda.synchronize()
        assert t.equal(r.view(t.int16), (dx.float() + dres.float()).half().view(t.int16)), (i, "r")
        assert t.equal(s_a.view(t.int32), s_ref.view(t.int32)), (i, "scales")
        assert bool(out.any()) and t.equal(out.view(t.int16), ref.view(t.int16)), (i, "output")
        assert t.equal(bare.view(t.int16), ref.view(t.int16)), (i, "output without r and y")


def _sum_of_squares(r, threads):
    """The fp32 sum of squares of a row in the kernel's order for `threads` threads: a thread's chunks of eight one after the other
    (a square of an fp16 value added to an fp32 sum rounds once), six DPP steps inside a wave, the waves in order."""
    K = r.shape[0]
    per = -(-K // (8 * threads))
    v = np.zeros(per * threads * 8)
    v[:K] = r.astype(np.float64)
    v = v.reshape(per, threads, 8)
    ss = np.zeros(threads, np.float32)
    for i in range(per):
        for e in range(8):
            ss = (ss.astype(np.float64) + v[i, :, e] ** 2).astype(np.float32)
    x = ss.reshape(-1, 4, 16)  # wave, row of lanes, lane
    for step in (1, 2, 4, 8):
        x = x + np.concatenate((np.zeros_like(x[:, :, :step]), x[:, :, :-step]), axis=2)
    x[:, 1::2] += x[:, 0::2, 15:]
    x[:, 2:] += x[:, 1, 15][:, None, None]
    total = np.float32(0)
    for w in x[:, 3, 15]:
        total = np.float32(total + w)
    return total


@pytest.mark.parametrize("M,threads", [(5, 1024), (128, 1024), (129, 512), (257, 256)])
@pytest.mark.parametrize("K", [32, 4096, 4128, 8192, 8224, 9216, 12288, 12320, 16384, 16416, 24608])
def test_the_sum_of_squares_has_one_order_for_each_number_of_rows(gpu, M, threads, K):
    """However a row is spread over threads, its sum is the documented one: the order of 1024 threads up to 128 rows, of 512 up to
    256, of 256 beyond.  The rows are ones with a few values of 4096, whose squares swallow the ones added to them, so that another
    order is another sum (many ulp); the square root is the hardware's, within one ulp."""
    t = gpu
    rng = np.random.default_rng(M + K)
    x = rng.choice([np.float16(-1), np.float16(1)], size=(M, K))
    x[rng.random((M, K)) < 0.005] = np.float16(4096)
    gain = (1 + 0.1 * rng.standard_normal(K)).astype(np.float16)
    y = t.empty((M, K), dtype=t.float16, device="cuda")
    w4a8.w4a8_add_rmsnorm_quantize(t.from_numpy(x).cuda(), None, t.from_numpy(gain).cuda(), 1e-5, y_out=y)
    t.cuda.synchronize()
    for m in sorted({0, M // 2, M - 1}):
        root = np.sqrt(np.float32(np.float32(_sum_of_squares(x[m], threads) / np.float32(K)) + np.float32(1e-5)))
        got = y[m].cpu().numpy().view(np.uint16)
        want = [((x[m].astype(np.float32) * (np.float32(1) / s)) * gain.astype(np.float32)).astype(np.float16).view(np.uint16)
                for s in (root, np.nextafter(root, np.float32(0)), np.nextafter(root, np.float32(np.inf)))]
        assert any(np.array_equal(got, w) for w in want), f"M={M} K={K} row {m}: {[int((got != w).sum()) for w in want]} values differ"
