"""GPU parity of the medium-M kernel (waves that split K, weights in registers): every tile and weight format the library
chooses, at shapes with fewer k steps than wave groups, K that ends inside a step, M and N off the tile, N a multiple of 4
(vector stores) and not.  The sums are integers, so the outputs have the bits of any other tile; sampled rows against the oracle."""
import numpy as np
import pytest

import paper_2311_09550_amd as w4a8
from paper_2311_09550_amd import synth

from parity import assert_equal_bits, assert_fp16_close

pytestmark = pytest.mark.gpu

TILED = w4a8.TILING_PREFILL_TILED
ROW32 = 8  # the large-M kernel's 32 x 128 tile


def _inputs(t, oracle, M, N, K, config_id):
    xq, wq, s_a, s_w = synth.uniform_codes(M, N, K, config_id=config_id)
    return (xq, wq, s_a, s_w), [t.from_numpy(a).cuda() for a in (xq, s_a, s_w)]


@pytest.mark.parametrize("M,N,K,tile", [
    (70, 21, 1600, 21), (70, 20, 1632, 21), (50, 4096, 11008, 21), (65, 20, 32, 22), (66, 21, 544, 22), (97, 20, 576, 22),
    (476, 555, 12960, 23), (296, 1032, 6912, 23), (314, 4889, 192, 24), (472, 1137, 544, 24), (430, 1288, 576, 24), (128, 5120, 5120, 24),
    (450, 6216, 448, 25), (424, 3557, 928, 25), (487, 2452, 1568, 25), (242, 4355, 1600, 26), (247, 4356, 1984, 26),
    (464, 3558, 1504, 27), (458, 3784, 1504, 27), (510, 4766, 928, 28), (433, 5412, 1856, 28), (1023, 2048, 11008, 27)])
def test_int4_tiles(gpu, oracle, M, N, K, tile):
    t = gpu
    assert w4a8.w4a8_route(w4a8.ROUTE_GEMM_TILED, M, N, K) == (TILED, tile, 1)
    (xq, wq, s_a, s_w), (dxq, dsa, dsw) = _inputs(t, oracle, M, N, K, 95)
    wp = oracle.pack_w4(wq)
    wt = w4a8.w4a8_tile_weights(t.from_numpy(wp).cuda())
    out = w4a8.w4a8_gemm_tiled(dxq, dsa, wt, dsw)
    acc = w4a8.w4a8_gemm_tuned(dxq, None, wt, None, w4a8.TILING_AUTO_TILED, want_acc=True, N=N)
    ref = w4a8.w4a8_gemm_tuned(dxq, dsa, wt, dsw, TILED, ROW32, N=N)
    acc_ref = w4a8.w4a8_gemm_tuned(dxq, None, wt, None, TILED, ROW32, want_acc=True, N=N)
    t.cuda.synchronize()
    assert t.equal(acc, acc_ref), "sums"
    assert_equal_bits(out.cpu().numpy().view(np.uint16), ref.cpu().numpy().view(np.uint16), f"tile {tile} M={M} N={N} K={K}")
    rows = sorted({0, M // 2, M - 1})
    acc_o, y32, _ = oracle.gemm(xq[rows], s_a[rows], wp, s_w)
    assert_equal_bits(acc.cpu().numpy()[rows], acc_o, "sampled rows acc")
    assert_fp16_close(out.cpu().numpy()[rows], y32, acc_o, "sampled rows out")


@pytest.mark.parametrize("M,I,K,tile", [(76, 32, 1568, 21), (65, 32, 32, 22), (76, 2688, 5792, 23), (421, 608, 576, 24), (453, 3168, 416, 25),
                                        (438, 1248, 2240, 26), (410, 2016, 1440, 27), (422, 2624, 928, 28)])
def test_swiglu_form(gpu, oracle, M, I, K, tile):
    """h has the bits of the plain GEMM over the same interleaved channels and silu_mul."""
    t = gpu
    assert w4a8.w4a8_route(w4a8.ROUTE_SWIGLU, M, 2 * I, K) == (TILED, tile, 1)
    (_, wq, _, _), (dxq, dsa, dsw) = _inputs(t, oracle, M, 2 * I, K, 96)
    wt = w4a8.w4a8_tile_weights(t.from_numpy(oracle.pack_w4(wq)).cuda())
    h = w4a8.w4a8_gemm_tiled_swiglu(dxq, dsa, wt, dsw)
    pairs = w4a8.w4a8_gemm_tuned(dxq, dsa, wt, dsw, TILED, ROW32, N=2 * I).reshape(M, I, 2)
    two = w4a8.w4a8_silu_mul(t.cat((pairs[:, :, 0], pairs[:, :, 1]), dim=1).contiguous())
    t.cuda.synchronize()
    assert_equal_bits(h.cpu().numpy().view(np.uint16), two.cpu().numpy().view(np.uint16), f"swiglu tile {tile} M={M} I={I} K={K}")


@pytest.mark.parametrize("M,N,K,tile", [
    (18, 4219, 672, 21), (426, 307, 1696, 21), (399, 332, 1632, 21), (483, 138, 320, 22), (501, 257, 672, 22), (465, 296, 672, 22),
    (468, 6050, 288, 26), (464, 2235, 832, 26), (419, 2628, 800, 26), (1, 20, 288, 29), (1, 21, 1056, 29), (16, 4096, 4096, 29),
    (444, 148, 544, 30), (440, 158, 1056, 30), (414, 148, 1440, 30), (336, 8162, 416, 31), (438, 4867, 1184, 31), (467, 4540, 896, 31),
    (512, 5120, 13824, 31)])
def test_int8_tiles(gpu, oracle, M, N, K, tile):
    t = gpu
    assert w4a8.w4a8_route(w4a8.ROUTE_W8A8, M, N, K) == (TILED, tile, 1)
    g = t.Generator(device="cuda").manual_seed(M + N + K)
    xq = t.randint(-128, 128, (M, K), generator=g, device="cuda", dtype=t.int8)
    w8 = t.randint(-128, 128, (N, K), generator=g, device="cuda", dtype=t.int8)
    wt = w4a8.w8a8_tile_weights(w8)
    s_a = t.rand(M, generator=g, device="cuda") * 1e-3
    s_w = t.rand(N, generator=g, device="cuda") * 1e-3
    acc, out = (w4a8.w8a8_gemm_tiled(xq, s_a, wt, s_w, want_acc=a) for a in (True, False))
    acc_ref, out_ref = (w4a8.w8a8_gemm_tiled(xq, s_a, wt, s_w, variant=ROW32, want_acc=a) for a in (True, False))
    t.cuda.synchronize()
    assert t.equal(acc, acc_ref), "sums"
    assert t.equal(out.view(t.int16), out_ref.view(t.int16)), "outputs"
    rows = sorted({0, M // 2, M - 1})
    acc_o, y32, _ = oracle.gemm_w8(xq[rows].cpu().numpy(), s_a[rows].cpu().numpy(), w8.cpu().numpy(), s_w.cpu().numpy())
    assert_equal_bits(acc[rows].cpu().numpy(), acc_o, "sampled rows acc")
    assert_fp16_close(out[rows].cpu().numpy(), y32, acc_o, "sampled rows out")


# with eight k groups: columns of tiles whole on an XCD (weights loaded with the non-temporal hint) and cut between two (without)
@pytest.mark.parametrize("entry,M,N,K,tile,whole", [
    ("tiled", 110, 245, 1984, 21, True), ("tiled", 127, 1857, 1952, 21, False), ("tiled", 33, 4432, 5888, 23, True), ("tiled", 36, 4212, 5760, 23, False),
    ("swiglu", 151, 1024, 1984, 21, True), ("swiglu", 126, 192, 1952, 21, False), ("swiglu", 35, 4480, 6144, 23, True), ("swiglu", 42, 4288, 5760, 23, False),
    ("w8a8", 183, 1266, 2880, 21, True), ("w8a8", 91, 1896, 3744, 21, False), ("w8a8", 76, 511, 3072, 29, True), ("w8a8", 44, 706, 2080, 29, False),
    ("w8a8", 150, 756, 3552, 30, True), ("w8a8", 57, 1809, 2048, 30, False)])
def test_columns_of_tiles_whole_on_an_xcd_and_cut(gpu, oracle, entry, M, N, K, tile, whole):
    """The same comparisons as above on both sides of the rule for the cache policy of the weights."""
    bm, bn = {21: (32, 32), 23: (32, 64), 29: (16, 16), 30: (16, 32)}[tile]
    rows, columns = -(-M // bm), -(-N // bn)
    assert rows > 1 and (-(-rows * columns // 8) % rows == 0) == whole
    if entry == "tiled":
        test_int4_tiles(gpu, oracle, M, N, K, tile)
    elif entry == "swiglu":
        test_swiglu_form(gpu, oracle, M, N // 2, K, tile)
    else:
        test_int8_tiles(gpu, oracle, M, N, K, tile)


def test_graph_replays(gpu, oracle):
    """Captured once, replayed with new inputs between eager work: the bits of the eager call every time."""
    t = gpu
    M, N, K = 128, 5120, 5120
    (_, wq, _, _), (dxq, dsa, dsw) = _inputs(t, oracle, M, N, K, 97)
    wt = w4a8.w4a8_tile_weights(t.from_numpy(oracle.pack_w4(wq)).cuda())
    out, stream = t.empty((M, N), dtype=t.float16, device="cuda"), t.cuda.Stream()
    w4a8.w4a8_init()
    with t.cuda.stream(stream):
        graph = t.cuda.CUDAGraph()
        with t.cuda.graph(graph, stream=stream):
            w4a8.w4a8_gemm_tiled(dxq, dsa, wt, dsw, out=out)
        for i in range(4):
            dxq.copy_(t.roll(dxq, i + 1, 0))
            graph.replay()
            eager = w4a8.w4a8_gemm_tiled(dxq, dsa, wt, dsw)
            stream.synchronize()
            assert t.equal(out.view(t.int16), eager.view(t.int16)), i
