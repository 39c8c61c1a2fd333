"""Which kernel the library's own choice runs, and which calls it refuses: pure functions of the shape (for the 256 compute
units that are assumed where there is no GPU).  No kernel is launched here."""
import ctypes
from concurrent.futures import ThreadPoolExecutor

import pytest

import paper_2311_09550_amd as w4a8
from paper_2311_09550_amd import (ROUTE_GEMM, ROUTE_GEMM_TILED, ROUTE_SPLITK, ROUTE_SPLITK_STATIC, ROUTE_SWIGLU, ROUTE_UNSIGNED,
                                  ROUTE_W8A8, TILING_DECODE_RESIDENT, TILING_DECODE_RESIDENT_TILED, TILING_DECODE_STREAM,
                                  TILING_DECODE_STREAM_TILED, TILING_PREFILL, TILING_PREFILL_TILED, w4a8_route)

P = ctypes.c_void_p(0x1000)  # aligned, non-NULL, never dereferenced


def test_route_answers_for_every_entry_and_refuses_what_the_entry_refuses():
    assert w4a8_route(ROUTE_GEMM, 4, 5120, 5120)[0] == TILING_DECODE_RESIDENT
    assert w4a8_route(ROUTE_GEMM, 1, 8192, 28672)[0] == TILING_DECODE_STREAM     # K beyond the persistent kernel's registers
    assert w4a8_route(ROUTE_GEMM, 777, 15360, 5120)[0] == TILING_PREFILL
    assert w4a8_route(ROUTE_GEMM_TILED, 16, 5120, 5120) == (TILING_DECODE_RESIDENT_TILED, 0, 1)
    assert w4a8_route(ROUTE_GEMM_TILED, 1, 8192, 28672)[0] == TILING_DECODE_STREAM_TILED
    assert w4a8_route(ROUTE_SPLITK, 2, 5120, 5120) == w4a8_route(ROUTE_GEMM_TILED, 2, 5120, 5120)
    for entry in (ROUTE_GEMM_TILED, ROUTE_SPLITK, ROUTE_SPLITK_STATIC, ROUTE_SWIGLU, ROUTE_W8A8, ROUTE_UNSIGNED):
        tiling, tile, slices = w4a8_route(entry, 1024, 27648, 5120)
        assert tiling == TILING_PREFILL_TILED and 1 <= tile <= (8 if entry == ROUTE_UNSIGNED else 20) and slices == 1
    assert w4a8_route(ROUTE_SPLITK, 128, 5120, 13824, 7, 4) == (TILING_PREFILL_TILED, 7, 4)
    for bad, code in (((ROUTE_GEMM, 0, 16, 32), -2), ((ROUTE_GEMM, 1, 16, 48), -2), ((7, 1, 16, 32), -7),
                      ((ROUTE_SPLITK, 1, 16, 256, 13, 0), -7), ((ROUTE_SPLITK, 1, 16, 256, 0, 65), -7),
                      ((ROUTE_SPLITK_STATIC, 512, 4096, 1024, 6, 8), -4), ((ROUTE_SWIGLU, 1, 96, 256), -2)):
        with pytest.raises(w4a8.W4A8Error) as e:
            w4a8_route(*bad)
        assert e.value.code == code, bad


def _on_a_thread(call):
    """The result of a call that may leave a HIP error behind, which the library keeps per thread."""
    with ThreadPoolExecutor(1) as pool:
        return pool.submit(call).result()


def _splitk(M, N, K, variant, splits, slabs, static=False):
    """Return code of the C entry with a workspace of `slabs` slabs (None: no workspace) at addresses that nothing reads: the
    entry refuses before any launch, and what it does not refuse ends in -5, there being no GPU in the CPU tests."""
    L = w4a8.lib()
    if static:
        return L.w4a8_gemm_tiled_splitk_static(P, P, P, P, P, M, N, K, variant, splits, None)
    ws, size = (None, 0) if slabs is None else (P, slabs * M * N * 4)
    return L.w4a8_gemm_tiled_splitk(P, P, P, P, P, M, N, K, variant, splits, ws, size, None)


# Slabs of raw sums that the entry asks a workspace for (variant 0: the library's choice; else a forced tile), 1 = none.
SLABS = [
    (16, 5120, 13824, 0, 1), (32, 5120, 5120, 0, 1), (64, 512, 13824, 0, 3), (50, 4096, 11008, 0, 3), (44, 6244, 47168, 0, 5),
    (61, 17674, 58112, 0, 1), (48, 24191, 55712, 0, 1),                     # no shape of the weight-streaming kernel in 8 slices
    (128, 5120, 5120, 0, 3), (128, 5120, 13824, 0, 6), (333, 4096, 11008, 0, 5), (1024, 5120, 5120, 0, 1),
    (140, 29215, 25248, 0, 2), (395, 20088, 22240, 0, 2),                   # long K, tiles up to the compute units
    (289, 4258, 10528, 4, 6), (10, 179, 13952, 3, 6), (135, 5120, 5120, 12, 3), (5, 12288, 4096, 8, 2), (600, 5120, 5120, 7, 1),
]


@pytest.mark.parametrize("M,N,K,variant,slabs", SLABS)
def test_splitk_asks_for_the_slabs_it_is_documented_to_ask_for(M, N, K, variant, slabs):
    """splits = 0: the size reported, the refusal of less (and of none), the static entry's refusal of more than its array,
    and that a forced tile is cut into as many slices; never more slices than slabs."""
    if variant == 0:
        assert w4a8.w4a8_gemm_tiled_workspace_bytes(M, N, K) == (slabs * M * N * 4 if slabs > 1 else 0)
    tiling, tile, used = w4a8_route(ROUTE_SPLITK, M, N, K, variant, 0)
    assert used <= slabs
    if variant:
        assert (tile, used) == (variant, slabs)
    if slabs > 1:
        assert _splitk(M, N, K, variant, 0, None) == -1
        assert _splitk(M, N, K, variant, 0, slabs - 1) == -4
    fits = slabs == 1 or slabs * M * N * 4 <= 16 << 20
    if not fits:
        assert _splitk(M, N, K, variant, 0, None, static=True) == -4
    import torch
    if not torch.cuda.is_available():  # accepted calls: only where nothing can be launched
        assert _on_a_thread(lambda: _splitk(M, N, K, variant, 0, slabs if slabs > 1 else None)) == -5
        assert not fits or _on_a_thread(lambda: _splitk(M, N, K, variant, 0, None, static=True)) == -5


def test_forced_slice_counts_ask_for_what_was_forced():
    assert _splitk(40, 1800, 10816, 0, 64, 63) == -4         # 43 slices are not empty, 64 slabs are asked for
    assert _splitk(40, 1800, 10816, 0, 64, None, static=True) == -4
    assert _splitk(100, 1800, 10816, 0, 64, 42) == -4        # the large-M kernel: 85 stages in 43 slices of two
    assert w4a8_route(ROUTE_SPLITK, 100, 1800, 10816, 0, 64)[2] == 43
    assert _splitk(64, 200000, 65536, 6, 2, 2) == -2         # sliced, and more than one launch can address


@pytest.mark.parametrize("model", ["7b", "13b", "70b"])
def test_plans_of_a_models_layers_are_remembered(model):
    """One pass over the linears of a layer makes the plans, the second none, for every token count of the sizes in use."""
    from paper_2311_09550_amd.synth import LLAMA_SHAPES
    made = w4a8.lib().w4a8_plans_made
    for M in [17, 24, 32, 33, 48, 50, 64, 100, 128, 200, 256, 333, 512, 700, 1024, 2048]:
        for again in (False, True):
            before = made()
            for name, (N, K) in LLAMA_SHAPES[model].items():
                w4a8_route(ROUTE_SPLITK, M, N, K)
                if name == "gate_up":
                    w4a8_route(ROUTE_SWIGLU, M, N, K)
            assert not again or made() == before, M


@pytest.mark.parametrize("model", ["7b", "13b", "70b"])
def test_tiles_over_int8_weights_are_remembered_too(model):
    """Every token count of the sizes in use, token generation among them; the forms over int4 weights keep plans of their own."""
    from paper_2311_09550_amd.synth import LLAMA_SHAPES
    made = w4a8.lib().w4a8_plans_made
    for M in [1, 4, 16, 17, 64, 128, 333, 512, 1024, 2048]:
        first = {name: w4a8_route(ROUTE_W8A8, M, N, K) for name, (N, K) in LLAMA_SHAPES[model].items()}
        before = made()
        for name, (N, K) in LLAMA_SHAPES[model].items():
            assert w4a8_route(ROUTE_W8A8, M, N, K) == first[name], (M, name)
        assert made() == before, M
        N, K = LLAMA_SHAPES[model]["qkv"]
        int4 = w4a8_route(ROUTE_GEMM_TILED, M, N, K)
        assert w4a8_route(ROUTE_W8A8, M, N, K) == first["qkv"] and w4a8_route(ROUTE_GEMM_TILED, M, N, K) == int4
    N, K = LLAMA_SHAPES[model]["down"]
    before = made()
    w4a8_route(ROUTE_W8A8, 77, N, K)
    assert made() == before + 1  # asked for the first time


def test_unsigned_storage_is_priced_for_its_own_tiles():
    """It has eight tiles, runs 64 x 128 on four waves and converts at twice the cost: the taller tiles pay earlier than over
    signed weights, 128 x 128 among them."""
    for (M, N, K), tile in {(1024, 5120, 5120): 3, (1024, 4096, 11008): 5, (256, 15360, 5120): 5, (64, 57344, 8192): 6,
                            (812, 1168, 9920): 7, (512, 27648, 5120): 1, (16, 27648, 5120): 8}.items():
        assert w4a8_route(ROUTE_UNSIGNED, M, N, K) == (TILING_PREFILL_TILED, tile, 1), (M, N, K)


@pytest.mark.parametrize("M,N,K,tiling", [
    (1, 27648, 5120, TILING_DECODE_RESIDENT), (16, 27648, 5120, TILING_DECODE_RESIDENT), (1, 57344, 8192, TILING_DECODE_RESIDENT),
    (4, 22016, 4096, TILING_DECODE_RESIDENT), (16, 32000, 4096, TILING_DECODE_RESIDENT), (16, 60829, 16384, TILING_DECODE_RESIDENT),
    (16, 8192, 16416, TILING_DECODE_STREAM), (17, 33061, 5376, TILING_DECODE_RESIDENT), (32, 57344, 8192, TILING_DECODE_RESIDENT),
    (17, 8192, 8224, TILING_DECODE_STREAM), (17, 8193, 8224, TILING_PREFILL), (32, 5120, 13824, TILING_DECODE_STREAM),
    (33, 8192, 2048, TILING_DECODE_STREAM), (33, 8193, 2048, TILING_PREFILL), (64, 8192, 2080, TILING_PREFILL),
    (64, 3746, 1824, TILING_DECODE_STREAM), (65, 3746, 1824, TILING_PREFILL),
])
def test_row_major_weights_are_streamed_where_that_is_the_faster_form_on_cold_weights(M, N, K, tiling):
    """Both sides of every line of the rule (256 compute units)."""
    assert w4a8_route(ROUTE_GEMM, M, N, K)[0] == tiling


def test_near_ties_go_to_weight_streaming():
    """Shapes at which the tiles are priced a few per cent below weight streaming and measured slower; and where they are the
    faster form all the same, or the only one with one slice."""
    for M, N, K in [(64, 27648, 5120), (64, 22016, 4096), (63, 8544, 1824), (61, 8778, 1888), (50, 33682, 2848), (31, 59552, 5888),
                    (54, 35603, 3872)]:
        for entry in (ROUTE_GEMM_TILED, ROUTE_SPLITK):
            assert w4a8_route(entry, M, N, K) == (TILING_DECODE_RESIDENT_TILED, 0, 1), (M, N, K)
    assert w4a8_route(ROUTE_SWIGLU, 64, 27648, 5120) == (TILING_DECODE_RESIDENT_TILED, 0, 1)
    assert w4a8_route(ROUTE_SPLITK, 62, 8219, 14976) == (TILING_DECODE_RESIDENT_TILED, 0, 3)
    for M in (48, 50, 64):  # many slices: streaming is the form that is priced too low
        assert w4a8_route(ROUTE_SPLITK, M, 8192, 28672) == (TILING_PREFILL_TILED, 13, 6)
    for M, N, K in [(63, 55468, 3520), (52, 47417, 1344), (64, 57344, 8192), (17, 1216, 16416)]:
        assert w4a8_route(ROUTE_GEMM_TILED, M, N, K)[0] == TILING_PREFILL_TILED, (M, N, K)


def test_several_slices_are_kept_where_they_are_faster_than_the_medium_m_kernel():
    """Slices of weight streaming against the medium-M kernel, each shape measured on cold weights: narrow outputs whose slabs are
    few and stored four values at a time are the slices', an odd N and wider outputs the medium-M kernel's."""
    for M, N, K in [(59, 1600, 11264), (63, 2944, 14976), (62, 1664, 10752), (48, 1024, 7488), (42, 1152, 6976), (32, 4160, 10176),
                    (38, 2432, 10240), (39, 1088, 6656)]:
        tiling, tile, slices = w4a8_route(ROUTE_SPLITK, M, N, K)
        assert (tiling, tile) == (TILING_DECODE_RESIDENT_TILED, 0) and slices > 1, (M, N, K)
        assert w4a8_route(ROUTE_GEMM_TILED, M, N, K) == (TILING_PREFILL_TILED, 21, 1), (M, N, K)  # no workspace, no slices
    for M, N, K in [(50, 4096, 11008), (62, 4096, 5760), (54, 3745, 9248), (62, 1359, 5920), (58, 8877, 6144), (51, 3520, 5760)]:
        tiling, tile, slices = w4a8_route(ROUTE_SPLITK, M, N, K)
        assert tiling == TILING_PREFILL_TILED and 21 <= tile <= 31 and slices == 1, (M, N, K)


def test_tiles_for_many_tokens_are_those_that_measured_faster():
    """Beyond 512 tokens: on the border between the large-M kernel and the medium-M kernel (21 .. 31), and between 64 x 192 (16) and
    64 x 256 (13), where choices by kManyTokensTileCosts alone took 4 to 28 % longer on cold weights."""
    for (M, N, K), tile in {(586, 3072, 1024): 6, (1263, 2240, 1024): 16, (1138, 2048, 1024): 16, (768, 3264, 3680): 28, (520, 3865, 3200): 28,
                            (689, 4224, 15808): 16, (629, 4331, 8128): 16,
                            (1085, 2880, 8416): 16, (615, 4296, 5792): 16}.items():
        for entry in (ROUTE_GEMM_TILED, ROUTE_SPLITK):
            assert w4a8_route(entry, M, N, K) == (TILING_PREFILL_TILED, tile, 1), (M, N, K)
    for (M, N, K), tile in {(2048, 10240, 8192): 32, (718, 21888, 13184): 33, (1024, 27648, 5120): 1, (1024, 5120, 5120): 15}.items():
        assert w4a8_route(ROUTE_SPLITK, M, N, K)[1] == tile, (M, N, K)
