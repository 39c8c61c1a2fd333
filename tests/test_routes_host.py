"""Which kernel the library's own choice runs, and which calls it refuses: pure functions of the shape (for the 256 compute
units that are assumed where there is no GPU).  No kernel is launched here."""
import ctypes

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
