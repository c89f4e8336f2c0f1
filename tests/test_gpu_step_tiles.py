"""The tiled GEMM kernels that hold a whole K step of fragments: every count of K steps around the number of their LDS stages,
tiles that stick out of C along M and N, every epilogue.  Against float64; tolerances as in test_product_routes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_product_routes import EPI, _product, route   # noqa: E402

TILE_256x128, TILE_128x64 = 10, 11   # positions in the enumeration of gemm_route.h


def raw_route(M, N, K, epi):
    import ctypes as C
    from paper_2410_07192_amd import binding as pf
    f = pf.lib.pf_gemm_route
    f.restype, f.argtypes = C.c_int32, [C.c_int32, C.c_int64, C.c_int64, C.c_int64, C.c_int32, C.c_int32]
    return f(pf.PF_DTYPE_BF16, M, N, K, EPI[epi], 0) & 255


TALL = [(4096, 2048, 4096), (4000, 2040, 2880), (3841, 1928, 3008)]
TALL_EPI = ("plain", "bias", "gelu", "resid", "pre", "dact")
SLIM = [(1659, 768, 3072), (600, 2048, 1024), (1000, 1032, 1088), (1500, 776, 1344)]
# M, N, K, epilogues, kernel: K steps 1 .. 6 with four stages, 1 .. 4 with two
SHORT = [(1999, 2040, 64 * k, TALL_EPI, "tile 128x128 deep") for k in range(1, 7)]
SHORT += [(1659, 3072, 64 * k, ("bias", "gelu", "resid"), "tile 128x128") for k in range(1, 5)]


@pytest.mark.parametrize("M,N,K", TALL)
def test_these_run_on_256x128_tiles(M, N, K):
    assert {raw_route(M, N, K, e) for e in TALL_EPI} == {TILE_256x128}


@pytest.mark.parametrize("M,N,K,epis,kernel", SHORT)
def test_these_run_on_128x128_tiles(M, N, K, epis, kernel):
    assert {route("bf16", M, N, K, e) for e in epis} == {(kernel, 1)}


@pytest.mark.parametrize("M,N,K", SLIM)
def test_these_run_on_128x64_tiles(M, N, K):
    assert {raw_route(M, N, K, e) for e in ("plain", "bias", "gelu", "resid", "dact")} == {TILE_128x64}


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", SLIM)
def test_numbers_of_128x64_tiles(M, N, K):
    _product("bf16", M, N, K, TALL_EPI)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", TALL)
def test_numbers_of_256x128_tiles(M, N, K):
    _product("bf16", M, N, K, TALL_EPI)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,epis,kernel", SHORT)
def test_numbers_around_the_number_of_stages(M, N, K, epis, kernel):
    _product("bf16", M, N, K, epis)
