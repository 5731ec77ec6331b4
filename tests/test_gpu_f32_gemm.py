"""The fp32 matrix-core products (gemm_f32.h) at the sizes where they can go wrong: one row, tiles cut off in every
dimension, contractions shorter than a k-slice and ending inside a 4-k chunk, and sizes on both sides of each
tile choice (16 x 32 and 32 x 32 with the slices split over wavefronts, 32 x 32, 64 x 64).  Forward and backward against the
float64 oracle at the fp32 tolerance of the other parity tests: sums of up to 2 x 1100 products carry a relative error
of a few 1e-7, the tolerance is 1e-4."""
import pytest

from tests.test_gpu_parity import run_fwd_bwd_case

pytestmark = pytest.mark.gpu


# T, d, F, K, and kernels of interest that the launchers take (s: k-slices split over wavefronts; test_gemm_plan.py checks them)
CASES = [
    (1, 4, 5, 2, "gate_up=32x32 down=16x32s dw=16x32s"),               # smaller than every tile and slice
    (17, 36, 33, 9, "gate_up=32x32 dz=16x32s dx=16x32s"),              # one row and one column past a tile
    (64, 128, 127, 16, "down=16x32s"),                                 # contraction over F ends inside a chunk
    (65, 132, 1025, 128, "down=16x32s dw=32x32"),                      # nine slices of the down product, the last one k long
    (300, 260, 1000, 100, "dw=32x32 dz=32x32"),                        # T ends inside a slice
    (300, 260, 1100, 100, "dw=64x64"),                                 # the same on the larger tiles, cut in d and F
    (1100, 260, 500, 60, "down=32x32 dx=32x32"),
    (1100, 260, 1031, 100, "gate_up=64x64 dz=64x64 down=32x32s dx=32x32s dw=32x32s"),
    (2100, 516, 200, 25, "down=64x64 dx=64x64"),                       # k-contiguous x k-major, two segments, cut in T and d
]


@pytest.mark.parametrize("T,d,F,K,kernels", CASES)
def test_f32_products_at_tile_edges(T, d, F, K, kernels):
    run_fwd_bwd_case("f32-tiles " + kernels, 97, T, d, F, K, "f32")


# Products over the channels whose contraction runs in shares (f32_shares; the tile of f32_tile is the one of the whole product): what down and dX take.
SHARE_CASES = [
    (64, 768, 2048, 256, "down=16x32s/4 dx=16x32s/5"),
    (100, 512, 1373, 172, "down=16x32s/4 dx=16x32s/4"),                # both ends of a share inside the contraction's tail, a slice cut in a chunk
    (65, 132, 1025, 128, "down=32x32/6 dx=16x32s/6"),                # 17 and 18 slices; a row and four columns past a tile
    (256, 512, 1376, 172, "down=16x32s dx=32x32/4"),
    (257, 772, 2050, 409, "down=16x32s dx=32x32/3"),
    (1100, 260, 1031, 100, "down=32x32/3 dx=32x32/4"),
    (1024, 512, 1376, 172, "down=32x32s dx=32x32/3"),                  # and whole
]


@pytest.mark.parametrize("T,d,F,K,kernels", SHARE_CASES)
def test_f32_products_in_shares(T, d, F, K, kernels):
    run_fwd_bwd_case("f32-shares " + kernels, 96, T, d, F, K, "f32")
