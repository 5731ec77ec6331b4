"""The fp32 matrix-core products (gemm_f32.h) at the sizes where they can go wrong: one row, tiles cut off in every
dimension, contractions shorter than a k-slice and ending inside a 4-k chunk, and sizes on both sides of each
tile choice (16 x 32 and 32 x 32 with the slices split over wavefronts, 32 x 32, 64 x 64).  Forward and backward against the
float64 oracle at the fp32 tolerance of the other parity tests: sums of up to 2 x 1100 products carry a relative error
of a few 1e-7, the tolerance is 1e-4."""
import pytest

from tests.test_gpu_parity import run_fwd_bwd_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,F,K", [
    (1, 4, 5, 2),              # smaller than every tile and slice
    (17, 36, 33, 9),           # one row and one column past a tile
    (64, 128, 127, 16),        # contraction over F ends inside a chunk
    (65, 132, 1025, 128),      # split k-slices, nine slices of the down product, the last one k long
    (300, 260, 1000, 100),     # weight gradients on 64 x 64 tiles, T ends inside a slice
    (1100, 260, 1031, 100),    # gate and up on 64 x 64 tiles
])
def test_f32_products_at_tile_edges(T, d, F, K):
    run_fwd_bwd_case("f32-tiles", 97, T, d, F, K, "f32")
