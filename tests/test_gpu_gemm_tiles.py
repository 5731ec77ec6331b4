"""bf16 products at the sizes where the choice of tile, the padded token rows and the split contraction can go wrong: every tile
shape at ragged edges, few tokens (64-row tiles, down and dX products cut into shares), shares of different lengths, token counts
one short of and one past a k-slice, experts with fewer rows than a slice.  Against the float64 oracle at the bf16 tolerance
of the other parity tests."""
import os
import subprocess
import sys

import pytest

from tests.test_gpu_experts import run_experts_case
from tests.test_gpu_parity import run_fwd_bwd_case

pytestmark = pytest.mark.gpu


# T, d, F, K, and kernels of interest that the launchers take (product=tile or product=tile/shares; test_gemm_routes.py checks them)
CASES = [
    (17, 512, 1365, 170, "gate_up=64x128 dx=64x128/2"),                # fewer tokens than a k-slice; shares of a contraction with a tail
    (33, 1024, 2736, 342, "gate_up=64x128 down=64x128/4"),             # one token past a slice
    (129, 256, 5461, 682, "dw=192x128 down=64x128/8 dx=64x128/8"),     # one row past a tile; 171 slices in shares of 21 and 22
    (1999, 768, 2048, 409, "dw=128x192 down=64x128"),  # token rows padded by 17
    (17, 64, 1030, 128, "gate_up=64x128 dw=64x128 down=64x128/4 dx=64x128/8"),
    (65, 64, 8200, 1025, "gate_up=128x128 dw=128x128"),
    (97, 544, 2736, 342, "dw=128x192"),
    (33, 768, 5461, 682, "down=64x128/8 dx=64x128/7"),
    (2100, 128, 1365, 170, "gate_up=192x128"),
    (4100, 128, 520, 65, "gate_up=128x192"),
    (2600, 64, 2736, 342, "dz=64x128 down=64x128/6"),
    (4100, 64, 2736, 342, "down=128x128/6 dx=128x128/7"),
    (900, 512, 5461, 682, "dz=192x128 dx=128x128/7"),
    (1537, 288, 5461, 682, "gate_up=128x128 down=128x128/6"),
    (1100, 288, 8200, 1025, "down=128x128/7 dx=128x128/8"),
    (513, 768, 8200, 1025, "dz=192x128"),
    (400, 1024, 8200, 1025, "dz=128x192"),
    (700, 1536, 4100, 512, "down=128x128/3 dx=128x128/2"),
    (1300, 1024, 8200, 1025, "down=192x128/4 dx=192x128/4"),
    # d % 64 == 32, which the large tiles of gemm_pingpong.h leave to these
    (700, 96, 8200, 1025, "gate_up=256x256"),
    (400, 1056, 8200, 1025, "gate_up=256x192"),
    (300, 992, 11008, 1376, "gate_up=192x256"),
    (1200, 1056, 2736, 342, "gate_up=256x128"),
    (900, 800, 11008, 1376, "gate=192x256"),
    (2200, 544, 5461, 682, "gate=256x256"),
    (1200, 1056, 8200, 1025, "gate=256x192"),
    (1700, 992, 4100, 512, "dz=256x128"),
]


@pytest.mark.parametrize("T,d,F,K,kernels", CASES)
def test_tiles_shares_and_padded_rows(T, d, F, K, kernels):
    run_fwd_bwd_case("tiles " + kernels, 98, T, d, F, K, "bf16")


def test_experts_with_fewer_rows_than_a_slice():
    run_experts_case("few rows", 980, [1, 0, 31, 33, 64, 5, 100, 2], 128, 333, 41, "bf16")


@pytest.mark.parametrize("tile", ["256", "192", "128"])
def test_contraction_tails_without_padding_on_every_tile(tile):
    """d % 32 != 0: gate, up and dZ' end inside a k-slice that nothing pads.  The environment (read once per process, hence the child
    process) names the tile; ragged rows and columns, several tiles, experts with and without rows."""
    code = ("from tests.test_gpu_experts import run_experts_case\n"
            "from tests.test_gpu_parity import run_fwd_bwd_case\n"
            "run_fwd_bwd_case('tails', 99, 300, 104, 530, 66, 'bf16')\n"
            "run_fwd_bwd_case('tails', 99, 777, 264, 1031, 129, 'bf16')\n"
            "run_experts_case('tails', 990, [300, 0, 40, 65], 104, 530, 66, 'bf16')\n"
            "print('ok')\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, env=dict(os.environ, MOC_GEMM_TILE=tile), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-3000:] + r.stderr[-3000:]
