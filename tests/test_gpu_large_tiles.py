"""bf16 products on the large tiles of gemm_pingpong.h where they can go wrong: every tile shape with ragged rows and columns, one and two
slices (the pipeline is deeper than that), odd numbers of slices, contraction ends inside a slice and inside the second operand pair, several
tiles to a workgroup, shares of different lengths, experts with no and few rows; and the products they leave to gemm_mfma.h (d % 64
== 32).  Against the float64 oracle at the bf16 tolerance of the other parity tests."""
import pytest
import torch

import paper_2511_09323_amd as moc
from paper_2511_09323_amd import inputs
from tests import parity as P
from tests.test_gpu_experts import run_experts_case
from tests.test_gpu_parity import gpu_layer, run_fwd_bwd_case

pytestmark = pytest.mark.gpu

# T, d, F, K, and kernels of interest that the launchers take (product=tile or product=tile/shares, pp: gemm_pingpong.h;
# test_gemm_routes.py checks them)
CASES = [
    (513, 64, 11008, 1376, "gate_up=pp128x256"),               # one row past a tile; a single slice, several tiles to a workgroup
    (700, 64, 11008, 1376, "gate_up=pp192x256"),
    (1025, 64, 5461, 682, "gate_up=pp256x128"),
    (5000, 192, 1030, 128, "gate_up=pp256x192"),               # three slices: an odd one at the end of every tile
    (1025, 128, 5461, 682, "gate_up=pp256x256"),
    (1025, 64, 11008, 1376, "dz=pp128x256"),
    (3000, 64, 4100, 512, "dz=pp256x128"),
    (65, 768, 5461, 682, "dw=pp256x256"),                      # one token past a slice
    (17, 320, 11008, 1376, "dw=pp256x128"),                    # fewer tokens than a slice
    (17, 576, 11008, 1376, "dw=pp256x192"),
    (300, 1536, 1365, 170, "dw=pp128x256"),
    (17, 320, 16001, 2000, "dw=pp192x256"),
    (6100, 2048, 200, 25, "down=pp192x256 dx=pp192x256"),      # a contraction of four slices that ends inside the last
    (4100, 1536, 520, 65, "down=pp256x128"),
    (5000, 1536, 200, 25, "dx=pp256x128"),                     # two operand pairs of four slices each
    (17, 64, 16001, 2000, "dx=pp256x128/16"),                  # 502 slices in shares of 31 and 32, one of them across both operand pairs
    (1025, 96, 5461, 682, "gate_up=256x256"),
    (513, 800, 8200, 1025, "gate_up=192x256"),
]


@pytest.mark.parametrize("T,d,F,K,kernels", CASES)
def test_large_tiles(T, d, F, K, kernels):
    run_fwd_bwd_case("large tiles " + kernels, 97, T, d, F, K, "bf16")


# Products over the channels whose weights come from memory (long_product), with the scratch that a workspace holds for their shares
LONG_CASES = [
    (40, 2048, 2050, 256, "down=64x128/8 dx=64x128/8"),        # as many shares as there is scratch for; a contraction of 32 slices and two channels
    (300, 2048, 2050, 256, "down=128x128/5 dx=128x128/5"),
    (130, 2112, 2000, 250, "down=64x128/5 dx=128x128/7"),
    (192, 2560, 2600, 325, "down=64x128/4 dx=128x128/6"),     # as many rows as a tile of 192 has
    (700, 2048, 2100, 262, "down=128x128/2 dx=pp128x256/5"),
    (900, 1536, 2100, 262, "dx=192x128/4"),
    (560, 2304, 3300, 412, "down=192x128/4"),
    (1100, 1280, 3300, 412, "down=128x128/2 dx=pp192x256/8"),
    (1500, 2048, 2056, 257, "down=128x128 dx=pp192x256/4"),
    (2047, 2048, 2056, 257, "dx=pp128x256/2"),
]


@pytest.mark.parametrize("T,d,F,K,kernels", LONG_CASES)
def test_long_products(T, d, F, K, kernels):
    run_fwd_bwd_case("long products " + kernels, 94, T, d, F, K, "bf16")


# Weight gradients in whole rounds of tiles and a second launch for the rows behind them, whose contraction runs in shares (batch3_split): rows of
# the first launch, its tile, tile and shares of the second.
SPLIT_CASES = [
    (2049, 1536, 3700, 462, "3584 pp256x256 pp128x256/7"),     # one token past a slice; 116 rows left
    (2300, 2048, 2731, 341, "2560 pp256x256 pp128x256/4"),     # 171: a second tile of 43
]
# 256 x 256 tiles in the second launch.  At this size a row of 2600 may have its K-th and K + 1-th gate values closer than the rounding of sums of 2048
# products (up to 2^-24 sqrt(2048) = 2.7e-6 of their size), so the gradients are taken from the stored set, whatever it is.
STORED_SPLIT_CASES = [(2600, 2048, 6200, 775, "5376 pp256x256 pp256x256/2")]


@pytest.mark.parametrize("T,d,F,K,plan", SPLIT_CASES)
def test_weight_gradients_in_two_launches(T, d, F, K, plan):
    run_fwd_bwd_case("split " + plan, 93, T, d, F, K, "bf16")


@pytest.mark.parametrize("T,d,F,K,plan", STORED_SPLIT_CASES)
def test_weight_gradients_in_two_launches_from_a_stored_set(T, d, F, K, plan):
    print("[case] split %s T=%d d=%d F=%d K=%d" % (plan, T, d, F, K), flush=True)
    L = inputs.make_layer(93, T, d, F, "bf16", with_dy=True)
    g = gpu_layer(L, "bf16")
    w = (g["wg"], g["wu"], g["wd"])
    _, idx, gvals, uvals = moc.moc_ffn_fwd(g["x"], *w, K)
    got = moc.moc_ffn_bwd(g["x"], *w, idx, gvals, uvals, g["dy"])
    torch.cuda.synchronize()
    want = P.oracle_backward_for(L, idx.cpu().numpy(), P.to_np(gvals), P.to_np(uvals))
    for name, a, b in zip(("dx", "dwg", "dwu", "dwd"), got, want):
        P.assert_close(name, P.to_np(a), b, P.TOL["bf16"])


# rows of the experts, d, F, K, kernels (a large tile of dw and down with its rounds of the workgroups: xN)
EXPERT_CASES = [
    ([700, 0, 1, 513, 300, 64, 257, 900], 128, 2736, 342, "gate_up=pp192x256 dz=128x128 dw=pp256x128"),      # one short of and past a tile, no and one row
    ([2000, 33], 192, 1030, 128, "gate_up=pp256x128"),
    # contractions over the channels, ragged (330 % 64 = 10), in two rounds, the second of which goes backwards
    ([2600, 2100, 0, 9, 4300, 2250, 1900, 3000], 1024, 330, 41, "gate_up=pp256x128 dz=pp256x128 dw=pp128x256 x1 down=pp192x256 x2 dx=pp192x256"),
]


@pytest.mark.parametrize("counts,d,F,K,kernels", EXPERT_CASES)
def test_experts_on_large_tiles(counts, d, F, K, kernels):
    """All products of the experts, as far as `kernels` says so: gate and up in one launch, down and dX (two operand pairs) with unequal row counts."""
    run_experts_case("large tiles " + kernels, 970, counts, d, F, K, "bf16")


@pytest.mark.parametrize("T,d,F,K", [(513, 64, 2731, 341), (1025, 128, 5461, 682), (2047, 1536, 200, 25)])
def test_nothing_outside_the_operands_counts(T, d, F, K):
    """Every operand lies between NaN: what a tile loads past an edge must not reach a result."""
    L = inputs.make_layer(96, T, d, F, "bf16", with_dy=True)

    def between_nan(a):
        t = P.to_dev(a, "bf16")
        buf = torch.full((t.numel() + 2 * 65536,), float("nan"), dtype=t.dtype, device="cuda")
        inner = buf[65536:65536 + t.numel()].view(t.shape)
        inner.copy_(t)
        return inner

    def run(place):
        x, wg, wu, wd, dy = (place(L[n]) for n in ("x", "wg", "wu", "wd", "dy"))
        ws = [torch.full((moc.workspace_bytes(T, d, F, K, torch.bfloat16, op) // 2 + 1,), float("nan"), dtype=torch.bfloat16, device="cuda")
              .view(torch.uint8) for op in (0, 1)]
        y, idx, gv, uv = moc.moc_ffn_fwd(x, wg, wu, wd, K, ws=ws[0])
        return (y, idx, gv, uv) + tuple(moc.moc_ffn_bwd(x, wg, wu, wd, idx, gv, uv, dy, ws=ws[1]))

    for a, b in zip(run(between_nan), run(lambda a: P.to_dev(a, "bf16"))):
        assert torch.isfinite(a.float()).all()
        assert torch.equal(a, b)


def _fwd_bwd(kind, L, F, K, fill):
    """Outputs of one forward and backward of a kind of layer on workspaces that hold `fill`."""
    x, wg, wu, wd, dy = (L[n] for n in ("x", "wg", "wu", "wd", "dy"))
    T, d = x.shape

    def ws(op):
        return torch.full((moc.workspace_bytes(T, d, F, K, torch.bfloat16, op) // 2 + 1,), fill, dtype=torch.bfloat16, device="cuda").view(torch.uint8)

    if kind == "dense":
        y, g, u = moc.moc_swiglu_fwd(x, wg, wu, wd, ws=ws(3))
        return (y, g, u) + tuple(moc.moc_swiglu_bwd(x, wg, wu, wd, g, u, dy, ws=ws(4)))
    if kind == "experts":
        off = [0, T // 2 + 13, T]
        w = [torch.stack([t, t.flip(0)]) for t in (wg, wu, wd)]
        y, idx, gv, uv = moc.moc_ffn_fwd_experts(x, off, *w, K, ws=ws(0))
        return (y, idx, gv, uv) + tuple(moc.moc_ffn_bwd_experts(x, off, *w, idx, gv, uv, dy, ws=ws(1)))
    if kind == "grouped":
        y, idx, gv, uv = moc.moc_ffn_fwd_grouped(x, wg, wu, wd, 2, 8, ws=ws(0))
    elif kind == "keyed":
        y, idx, gv, uv = moc.moc_ffn_fwd_keyed(x, wg, wu, wd, K, "abs_silu", ws=ws(5))
    else:
        y, idx, gv, uv = moc.moc_ffn_fwd(x, wg, wu, wd, K, ws=ws(0))
    return (y, idx, gv, uv) + tuple(moc.moc_ffn_bwd(x, wg, wu, wd, idx, gv, uv, dy, ws=ws(1)))


@pytest.mark.parametrize("kind,T,d,F,K", [
    ("rows", 6100, 2048, 200, 25), ("all", 6100, 2048, 200, 200), ("grouped", 6100, 2048, 200, 50), ("keyed", 6100, 2048, 200, 25),
    ("dense", 6100, 2048, 200, 200), ("experts", 12000, 2048, 200, 25),
    ("rows", 520, 1024, 29990, 25000),                         # lists too long for the registers: topk_rows_lds_kernel
])
def test_dense_operands_are_zero_to_the_end_of_their_rows(kind, T, d, F, K):
    """Slices of the large tiles are 64 wide, those of gemm_mfma.h 32: with F % 64 in 1 .. 32 only the former read the last 32 columns of Z', dG and dU,
    which everything that writes those arrays has to clear, whatever the workspace held."""
    L = {n: P.to_dev(a, "bf16") for n, a in inputs.make_layer(95, T, d, F, "bf16", with_dy=True).items()}
    for a, b in zip(_fwd_bwd(kind, L, F, K, float("nan")), _fwd_bwd(kind, L, F, K, 0.0)):
        assert torch.isfinite(a.float()).all()
        assert torch.equal(a, b)
