"""The row selection of row_cut.h on rows that its usual path (one histogram, a handful of values in the cut's bin) does not
resolve: outliers that push everything else into one bin, more ties than a wavefront ranks, cuts at zero and among the negative
values, powers of two over the whole exponent range.  Index sets are compared exactly; the values are exact by construction
(given fp32 rows, or one-hot inputs that make the gate a column of W_gate)."""
import numpy as np
import pytest
import torch

import paper_2511_09323_amd as moc
from oracle import moc_oracle as O
from paper_2511_09323_amd import inputs
from tests import parity as P
from tests.test_gpu_parity import _topk_case

pytestmark = pytest.mark.gpu


def hard_rows(F, seed):
    rng = np.random.default_rng(seed)
    g = rng.standard_normal((8, F)).astype(np.float32)
    g[0, F // 2] = 1e6                                                   # one outlier: all others share a bin
    g[1] = np.sign(g[1]) * np.exp2(np.floor(rng.uniform(-120, 120, F)))  # geometric
    g[2] = np.round(g[2] * 2) / 2                                        # hundreds of ties per value
    g[3] = -np.abs(g[3]) - 1                                             # all negative
    g[4] = np.where(rng.random(F) < 0.9, 0.0, g[4])                      # mostly (signed) zeros
    g[4, ::3] *= -1
    g[5] = np.where(rng.random(F) < 0.5, 1.0, np.nextafter(np.float32(1), np.float32(2)))
    g[6] *= 1e-42                                                        # denormal
    g[7, :] = -2.5
    return g.astype(np.float32)


@pytest.mark.parametrize("F", [5, 64, 1376, 5461, 11008])
def test_rows_the_usual_path_does_not_resolve(F):
    g = hard_rows(F, F)
    for K in sorted({1, F // 8, F // 2, F - 1, F} - {0}):
        _topk_case(g, K)


def padded(g):
    """The rows with a pitch of whole 16-byte blocks (odd rows then stay in registers), infinities and NaN behind their ends."""
    n, F = g.shape
    base = torch.full((n, (F + 3) // 4 * 4 + 4), float("inf"), device="cuda")
    base[::2, F:] = float("nan")
    base[:, :F] = torch.from_numpy(g).cuda()
    return base[:, :F]


def check_rows(g, K):
    _topk_case(g, K)
    idx, gsel = moc.moc_topk_rows(padded(g), K)
    torch.cuda.synchronize()
    want = by_key(g, K)
    np.testing.assert_array_equal(idx.cpu().numpy(), want)
    np.testing.assert_array_equal(gsel.cpu().numpy(), np.take_along_axis(g, want, axis=1))


def outlier_rows(F, seed):
    """Rows whose bins end far below the maximum: one outlier, outliers that share the last bin with and without the cut among them,
    positive values so few that the sampled quarter of the row may hold none."""
    rng = np.random.default_rng(seed)
    g = rng.standard_normal((6, F)).astype(np.float32)
    g[0, F // 3] = 1000.0
    n = max(1, F // 20)
    g[1, rng.permutation(F)[:n]] = 1000.0 + np.arange(n)                 # distinct
    g[2, rng.permutation(F)[:n]] = 1000.0                                # equal
    g[3] = rng.standard_t(1.5, F)
    g[4] = np.where(np.arange(F) % 4 == 1, np.abs(g[4]), -np.abs(g[4]))  # nothing positive in the sampled quarter
    g[5] = np.where(np.arange(F) % 4 == 0, 1e37 * np.abs(g[5]), g[5])    # all of the sampled quarter far above the rest
    return g.astype(np.float32)


@pytest.mark.parametrize("F", [64, 1376, 5461, 11008, 14336])
def test_rows_with_outliers(F):
    g = outlier_rows(F, F)
    for K in sorted({1, F // 40, F // 20, F // 20 + 1, F // 8, F // 5, F // 3} - {0}):
        check_rows(g, K)


@pytest.mark.parametrize("F", [9, 1376, 5461, 11007])
def test_cuts_below_zero(F):
    """More than a third of the row: bins on both sides of zero; K on both sides of that line, of the slots a thread writes at a time
    (256 and 512), and the whole row."""
    g = np.concatenate([outlier_rows(F, F + 2), hard_rows(F, F + 2)])
    g[0] -= 0.5
    for K in sorted({F // 3, F // 3 + 1, F // 2 + 3, 3 * F // 4, F - 1, F, min(F, 256), min(F, 257), min(F, 513)}):
        check_rows(g, K)


@pytest.mark.parametrize("F", [64, 1376, 2051, 5461, 11008, 32768])
def test_ties_at_the_ends_of_a_thread_wavefront_and_chunk(F):
    """Two values only: the cut's channel is the K-th of the equal ones, at every kind of place."""
    g = np.full((3, F), 1.0, dtype=np.float32)
    g[1, ::3] = 2.0
    g[2, F // 2:] = 2.0
    for K in sorted({k for k in (1, 4, 5, 255, 256, 257, 1023, 1024, 1025, 2048, 2049, 4097, F // 2, F // 2 + 1, F - 1) if 1 <= k <= F}):
        check_rows(g, K)


@pytest.mark.parametrize("B,d,F", [(1, 64, 5), (1, 512, 1376), (3, 256, 5461), (4, 128, 11008), (2, 64, 32768)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_decode_selection_on_hard_rows(B, d, F, dtype):
    L = inputs.make_layer(96, B, d, F, dtype)
    rows = inputs.round_to_bf16(hard_rows(F, F + 1))                     # row r is the gate of a token whose input is one-hot at r
    L["wg"][:, :8] = rows.T
    for first in (0, 4):
        L["x"] = np.zeros((B, d), dtype=np.float32)
        for b in range(B):
            L["x"][b, (first + b) % 8] = 1.0
        G = {k: P.to_dev(v, dtype) for k, v in L.items()}
        want = rows[[(first + b) % 8 for b in range(B)]]
        for K in sorted({1, F // 8, F // 2, 3 * F // 4, F} - {0}):
            y, idx = moc.moc_ffn_decode(G["x"], G["wg"], G["wu"], G["wd"], K)
            torch.cuda.synchronize()
            ref = np.stack([np.flatnonzero(r) for r in O.topk_mask(want, K)])
            np.testing.assert_array_equal(idx.cpu().numpy(), ref)
            assert torch.isfinite(y).all()


def by_key(g, K):
    """The K channels of each row with the largest float keys (+NaN above +inf, -NaN below -inf, -0.0 equal to +0.0), ties to
    the lower channel, ascending."""
    u = (g + np.float32(0)).view(np.uint32).astype(np.int64)
    key = np.where(u >> 31, 0xFFFFFFFF - u, u + 0x80000000)
    return np.sort(np.argsort(-key, axis=1, kind="stable")[:, :K], axis=1)


def nonfinite_rows(F, seed):
    rng = np.random.default_rng(seed)
    g = rng.standard_normal((12, F)).astype(np.float32)
    inf = np.float32(np.inf)
    g[0, rng.random(F) < 0.9] = -inf                                     # a mask
    g[1] = -inf
    g[2, rng.random(F) < 0.3] = inf
    g[3, ::7], g[3, 1::7] = np.nan, -np.nan
    g[4] = np.nan
    g[5] = np.where(rng.random(F) < 0.5, -inf, -np.abs(g[5]))
    g[6] = np.where(rng.random(F) < 0.5, -3e38, 1e-6 * np.abs(g[6]))     # far below what the bins can count
    g[7, ::5], g[7, 2::5], g[7, 3::5] = -np.nan, inf, np.finfo(np.float32).min
    g[8, 1::9], g[8, 4::9] = np.nan, inf                                 # the cut among finite values below both
    g[9] = np.where(rng.random(F) < 0.5, np.float32(0), -inf)            # among zeros, among -inf
    g[9, ::17] = np.nan
    g[10] = np.where(rng.random(F) < 0.6, np.where(rng.random(F) < 0.5, np.float32(-0.0), np.float32(0)), -np.abs(g[10]))
    g[11] = np.exp2(rng.uniform(-120, 120, F)) * np.where(rng.random(F) < 0.5, -1, 1)     # by the digits of the keys
    return g


@pytest.mark.parametrize("F", [5, 64, 1376, 5461, 11008])
def test_rows_with_infinities_and_nans(F):
    g = nonfinite_rows(F, F)
    for K in sorted({1, F // 8, F // 2, F - 1, F} - {0}):
        idx, gsel = moc.moc_topk_rows(torch.from_numpy(g).cuda(), K)
        torch.cuda.synchronize()
        want = by_key(g, K)
        np.testing.assert_array_equal(idx.cpu().numpy(), want)
        np.testing.assert_array_equal(gsel.cpu().numpy(), np.take_along_axis(g, want, axis=1))
        idx, gsel = moc.moc_topk_rows(padded(g), K)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(idx.cpu().numpy(), want)


@pytest.mark.parametrize("B,d,F", [(1, 64, 5), (3, 256, 1376), (4, 128, 11008)])
def test_decode_selection_with_infinities(B, d, F):
    rows = inputs.round_to_bf16(nonfinite_rows(F, F + 1)[[0, 1, 5, 6, 8, 9, 10, 11]])
    if np.isinf(rows[3]).any():
        rows[3] = np.where(np.isinf(rows[3]), np.float32(-1e38), rows[3])
    L = inputs.make_layer(97, B, d, F, "f32")
    for row in rows:                                                     # one-hot tokens: 0 * -inf would be a NaN, so one row at a time
        L["x"] = np.zeros((B, d), dtype=np.float32)
        L["x"][:, 0] = 1.0
        L["wg"][:, 0] = row
        G = {k: P.to_dev(v, "f32") for k, v in L.items()}
        for K in sorted({1, F // 8, F // 2, F} - {0}):
            _, idx = moc.moc_ffn_decode(G["x"], G["wg"], G["wu"], G["wd"], K)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(idx.cpu().numpy(), np.repeat(by_key(row[None], K), B, axis=0))


@pytest.mark.parametrize("B,K,d", [(1, 3662, 4096), (1, 3663, 4096), (1, 4096, 4096), (1, 4097, 4096), (1, 8192, 4096), (2, 2730, 4096),
                                   (2, 2731, 4096), (4, 1525, 4096), (4, 1526, 4096), (4, 2730, 4096), (4, 2731, 4096), (4, 8192, 4096),
                                   (1, 4150, 512), (1, 4151, 512), (3, 2730, 1024), (3, 2731, 1024), (4, 5000, 4608), (2, 8192, 4608)])
def test_decode_on_both_sides_of_the_three_launch_line(B, K, d):
    """Half of F for one token, a third for more; below 8.5 MB of selected rows (two rows of d bf16 per selected channel) and where the
    rows are too long for the fused gather always."""
    F = 8192
    gen = torch.Generator(device="cuda").manual_seed(K)
    x = torch.randn((B, d), generator=gen, device="cuda").bfloat16()
    wg, wu, wd = [(torch.randn((F, d), generator=gen, device="cuda") * 0.02).bfloat16() for _ in range(3)]
    y, idx = moc.moc_ffn_decode(x, wg, wu, wd, K)
    g, u = x.float() @ wg.float().T, x.float() @ wu.float().T
    mask = torch.zeros_like(g).scatter_(1, idx.long(), 1.0)
    assert (mask.sum(1) == K).all() and (idx[:, 1:] > idx[:, :-1]).all()
    # what is selected lies above what is not, up to the rounding of sums of 4096 terms of size 0.02
    low = torch.where(mask > 0, g, float("inf")).amin(1)
    high = torch.where(mask > 0, float("-inf"), g).amax(1)
    assert (low >= high - 1e-4).all()
    ref = (torch.nn.functional.silu(g) * u * mask) @ wd.float()
    assert (y.float() - ref).norm() <= 1e-2 * ref.norm()                 # one rounding to 8 bits: 2e-3
