"""bf16 decode with both projections as streams (decode_dense.h): layers that decode_dense_pays sends there and where the kernels can go wrong: a last
slice of columns that hangs over d, ranges of channels that end inside a step of 32 or a group of four, one range (nothing to add) and many,
wavefronts with more steps than pieces under way or none, every number of chunks of the selection, every group size, all channels
selected.  Against the float64 oracle at the bf16 tolerance of the other parity tests."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2511_09323_amd as moc
from tests import test_gpu_keyed
from tests.test_gpu_grouped import run_grouped_decode
from tests.test_gpu_parity import run_decode_case

pytestmark = pytest.mark.gpu


# (tests/test_gemm_routes.py has the ranges of channels that the down projection of each takes)
CASES = [
    (16, 64, 1024, 512), (7, 512, 5, 5), (6, 576, 37, 37),              # one range; five channels; a slice of which half lies past d
    (16, 512, 129, 60), (16, 768, 2051, 1000), (7, 1024, 4099, 3700),   # part-filled steps and fours
    (16, 1536, 4096, 512), (10, 2048, 5461, 683), (6, 2048, 5461, 1100),
    (16, 2112, 2900, 400), (12, 4096, 2052, 300),                       # slices of 128 columns, the last one half past d
    (16, 4096, 11008, 1376), (5, 512, 23440, 10000), (16, 1024, 12345, 2500), (13, 512, 32768, 12000),      # three, six and sixteen chunks of the selection
    (3, 4096, 4100, 4100), (4, 2048, 8200, 6200),                       # few tokens that select most channels
]
GROUPED_CASES = [(16, 4096, 2052, 1, 4), (13, 2048, 5464, 2, 8), (16, 512, 1376, 3, 4), (16, 1536, 8208, 3, 16)]


@pytest.mark.parametrize("B,d,F,K", CASES)
def test_dense(B, d, F, K):
    run_decode_case("dense", 71, B, d, F, K, "bf16")


@pytest.mark.parametrize("B,d,F,a,b", GROUPED_CASES)
def test_dense_grouped(B, d, F, a, b):
    run_grouped_decode("dense", 72, B, d, F, a, b, "bf16")


def _layer(B, d, F, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.randn(s, device="cuda", generator=gen)
    return r(B, d).bfloat16(), [(r(F, d) * 0.02).bfloat16() for _ in range(3)]


def test_rows_that_are_not_finite_reach_only_tokens_that_selected_them():
    """Infinities and a NaN in rows of W_down (and W_up): a token that did not select the channel gets what it would without them."""
    B, d, F, K = 16, 2048, 5461, 683
    x, (wg, wu, wd) = _layer(B, d, F, 3)
    y0, idx = moc.moc_ffn_decode(x, wg, wu, wd, K)
    selected = torch.zeros(B, F, dtype=torch.bool, device="cuda").scatter_(1, idx.long(), True)
    some = [int(j) for j in torch.nonzero((selected.sum(0) > 0) & (selected.sum(0) < B)).flatten()[[0, 77, -1]]]
    wd[some[0], 5], wd[some[1], 700], wd[some[2], d - 1] = float("inf"), float("nan"), float("-inf")
    wu[some[1], 3] = float("inf")
    y, idx2 = moc.moc_ffn_decode(x, wg, wu, wd, K)
    assert torch.equal(idx, idx2)
    clean = torch.ones(B, d, dtype=torch.bool, device="cuda")
    for j, c in ((some[0], 5), (some[1], None), (some[2], d - 1)):
        if c is None:
            clean[selected[:, j]] = False      # (its u is infinite or NaN)
        else:
            clean[selected[:, j], c] = False
    assert torch.isfinite(y[clean]).all() and not torch.isfinite(y[~clean]).any()
    # the same sums but for the order of the additions: at most two bf16 steps apart
    torch.testing.assert_close(y[clean].float(), y0[clean].float(), rtol=2 ** -6, atol=1e-3 * y0.float().abs().max().item())


def test_calls_that_follow_each_other_share_a_workspace():
    """Counters and shares of one call must not reach the next: large and small layers in turn, and replays of a captured call."""
    sizes = [(16, 2048, 5461, 683), (16, 512, 1024, 1000), (16, 4096, 2052, 500)]
    layers = [(_layer(B, d, F, 9 + i), K) for i, (B, d, F, K) in enumerate(sizes)]
    ws = torch.full((max(moc.workspace_bytes(B, d, F, K, torch.bfloat16, 2) for B, d, F, K in sizes),), 255, dtype=torch.uint8, device="cuda")
    want = [moc.moc_ffn_decode(x, *w, K)[0] for (x, w), K in layers]
    for _ in range(3):
        for ((x, w), K), y in zip(layers, want):
            assert torch.equal(moc.moc_ffn_decode(x, *w, K, ws=ws)[0], y)
    (x, w), K = layers[0]
    out = (torch.empty_like(x), None)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        moc.moc_ffn_decode(x, *w, K, ws=ws, out=out)
    for i in range(4):
        out[0].zero_()
        (x2, w2), K2 = layers[1 + i % 2]
        moc.moc_ffn_decode(x2, *w2, K2, ws=ws)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[0], want[0])


@pytest.mark.parametrize("key", ["silu", "abs_silu"])
def test_dense_keyed(key):
    test_gpu_keyed.test_keyed_decode(16, 1536, 4096, 700, key)


def replays_of_a_persistent_call():
    """(in a process with MOC_DECODE_PERSISTENT=1)  Replays repeat the host's share of the tag, the workspace's generation tells them apart: streamed
    calls between them must leave it alone."""
    B, d, F, K = 16, 1024, 8192, 1024
    x, w = _layer(B, d, F, 21)
    dt = torch.bfloat16
    ws = torch.full((moc.workspace_bytes(B, d, F, K, dt, 2),), 0xAB, dtype=torch.uint8, device="cuda")
    out = (torch.empty_like(x), torch.empty((B, K), dtype=torch.int32, device="cuda"))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        moc.moc_ffn_decode(x, *w, K, ws=ws, out=out)
    for i in range(6):
        x.copy_(_layer(B, d, F, 30 + i)[0])
        want = moc.moc_ffn_decode(x, *w, K)      # (a workspace of its own)
        if i % 3 != 2:
            moc.moc_ffn_decode_keyed(x, *w, K, "silu", ws=ws)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[1], want[1]) and torch.equal(out[0], want[0]), "replay %d" % i


def test_streamed_calls_between_replays_of_a_persistent_call():
    code = "import tests.test_gpu_decode_dense as t\nt.replays_of_a_persistent_call()\nprint('ok')\n"
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, env=dict(os.environ, MOC_DECODE_PERSISTENT="1"), capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-3000:] + r.stderr[-3000:]
