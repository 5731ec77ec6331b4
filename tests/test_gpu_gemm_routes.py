"""The kernels that run are those the cases name: every case of test_gpu_large_tiles.py and test_gpu_gemm_tiles.py once under the profiler.  (That
the names are what the functions of gemm_plan.h say is test_gemm_routes.py's, on the CPU; here the launchers show that they follow them.)"""
import re

import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import paper_2511_09323_amd as moc
from tests.test_gpu_experts import MIXTRAL_180M
from tests.test_gpu_gemm_tiles import CASES as TILE_CASES
from tests.test_gpu_large_tiles import CASES, EXPERT_CASES

pytestmark = pytest.mark.gpu


def normal(*shape):
    return torch.randn(shape, device="cuda", dtype=torch.bfloat16)


def kernels_of(call):
    """Names of the library's kernels that `call` launches, in their order."""
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    events = [e for e in p.events() if "moc::" in e.name and "kernel" in e.name]
    return [e.name for e in sorted(events, key=lambda e: e.time_range.start)]


def products_of(call):
    """product=tile of the products of one forward and backward; shares end in /."""
    call()
    torch.cuda.synchronize()
    names = kernels_of(call)
    if not any("bwd_expand" in n for n in names):      # the profiler's first use in a process may come too late for it
        names = kernels_of(call)
    tiles, before = [], None
    for n in names:
        m = re.search(r"gemm_bf16_(pp|mfma)(?:_[a-z]+)?_kernel<(\d+), (\d+),", n)
        if m:
            tiles.append("%s%sx%s" % ("pp" if m.group(1) == "pp" else "", m.group(2), m.group(3)))
        elif "reduce_shares_kernel" in n:
            tiles[-1] += "/"
        elif "topk_rows" in n:
            before = len(tiles)
    order = (["gate_up"] if before == 1 else ["gate", "up"]) + ["down", "dz", "dw", "dx"]
    assert len(order) == len(tiles), names
    return ["%s=%s" % p for p in zip(order, tiles)]


def wanted(kernels):
    return {re.sub(r"/\d+$", "/", w) for w in kernels.split() if "=" in w}


@pytest.mark.parametrize("T,d,F,K,kernels", CASES + TILE_CASES)
def test_layers_run_the_kernels_they_name(T, d, F, K, kernels):
    x, dy, w = normal(T, d), normal(T, d), [normal(F, d) for _ in range(3)]

    def call():
        _, idx, gv, uv = moc.moc_ffn_fwd(x, *w, K)
        moc.moc_ffn_bwd(x, *w, idx, gv, uv, dy)

    got = products_of(call)
    assert wanted(kernels) <= set(got), got


@pytest.mark.parametrize("counts,d,F,K,kernels", EXPERT_CASES + [(MIXTRAL_180M, 512, 1376, 256, "gate_up=pp256x256 dz=pp256x128 dw=pp192x256")])
def test_experts_run_the_kernels_they_name(counts, d, F, K, kernels):
    T, E = sum(counts), len(counts)
    off = [sum(counts[:e]) for e in range(E + 1)]
    x, dy, w = normal(T, d), normal(T, d), [normal(E, F, d) for _ in range(3)]

    def call():
        _, idx, gv, uv = moc.moc_ffn_fwd_experts(x, off, *w, K)
        moc.moc_ffn_bwd_experts(x, off, *w, idx, gv, uv, dy)

    got = products_of(call)
    assert wanted(kernels) <= set(got), got
