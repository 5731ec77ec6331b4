"""The streamed gate projection of bf16 decode with 2 to 16 tokens (decode_gate_stream_kernel) where it can go wrong: every number of k steps
per wavefront and shapes that leave wavefronts without any, fewer rows than workgroups, part-filled blocks of 16 rows, rows that do not divide
into fours, every group size, and the layers next to its range, which other kernels take (d % 64 != 0, d > 4096, one token).  Against the
float64 oracle at the bf16 tolerance of the other parity tests."""
import pytest
import torch

import paper_2511_09323_amd as moc
from tests.test_gpu_grouped import run_grouped_decode
from tests.test_gpu_parity import run_decode_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,d,F,K", [
    (2, 64, 5, 2), (16, 64, 1024, 128),           # one step: seven wavefronts have none; one row past a workgroup's four
    (3, 512, 1376, 172), (5, 576, 4099, 512),     # one step each; nine steps in twos, the last wavefronts empty
    (4, 768, 8192, 1024), (16, 1024, 8200, 1025),  # 32 rows a workgroup, exactly two blocks, and the first of a third
    (7, 1536, 333, 40), (15, 2048, 12345, 1543),  # three steps of four; 48 and 49 rows
    (2, 2112, 700, 87), (16, 4096, 4100, 512),    # 33 steps in fives; eight each
    (16, 96, 300, 37), (2, 4160, 300, 37), (1, 4096, 300, 37),
    (5, 64, 5, 2), (6, 2112, 700, 87),            # as with two tokens above, which few rows send to the dot products
    (5, 512, 23440, 2930), (2, 1024, 11720, 1465), (3, 2048, 5860, 732), (2, 4096, 1465, 183),      # the first F with non-temporal loads
    (5, 512, 23434, 2930), (3, 1024, 11716, 1465), (5, 2048, 5859, 732), (5, 4096, 1464, 183),      # and without
])
def test_streamed_gate(B, d, F, K):
    run_decode_case("streamed gate", 88, B, d, F, K, "bf16")


@pytest.mark.parametrize("B,d,F,a,b", [(2, 64, 8, 2, 8), (16, 512, 4104, 2, 8), (5, 1024, 12304, 3, 16), (4, 4096, 2052, 1, 4), (9, 576, 3000, 4, 8),
                                       (3, 1536, 4096, 2, 8), (2, 2048, 2052, 1, 4), (4, 2048, 5464, 2, 8),      # one block a workgroup, and more
                                       (5, 2048, 8192, 2, 8), (2, 4096, 3008, 3, 16)])                           # non-temporal
def test_streamed_gate_with_grouped_selection(B, d, F, a, b):
    run_grouped_decode("streamed gate", 87, B, d, F, a, b, "bf16")


@pytest.mark.parametrize("K", [8191, 8192, 8200, 8312, 9000])
def test_gather_with_more_slots_than_lanes(K):
    """16 tokens, 16 shares of the channels: a wavefront of the gather has 64, 65 and up to 71 slots, and reads the channels of 64 at a time."""
    run_decode_case("gather", 86, 16, 64, 9000, K, "bf16")


@pytest.mark.parametrize("B,d,F,K", [(3, 576, 1030, 128), (16, 4096, 523, 65)])
def test_nothing_outside_the_operands_counts(B, d, F, K):
    """x and W_gate lie between NaN: what is requested past a row, a token or a workgroup's rows must not reach a result."""
    gen = torch.Generator(device="cuda").manual_seed(5)

    def between_nan(*shape):
        n = 1
        for s in shape:
            n *= s
        buf = torch.full((n + 2 * 65536,), float("nan"), dtype=torch.bfloat16, device="cuda")
        inner = buf[65536:65536 + n].view(shape)
        inner.copy_(torch.randn(shape, generator=gen, device="cuda"))
        return inner

    x, w = between_nan(B, d), [between_nan(F, d) for _ in range(3)]
    y, idx = moc.moc_ffn_decode(x, *w, K)
    y2, idx2 = moc.moc_ffn_decode(x.clone(), *[t.clone() for t in w], K)
    torch.cuda.synchronize()
    assert torch.isfinite(y).all()
    assert torch.equal(y, y2) and torch.equal(idx, idx2)
