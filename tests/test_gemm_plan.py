"""The size arithmetic of the matrix-core products (csrc/gemm_plan.h), compiled for the CPU with overflow checks: offsets at sizes at which
a GPU test would need hundreds of gigabytes, and which kernel each case of the fp32 GPU tests takes, so that those tests reach what they
say (bf16: test_gemm_routes.py)."""
import os
import subprocess

import pytest

from tests.test_gpu_f32_gemm import CASES as F32_CASES, SHARE_CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include "gemm_plan.h"
using namespace moc;
#define EXPECT(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)
static const int kCus = 256;      // of an MI355X

static void offsets() {
    // k rows of a slice, clamped to the last one of the contraction: up to 32-bit sizes of everything but a slice
    for (int bk : {32, 64, 128})
        for (int ld : {8, 2736, 11008, 32768, (1 << 24) - 8})
            for (int left : {1, 2, bk - 1, bk, bk + 1, 196608, 1 << 30}) {
                if ((int64_t)bk * ld >= (1ll << 31)) continue;      // refused by the launchers
                for (int r = 0; r < bk; ++r)
                    EXPECT(std::min(r * ld, last_row_offset(left, bk, ld)) == (int64_t)std::min(r, left - 1) * ld);
            }
    std::puts("ok");
}

static void f32(int T, int d, int F) {
    static const char* const names[4] = {"64x64", "32x32", "32x32s", "16x32s"};
    auto tile = [&](int M, int N, int batch, int64_t k, bool ascending) { return names[(int)f32_tile(M, N, batch, k, ascending, kCus)]; };
    std::printf("gate_up=%s down=%s dz=%s dw=%s dx=%s\n", tile(T, F, 2, d, true), tile(T, d, 1, F, false), tile(T, F, 1, d, false),
                tile(F, d, 3, T, false), tile(T, d, 1, 2 * (int64_t)F, false));
}
// what the products over the channels take, with the scratch that the layer has for their shares
static void f32_over_channels(int T, int d, int F) {
    static const char* const names[4] = {"64x64", "32x32", "32x32s", "16x32s"};
    const size_t scratch = (size_t)T * ((F + kColPad - 1) / kColPad * kColPad) * 2 * sizeof(float);
    for (int two : {0, 1}) {
        const F32Shares r = f32_shares(T, d, F, two * F, scratch, kCus);
        std::printf(r.shares > 1 ? "%s=%s/%d " : "%s=%s ", two ? "dx" : "down", names[(int)r.tile], r.shares);
    }
    std::puts("");
}
int main(int argc, char** argv) {
    if (argc == 5) f32_over_channels(std::atoi(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]));
    if (argc == 1) offsets();
    else if (argc == 4) f32(std::atoi(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]));
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I" + os.path.join(ROOT, "paper_2511_09323_amd", "csrc"), str(d / "plan.cpp"), "-o", str(d / "plan")], check=True)
    return lambda *a: subprocess.run([str(d / "plan")] + [str(x) for x in a], capture_output=True, text=True)


def test_row_offsets_of_long_contractions(plan):
    r = plan()
    assert r.returncode == 0, r.stdout + r.stderr


def test_cases_take_the_kernels_they_name(plan):
    for T, d, F, _, want in F32_CASES:
        got = plan(T, d, F).stdout.split()
        assert set(want.split()) <= set(got), (T, d, F, want, got)


def test_share_cases_take_the_shares_they_name(plan):
    for T, d, F, _, want in SHARE_CASES:
        r = plan(T, d, F, "shares")
        assert r.stdout.split() == want.split(), (T, d, F, want, r.stdout, r.stderr)


def test_cases_reach_every_tile():
    named = " ".join(c[4] for c in F32_CASES).split()
    for product, wanted in (("gate_up", ("64x64", "32x32")), ("down", ("64x64", "32x32", "32x32s", "16x32s")),
                            ("dz", ("64x64", "32x32", "16x32s")), ("dw", ("64x64", "32x32", "16x32s")), ("dx", ("64x64", "32x32", "32x32s", "16x32s"))):
        assert {"%s=%s" % (product, s) for s in wanted} <= set(named), product
