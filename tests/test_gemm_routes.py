"""Which kernel every bf16 product takes (csrc/gemm_plan.h: gemm_route, group_route), compiled for the CPU: the cases of
test_gpu_large_tiles.py reach the tiles they name, and the routes keep to what the launchers can run."""
import os
import subprocess

import pytest

from tests.test_gpu_large_tiles import CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "gemm_plan.h"
using namespace moc;
#define EXPECT(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)
static const int kCus = 256;      // of an MI355X

static void say(const char* what, const GemmRoute& r) {
    if (r.pp) std::printf("%s=pp%dx%d", what, kPpTile[r.tile].bm, kPpTile[r.tile].bn);
    else std::printf("%s=%dx%d", what, kGemmTile[r.tile].bm, kGemmTile[r.tile].bn);
    if (r.shares > 1) std::printf("/%d", r.shares);
    std::printf(" ");
}
static GemmRoute several(int n, int M, int N, int K, bool pp, double* cost) {
    return group_route(kTilesAll, [&](const GemmTile& t) { return n * tile_count(M, N, t); }, [&](const PpTile& t) { return n * tile_count(M, N, t); },
                       slice_count(K, 0), pp_slice_count(K, 0), pp, kCus, -1, cost);
}
// the products of one forward + backward, d a multiple of 32; x W^T products go to the large tiles for multiples of 64 only
static void products(int T, int d, int F) {
    double cost, single;
    const bool kc = d % 64 == 0;
    const GemmRoute both = several(2, T, F, d, kc, &cost);
    cheapest_tile(kTilesAll, [&](const GemmTile& t) { return tile_count(T, F, t); }, slice_count(d, 0), kCus, -1, &single);
    const GemmRoute one = gemm_route(kTilesAll, T, F, d, 0, 2, kc, 0, kCus);
    if (cost < 2.0 * single) say("gate_up", both);
    else say("gate", one);
    say("dz", one);
    say("dw", several(3, F, d, T, true, &cost));
    const size_t ldf = (F + 63) / 64 * 64;
    say("down", gemm_route(kTilesAll, T, d, F, 0, 2, true, T * ldf * 6, kCus));
    say("dx", gemm_route(kTilesAll, T, d, F, F, 2, true, T * ldf * 4, kCus));
    std::puts("");
}
static void routes() {
    for (int M : {1, 17, 256, 257, 2047, 8192, 100000})
        for (int N : {8, 512, 2048, 5461, 11008})
            for (int K : {1, 64, 65, 1376, 5461, 32768})
                for (size_t scratch : {(size_t)0, (size_t)1 << 20, (size_t)1 << 28}) {
                    const GemmRoute r = gemm_route(kTilesAll, M, N, K, 0, 2, true, scratch, kCus), plain = gemm_route(kTilesAll, M, N, K, 0, 2, false, 0, kCus);
                    EXPECT(r.tile >= 0 && r.tile < (r.pp ? kPpTiles : kGemmTiles));
                    EXPECT(!plain.pp && plain.shares == 1);
                    EXPECT(r.shares == 1 || (size_t)r.shares * M * N * 4 <= scratch);
                    // no share without a slice
                    EXPECT(r.shares <= (r.pp ? pp_slice_count(K, 0) / 4 : slice_count(K, 0) / 8) || r.shares == 1);
                    EXPECT(r.pp || r.shares == 1 || ((kTilesShares >> r.tile) & 1));
                    // a tile named by the environment is one of gemm_mfma.h's
                    EXPECT(gemm_route(kTilesAll, M, N, K, 0, 2, false, 0, kCus, 1).tile == 1);
                }
    std::puts("ok");
}
int main(int argc, char** argv) {
    if (argc == 1) routes();
    else if (argc == 4) products(std::atoi(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]));
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("routes")
    (d / "routes.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I" + os.path.join(ROOT, "paper_2511_09323_amd", "csrc"), str(d / "routes.cpp"), "-o", str(d / "routes")], check=True)
    return lambda *a: subprocess.run([str(d / "routes")] + [str(x) for x in a], capture_output=True, text=True)


def test_routes_stay_within_what_the_launchers_take(plan):
    r = plan()
    assert r.returncode == 0, r.stdout + r.stderr


def test_cases_take_the_kernels_they_name(plan):
    for T, d, F, _, want in CASES:
        got = plan(T, d, F).stdout.split()
        assert set(want.split()) <= set(got), (T, d, F, want, got)


def test_cases_reach_every_large_tile():
    named = " ".join(c[4] for c in CASES).split()
    shapes = ("pp256x256", "pp192x256", "pp256x192", "pp128x256", "pp256x128")
    for product in ("gate_up", "dw"):
        assert {"%s=%s" % (product, s) for s in shapes} <= set(named), product
    for product in ("dz", "down", "dx"):
        assert any(n.startswith(product + "=pp") and "/" not in n for n in named), product
    assert any(n.startswith("dx=pp") and "/" in n for n in named)
