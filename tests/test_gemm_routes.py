"""Which kernel every bf16 product takes, by the functions of csrc/gemm_plan.h that the launchers call, compiled for the CPU: the cases of
test_gpu_large_tiles.py and test_gpu_gemm_tiles.py reach the tiles they name, and the routes keep to what the launchers can run."""
import os
import re
import subprocess

import pytest

from tests.test_gpu_decode_dense import CASES as DENSE_CASES, GROUPED_CASES as DENSE_GROUPED_CASES
from tests.test_gpu_experts import MIXTRAL_180M
from tests.test_gpu_gemm_tiles import CASES as TILE_CASES
from tests.test_gpu_large_tiles import CASES, EXPERT_CASES, LONG_CASES, SPLIT_CASES, STORED_SPLIT_CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>
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
static int ldf(int F) { return (F + kColPad - 1) / kColPad * kColPad; }
static int fs(int F) { return (F + 7) / 8 * 8; }
// the operands of x W^T products to [T, F], of products over the channels to [T, d], and of weight gradients
static PpSizes to_channels(int T, int d, int F, int elem) { return PpSizes{T, F, d, 0, d, d, false, false, false, fs(F), ldf(F), 0, elem}; }
static PpSizes to_model(int T, int d, int F, int F2) { return PpSizes{T, d, F, F2, ldf(F), d, false, true, true, d, d, 0, 2}; }
static PpSizes to_weights(int T, int d, int F) { return PpSizes{F, d, T, 0, ldf(F), d, true, true, true, d, d, 0, 2}; }
// the products of one forward + backward, d a multiple of 32
static void products(int T, int d, int F) {
    const bool kc = pp_sizes_ok(to_channels(T, d, F, 4)) && pp_sizes_ok(to_channels(T, d, F, 2));
    const PairRoute pair = pair_route(T, F, d, kc, kCus);
    if (pair.together) say("gate_up", pair.route);
    else say("gate", gemm_route(kTilesAll, T, F, d, 0, 2, kc, 0, kCus));
    say("dz", gemm_route(kTilesAll, T, F, d, 0, 2, kc, 0, kCus));
    say("dw", batch3_route(F, d, T, pp_sizes_ok(to_weights(T, d, F)), kCus));
    say("down", gemm_route(kTilesKm, T, d, F, 0, 2, pp_sizes_ok(to_model(T, d, F, 0)), (size_t)T * ldf(F) * 6, kCus));
    say("dx", gemm_route(kTilesKm, T, d, F, F, 2, pp_sizes_ok(to_model(T, d, F, F)), (size_t)T * ldf(F) * 4, kCus));
    std::puts("");
}
// the products over the channels with all of a workspace's scratch
static void over_channels(int T, int d, int F) {
    for (int two : {0, 1}) {
        EXPECT(two == 0 || long_product(T, d, F, F));
        const size_t scratch = std::max((size_t)T * ldf(F) * (two ? 4 : 6), share_scratch_wanted(T, d, F, two * F));
        say(two ? "dx" : "down", gemm_route(kTilesKm, T, d, F, two * F, 2, pp_sizes_ok(to_model(T, d, F, two * F)), scratch, kCus));
    }
    std::puts("");
}
// the weight gradients with what a workspace has for them
static void weights(int T, int d, int F) {
    const size_t dense = (size_t)T * ldf(F) * 2, want = share_scratch_wanted(T, d, F, F), scratch = dense + (want > 2 * dense ? want - 2 * dense : 0);
    const Batch3Split s = batch3_split(F, d, T, batch3_route(F, d, T, pp_sizes_ok(to_weights(T, d, F)), kCus), scratch, kCus);
    EXPECT(s.rows == 0 || (s.rows < F && s.rows % kPpTile[s.main].bm == 0 && (size_t)3 * s.shares * (F - s.rows) * d * 4 <= scratch));
    EXPECT(s.rows == 0 || s.rest == 0 || s.rest == 3);
    if (s.rows) std::printf("%d pp%dx%d pp%dx%d/%d\n", s.rows, kPpTile[s.main].bm, kPpTile[s.main].bn, kPpTile[s.rest].bm, kPpTile[s.rest].bn, s.shares);
    else std::puts("whole");
}
// of experts with `counts` rows
static void experts(int d, int F, int n, const int* counts) {
    const std::vector<int> rows(counts, counts + n), ks(n, d), kf(n, F), no(n, 0);
    bool channels = true, model = true, two = true, weights = true;
    std::vector<int> wm, wk, wno;
    for (int c : rows) {
        if (c == 0) continue;
        channels = channels && pp_sizes_ok(to_channels(c, d, F, 4)) && pp_sizes_ok(to_channels(c, d, F, 2));
        model = model && pp_sizes_ok(to_model(c, d, F, 0));
        two = two && pp_sizes_ok(to_model(c, d, F, F));
        weights = weights && pp_sizes_ok(to_weights(c, d, F));
        for (int k = 0; k < 3; ++k) { wm.push_back(F); wk.push_back(c); wno.push_back(0); }
    }
    double cost;
    const int t = channels ? grouped_pair_tile(n, rows.data(), F, d, kCus) : -1;
    if (t >= 0) say("gate_up", GemmRoute{true, t, 1});
    else say("gate", grouped_route(kTilesGroup, n, rows.data(), F, ks.data(), no.data(), channels, kCus, -1, &cost));
    const auto rounds = [&](const GemmRoute& r, int m, const int* M, int N) {      // rounds of the busiest XCD's workgroups
        if (!r.pp) return;
        int64_t tiles = 0;
        for (int z = 0; z < m; ++z) tiles += tile_count(M[z], N, kPpTile[r.tile]);
        std::printf("x%d ", (int)((tiles + kCus - 1) / kCus));
    };
    const GemmRoute dz = grouped_route(kTilesGroup, n, rows.data(), F, ks.data(), no.data(), channels, kCus, -1, &cost);
    say("dz", dz);
    const GemmRoute dw = grouped_route(kTilesKmGroup, (int)wm.size(), wm.data(), d, wk.data(), wno.data(), weights, kCus, -1, &cost);
    say("dw", dw);
    rounds(dw, (int)wm.size(), wm.data(), d);
    const GemmRoute down = grouped_route(kTilesKmGroup, n, rows.data(), d, kf.data(), no.data(), model, kCus, -1, &cost);
    say("down", down);
    rounds(down, n, rows.data(), d);
    say("dx", grouped_route(kTilesKmGroup, n, rows.data(), d, kf.data(), kf.data(), two, kCus, -1, &cost));
    std::puts("");
}
static void routes() {
    for (int M : {1, 17, 256, 257, 2047, 8192, 100000})
        for (int N : {8, 512, 2048, 5461, 11008})
            for (int K : {1, 64, 65, 1376, 5461, 32768})
                for (size_t scratch : {(size_t)0, (size_t)1 << 20, (size_t)1 << 28}) {
                    const GemmRoute r = gemm_route(kTilesAll, M, N, K, 0, 2, true, scratch, kCus), plain = gemm_route(kTilesAll, M, N, K, 0, 2, false, 0, kCus);
                    EXPECT(r.tile >= 0 && r.tile < (r.pp ? kPpTiles : kGemmTiles));
                    // where both may run, the large tiles leave no product to the same shapes of gemm_mfma.h: with a k-major B two of them are not built
                    EXPECT(r.pp || r.tile > 3);
                    const GemmRoute km = gemm_route(kTilesKm, M, N, K, 0, 2, true, scratch, kCus);
                    EXPECT(km.pp == r.pp && km.tile == r.tile && km.shares == r.shares);
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
// Byte offsets that gemm_bf16_pp_kernel forms in 32 bits: within an operand of `rows` rows (k-contiguous) or columns (k-major), to the
// end of the last tile and of the last slice; its readable bytes; within a tile's rows of the result.
static int64_t last_offset(bool km, int64_t rows, int64_t ld, int64_t k) {
    const int64_t row = (rows + 255) / 256 * 256 - 1, last_k = (k + kPpBK - 1) / kPpBK * kPpBK - 1;
    return 2 * (km ? last_k * ld + row : row * ld + last_k);
}
static int64_t readable(bool km, int64_t rows, int64_t ld, int64_t k) { return 2 * ld * (km ? k : rows); }
static void check_offsets(const PpSizes& s) {
    const int64_t lim = 1ll << 32;
    for (int k : {s.Kc, s.Kc2}) {
        if (k == 0) continue;
        EXPECT(last_offset(s.akm, s.M, s.lda, k) + 16 <= lim && readable(s.akm, s.M, s.lda, k) < lim);
        EXPECT(last_offset(s.bkm, s.N, s.ldb, k) + 16 <= lim && readable(s.bkm, s.N, s.ldb, k) < lim);
    }
    EXPECT(256 * s.ldc * s.elem <= 1ll << 31);      // (0xFFFFFF00, where columns past the last go, is out of range)
}
// The largest value of one size that is taken, as the kernel's limit is approached; nothing that passes 4 GiB is.
template <class Set> static int64_t largest(const PpSizes& base, int64_t hi, int64_t step, const Set& set) {
    int64_t best = 0;
    for (int64_t lo = 1, up = hi / step; lo <= up;) {
        const int64_t mid = (lo + up) / 2;
        PpSizes s = base;
        set(s, mid * step);
        if (pp_sizes_ok(s)) { best = mid * step; lo = mid + 1; check_offsets(s); }
        else up = mid - 1;
    }
    return best;
}
static void sizes() {
    const int64_t lim = 1ll << 32;
    for (int64_t ld : {64, 512, 4096, 5504, 11008, 32768, 1 << 20}) {
        // x W^T: rows of x
        const PpSizes kc{256, 256, 64, 0, ld, 64, false, false, false, 256, 256, 0, 4};
        const int64_t m = largest(kc, 1ll << 30, 1, [](PpSizes& s, int64_t v) { s.M = (int)v; });
        EXPECT(m > 0 && m * ld * 2 < lim && (m + 300) * ld * 2 >= lim - 131072);
        // down and dX: the contraction over B's rows, ragged, A's rows padded
        const PpSizes km{256, (int)std::min<int64_t>(ld, 256), 64, 0, 0, ld, false, true, true, 256, 256, 0, 2};
        for (int add : {0, 1, 33}) {
            const int64_t k = largest(km, (1ll << 30) / 64, 64, [&](PpSizes& s, int64_t v) {
                s.Kc = (int)v + add;
                s.lda = (v + add + 63) / 64 * 64;
            });
            EXPECT(k > 0 && k * ld * 2 < lim);
        }
        // weight gradients: the contraction over the tokens
        const PpSizes kk{(int)std::min<int64_t>(ld, 300), 64, 64, 0, ld, 64, true, true, true, 256, 256, 0, 2};
        const int64_t t = largest(kk, 1ll << 30, 1, [](PpSizes& s, int64_t v) { s.Kc = (int)v; });
        EXPECT(t > 0 && t * ld * 2 < lim && (t + 300) * (ld + 1) * 2 >= lim - 131072);
        // pitch of the result
        for (int elem : {2, 4}) {
            const int64_t c = largest(kc, 1ll << 30, 16 / elem, [&](PpSizes& s, int64_t v) { s.ldc = v; s.elem = elem; });
            EXPECT(256 * c * elem < 1ll << 31 && 256 * (c + 16) * elem >= 1ll << 31);
        }
    }
    const PpSizes good{256, 256, 64, 0, 64, 256, false, true, true, 256, 256, 0, 2};
    EXPECT(pp_sizes_ok(good));
    const auto refused = [&](auto change) {
        PpSizes s = good;
        change(s);
        return !pp_sizes_ok(s);
    };
    EXPECT(refused([](PpSizes& s) { s.Kc = 63; s.a_zero_padded = false; }));      // a ragged contraction that nothing covers
    EXPECT(refused([](PpSizes& s) { s.Kc = 65; }));                              // rows of A end before the slice
    EXPECT(refused([](PpSizes& s) { s.Kc = 63; s.bkm = false; }));
    EXPECT(refused([](PpSizes& s) { s.akm = true; s.bkm = false; }));
    // weight gradients over two operand pairs: the kernel knows the readable bytes of A's first only
    EXPECT(!refused([](PpSizes& s) { s.akm = true; }));
    EXPECT(refused([](PpSizes& s) { s.akm = true; s.Kc2 = 32; }));
    EXPECT(!refused([](PpSizes& s) { s.Kc2 = 32; }));
    EXPECT(refused([](PpSizes& s) { s.out_n = 252; }));                          // half a 16-byte piece
    EXPECT(refused([](PpSizes& s) { s.ldc = 260; }));
    EXPECT(refused([](PpSizes& s) { s.stride = 4; }));
    std::puts("ok");
}
// Weight gradients of experts on whole XCDs: who owns what, and when.
static void owners() {
    int own[24];
    const auto take = [&](std::vector<int> rows, int F, int d, int bm, int bn) {
        std::sort(rows.rbegin(), rows.rend());
        std::vector<int> slices, tiles;
        for (int r : rows)
            for (int k = 0; k < 3; ++k) {
                slices.push_back(pp_slice_count(r, 0));
                tiles.push_back((F + bm - 1) / bm * ((d + bn - 1) / bn));
            }
        std::fill(own, own + 24, -1);
        const bool whole = pp_owners((int)slices.size(), slices.data(), tiles.data(), 32, own);
        for (size_t z = 0; z < slices.size(); ++z) EXPECT(whole ? own[z] >= 0 && own[z] < 8 : own[z] == -1);
        return whole;
    };
    EXPECT(take({6000, 2500, 3000, 4100, 5200, 3300, 3900, 4768}, 2048, 768, 256, 192));      // 32 tiles a problem: whole
    EXPECT(take({700, 1, 513, 300, 64, 257, 900}, 2736, 128, 256, 128));                      // (a case of test_gpu_large_tiles.py)
    EXPECT(!take({4000, 4000}, 2048, 768, 256, 192));                                         // fewer problems than XCDs
    EXPECT(!take({25000, 1000, 1000, 1000, 1000, 1000, 1000, 768}, 4096, 768, 256, 192));     // one expert has most rows: two of its 64 tiles to a workgroup
    EXPECT(!take({4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096}, 11008, 1024, 128, 256));   // many rounds: nothing shared beyond them
    std::puts("ok");
}
static void gate() {
    struct Row { int B, d, F; bool grouped, pays; };
    for (const Row& r : {Row{1, 4096, 11008, false, false}, Row{2, 4096, 11008, false, true}, Row{4, 4096, 11008, true, true},
                         // few rows a workgroup: the dot products, at any width
                         Row{2, 2560, 640, false, false}, Row{4, 3072, 768, false, false}, Row{3, 4096, 1024, false, false}, Row{2, 1024, 1024, false, false},
                         Row{2, 512, 512, false, false}, Row{4, 512, 1376, false, true}, Row{4, 1024, 2736, false, true},
                         // the bytes of W_gate decide, not the width
                         Row{3, 2048, 5461, false, false}, Row{3, 2048, 16384, false, true}, Row{3, 1536, 8192, false, true}, Row{3, 3072, 1900, false, false}, Row{3, 3072, 2000, false, true},
                         Row{3, 2048, 2048, true, true}, Row{3, 1536, 4096, true, true}, Row{4, 2048, 5464, true, false}, Row{4, 2560, 6824, true, true},
                         Row{5, 2048, 5461, false, true}, Row{16, 64, 8, true, true}, Row{5, 2560, 640, false, true}}) {
        if (gate_stream_pays(r.B, r.d, r.F, r.grouped, kCus) != r.pays) std::printf("%d tokens, %d x %d\n", r.B, r.d, r.F);
        EXPECT(gate_stream_pays(r.B, r.d, r.F, r.grouped, kCus) == r.pays);
    }
    EXPECT(!gate_stream_nontemporal(2048, 5464) && gate_stream_nontemporal(2048, 5860) && gate_stream_nontemporal(1024, 16384));
    EXPECT(!gate_stream_nontemporal(4096, 1024) && gate_stream_nontemporal(4096, 1536) && gate_stream_nontemporal(4096, 11008) && gate_stream_nontemporal(4096, 32768));
    std::puts("ok");
}
// Decode with both projections as streams: the width of the down projection's slices and its ranges of channels, or "gather".
static void dense(int B, int d, int F, int K, bool grouped) {
    if (d % 64 != 0 || d > 4096 || !gate_stream_pays(B, d, F, grouped, kCus) || !decode_dense_pays(B, d, F, K, grouped)) std::puts("gather");
    else std::printf("%d/%d\n", d <= kDownNarrowMaxD ? 64 : 128, down_stream_ranges(B, d, F, K, kCus));
}
int main(int argc, char** argv) {
    if (argc == 1) routes();
    else if (!std::strcmp(argv[1], "dense")) dense(std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4]), std::atoi(argv[5]), std::atoi(argv[6]) != 0);
    else if (argc == 2) (!std::strcmp(argv[1], "gate") ? gate : !std::strcmp(argv[1], "owners") ? owners : sizes)();
    else if (!std::strcmp(argv[1], "experts")) {
        std::vector<int> counts;
        for (int i = 4; i < argc; ++i) counts.push_back(std::atoi(argv[i]));
        experts(std::atoi(argv[2]), std::atoi(argv[3]), (int)counts.size(), counts.data());
    } else if (!std::strcmp(argv[1], "long")) over_channels(std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4]));
    else if (!std::strcmp(argv[1], "weights")) weights(std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4]));
    else products(std::atoi(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]));
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


def test_sizes_that_large_tiles_take(plan):
    """Every 32-bit offset of gemm_bf16_pp_kernel, up to the largest operands that pp_sizes_ok admits (near 4 GiB)."""
    r = plan("sizes")
    assert r.returncode == 0, r.stdout + r.stderr


def test_weight_gradients_of_experts_on_whole_xcds(plan):
    r = plan("owners")
    assert r.returncode == 0, r.stdout + r.stderr


def test_decodes_that_take_the_streamed_gate(plan):
    """By rows per workgroup and bytes of W_gate (gate_stream_pays, gate_stream_nontemporal)."""
    r = plan("gate")
    assert r.returncode == 0, r.stdout + r.stderr


# ranges of channels of test_gpu_decode_dense.py's cases, in their order
DENSE_RANGES = ["64/8", "64/1", "64/1", "64/2", "64/16", "64/16", "64/8", "64/8", "64/8", "128/8", "128/8", "128/8", "64/32", "64/16", "64/16", "128/8", "64/8"]
DENSE_GROUPED_RANGES = ["128/8", "64/8", "64/8", "64/8"]


def test_decode_cases_take_the_streams(plan):
    got = [plan("dense", *c, 0).stdout.strip() for c in DENSE_CASES]
    assert got == DENSE_RANGES
    got = [plan("dense", B, d, F, F // b * a, 1).stdout.strip() for B, d, F, a, b in DENSE_GROUPED_CASES]
    assert got == DENSE_GROUPED_RANGES


@pytest.mark.parametrize("B,d,F,requested,grouped,want", [
    (16, 4096, 11008, 1.19, 0, "gather"), (16, 4096, 11008, 1.2, 0, "128/8"), (5, 1536, 4096, 1.19, 0, "gather"), (16, 1536, 4096, 1.2, 0, "64/8"),
    # d between 2048 and 4096: with the tokens and the idle compute units
    (16, 2560, 6816, 1.86, 0, "gather"), (16, 2560, 6816, 1.88, 0, "128/8"), (5, 2560, 6816, 1.4, 0, "gather"), (5, 2560, 6816, 1.41, 0, "128/8"),
    (16, 3072, 8192, 1.64, 0, "gather"), (16, 3072, 8192, 1.65, 0, "128/8"), (5, 3072, 8192, 1.34, 0, "128/8"), (16, 3584, 9552, 1.43, 0, "128/8"),
    (16, 1024, 6144, 1.99, 0, "gather"), (16, 1024, 6144, 2.0, 0, "64/16"),                                         # long columns
    (4, 4096, 11008, 2.99, 0, "gather"), (4, 4096, 11008, 3.0, 0, "128/8"), (4, 2048, 5461, 4, 0, "gather"),        # few tokens
    (16, 4096, 11008, 2.99, 1, "gather"), (12, 4096, 11008, 3, 1, "128/8"), (4, 4096, 11008, 4, 1, "gather"),       # grouped
    (16, 512, 1376, 5.99, 0, "gather"), (16, 512, 1376, 6, 0, "64/8"), (16, 2560, 1376, 8, 0, "gather"),            # small layers
])
def test_lines_of_the_streamed_decode(plan, B, d, F, requested, grouped, want):
    K = -(-int(requested * F * 1000) // (1000 * B)) if want != "gather" else int(requested * F / B)
    assert plan("dense", B, d, F, K, grouped).stdout.strip() == want


def test_cases_take_the_kernels_they_name(plan):
    for T, d, F, _, want in CASES + TILE_CASES:
        got = plan(T, d, F).stdout.split()
        assert set(want.split()) <= set(got), (T, d, F, want, got)


def test_long_cases_take_the_kernels_they_name(plan):
    for T, d, F, _, want in LONG_CASES:
        got = plan("long", T, d, F).stdout.split()
        assert set(want.split()) <= set(got), (T, d, F, want, got)


def test_weight_gradients_are_split_as_named(plan):
    for T, d, F, _, want in SPLIT_CASES + STORED_SPLIT_CASES:
        r = plan("weights", T, d, F)
        assert r.stdout.strip() == want, (T, d, F, want, r.stdout)
    # few tokens, also where a split would save a little; one round; a few tiles
    for T, d, F in ((1984, 2048, 5461), (2400, 1536, 4096), (4096, 768, 2048), (8192, 2048, 200)):
        assert plan("weights", T, d, F).stdout.strip() == "whole", (T, d, F)


def test_expert_cases_take_the_kernels_they_name(plan):
    # (the Mixtral shape: weight gradients of 24 problems in two rounds)
    for counts, d, F, _, want in EXPERT_CASES + [(MIXTRAL_180M, 512, 1376, 256, "gate_up=pp256x256 dz=pp256x128 dw=pp192x256 x2")]:
        got = plan("experts", d, F, *counts).stdout
        at = 0
        for word in want.split():                        # (in order: xN belongs to the product before it)
            at = got.find(word + " ", at)
            assert at >= 0, (counts, d, F, want, got)


def test_cases_reach_every_large_tile():
    named = " ".join(c[4] for c in CASES).split()
    shapes = ("pp256x256", "pp192x256", "pp256x192", "pp128x256", "pp256x128")
    for product in ("gate_up", "dw"):
        assert {"%s=%s" % (product, s) for s in shapes} <= set(named), product
    for product in ("dz", "down", "dx"):
        assert any(n.startswith(product + "=pp") and "/" not in n for n in named), product
    assert any(n.startswith("dx=pp") and "/" in n for n in named)
    experts = " ".join(c[4] for c in EXPERT_CASES)
    for product in ("gate_up", "dz", "dw", "down", "dx"):
        assert product + "=pp" in experts, product
    assert re.search(r"down=pp\S+ x2", experts)


def test_cases_reach_every_basic_tile():
    """Every tile of gemm_mfma.h by a product that takes it without MOC_GEMM_TILE."""
    named = set(" ".join(c[4] for c in TILE_CASES).split())
    small = ("128x192", "192x128", "128x128", "64x128")
    for product, wanted in (("gate_up", ("256x256", "256x192", "192x256", "256x128") + small), ("gate", ("256x256", "256x192", "192x256")),
                            ("dz", ("256x128", "128x192", "192x128", "64x128")), ("dw", small),
                            ("down", ("192x128/4", "128x128/6", "64x128/4")), ("dx", ("192x128/4", "128x128/7", "64x128/8"))):
        assert {"%s=%s" % (product, s) for s in wanted} <= named, product
