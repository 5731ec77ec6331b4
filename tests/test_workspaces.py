"""What the workspaces hold and where (csrc/api_common.h), compiled for the host: arrays of different paths that share memory."""
import subprocess

import pytest

from paper_2511_09323_amd import build

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "api_common.h"
#include "decode_persist.h"
namespace mocapi {      // (as without an environment)
Options::Options() { std::memset(this, 0, sizeof(*this)); }
const Options& options() {
    static const Options o;
    return o;
}
}  // namespace mocapi
using namespace mocapi;
#define EXPECT(c) do { if (!(c)) { std::printf("line %d: %s (T %d d %d F %d)\n", __LINE__, #c, D.T, D.d, D.F); std::exit(1); } } while (0)

static bool apart(const void* a, size_t na, const void* b, size_t nb) {
    return static_cast<const char*>(a) + na <= b || static_cast<const char*>(b) + nb <= a;
}
// Decode with both projections as streams writes nothing that the persistent kernel reads a tag or the generation from: g2, zt and DecodeSync.
static void decode() {
    for (int T : {2, 3, 4, 5, 16})
        for (int F : {5, 1376, 5461, 11008, 32768})
            for (int d : {64, 2048, 4096}) {
                const Dims D(moc_shape{T, d, F, (F + 7) / 8, MOC_BF16});
                char* const base = static_cast<char*>(std::malloc(1));      // (an address; nothing is read or written)
                const DecodeWs W(base, D);
                const size_t row = (size_t)T * D.ldF * sizeof(float), slots = T <= 4 ? 4 : 16;
                struct { const void* p; size_t n; } streams[] = {{W.sd, row}, {W.ud, row}, {W.arrived, 64 * sizeof(uint32_t)}},
                    tagged[] = {{W.g2, 2 * row}, {W.zt, (size_t)F * (1 + slots) * 8}, {W.sync, sizeof(DecodeSync)}};
                for (const auto& s : streams) {
                    EXPECT((const char*)s.p >= base && (const char*)s.p + s.n <= base + W.bytes);
                    for (const auto& t : tagged) EXPECT(apart(s.p, s.n, t.p, t.n));
                    for (const void* used : {(const void*)W.g, (const void*)W.gkeys}) EXPECT(apart(s.p, s.n, used, row));
                    EXPECT(apart(s.p, s.n, W.gsel, (size_t)T * D.K * 4) && apart(s.p, s.n, W.idx, (size_t)T * D.K * 4));
                    EXPECT(apart(s.p, s.n, W.part, (size_t)decode_splits(T, D.K) * T * d * 4));
                }
                for (int i = 0; i < 3; ++i) EXPECT(apart(streams[i].p, streams[i].n, streams[(i + 1) % 3].p, streams[(i + 1) % 3].n));
                std::free(base);
            }
}
static size_t moc_workspace(const Dims& D, int dtype, int op) { return dtype == MOC_BF16 ? workspace_for<bf16_t>(D, op) : workspace_for<float>(D, op); }
static bool same(const GemmRoute& a, const GemmRoute& b) { return a.pp == b.pp && a.tile == b.tile && a.shares == b.shares; }
// Scratch for shares (bf16): the routes of down, dX and the weight gradients are those with as much as eight shares or 72 MB; a layer that would not use
// it has none, and its arrays lie as without; a workspace for many tokens serves fewer.
static void shares() {
    for (int d : {64, 256, 512, 768, 1024, 1536, 2048, 4096})
        for (int F : {d, 8 * d / 3, 4 * d}) {
            size_t fwd = 0, bwd = 0;
            for (int T = 16; T <= 9000; T += 1 + T / 24) {
                const Dims D(moc_shape{T, d, F, (F + 7) / 8, MOC_BF16});
                const FwdWs<bf16_t> W(nullptr, D, false), X(nullptr, D, false, false, false);
                const BwdWs<bf16_t> V(nullptr, D, false), Y(nullptr, D, false, false);
                EXPECT(W.bytes >= fwd && V.bytes >= bwd);
                fwd = W.bytes;
                bwd = V.bytes;
                const size_t most = std::min((size_t)8 * T * d * 4, (size_t)72 << 20), dense = (size_t)T * D.ldF * 2;
                const auto route = [&](bool dx, size_t scratch) {
                    const PpSizes s{T, d, F, dx ? F : 0, D.ldF, d, false, true, true, d, d, 0, 2};
                    return gemm_route(kTilesKm, T, d, F, dx ? F : 0, 2, pp_sizes_ok(s), scratch, 256);
                };
                EXPECT(same(route(false, W.share_bytes), route(false, std::max(most, 3 * dense))));
                EXPECT(same(route(true, V.share_bytes), route(true, Y.share_bytes + (most - std::min(most, 2 * dense)))));
                const PpSizes s{F, d, T, 0, D.ldF, d, true, true, true, d, d, 0, 2};
                const GemmRoute whole = batch3_route(F, d, T, pp_sizes_ok(s), 256);
                const Batch3Split a = batch3_split(F, d, T, whole, V.dw_share_bytes, 256), 
                                   b = batch3_split(F, d, T, whole, Y.dw_share_bytes + (most - std::min(most, 2 * dense)), 256);
                EXPECT(a.rows == b.rows && a.shares == b.shares);
                EXPECT(X.bytes <= W.bytes && Y.bytes <= V.bytes && X.share_bytes == 0);
            }
        }
    // whole products with whatever scratch
    for (const moc_shape& s : {moc_shape{4096, 768, 2048, 256, MOC_BF16}, moc_shape{4096, 512, 1376, 172, MOC_BF16}, moc_shape{8192, 2048, 5461, 683, MOC_BF16},
                               moc_shape{3000, 64, 256, 32, MOC_BF16}, moc_shape{700, 512, 1376, 172, MOC_F32}}) {
        const Dims D(s);
        const size_t e = s.dtype == MOC_BF16 ? 2 : 4, row = (size_t)D.T * D.ldF;
        const auto up = [](size_t n) { return (n + 255) / 256 * 256; };
        EXPECT(moc_workspace(D, s.dtype, MOC_OP_FWD) == up(row * 4) + 2 * up(row * e));
        EXPECT(moc_workspace(D, s.dtype, MOC_OP_BWD) == up((size_t)D.T * D.nw * 4) + up((size_t)D.T * D.nw * 2) + up(row * e) + 3 * up(((size_t)D.T + 248) * D.ldF * e));
    }
}
int main(int argc, char**) {
    if (argc == 1) decode();
    else shares();
    std::puts("ok");
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("workspaces")
    (d / "p.hip").write_text(PROGRAM)
    subprocess.run([build.HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-I" + build.CSRC, str(d / "p.hip"), "-o", str(d / "p")], check=True,
                   capture_output=True, text=True)
    return lambda *a: subprocess.run([str(d / "p")] + [str(x) for x in a], capture_output=True, text=True)


def test_streamed_decode_writes_no_word_of_the_persistent_kernel(program):
    r = program()
    assert r.returncode == 0, r.stdout + r.stderr


def test_scratch_for_shares_is_there_where_it_is_used(program):
    r = program("shares")
    assert r.returncode == 0, r.stdout + r.stderr
