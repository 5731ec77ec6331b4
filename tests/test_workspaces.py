"""What the workspaces hold and where (csrc/api_common.h), compiled for the host: arrays of different paths that share memory."""
import subprocess

import pytest

from paper_2511_09323_amd import build

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "api_common.h"
#include "decode_persist.h"
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
int main() {
    decode();
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
