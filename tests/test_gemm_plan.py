"""The size arithmetic of the matrix-core products (csrc/gemm_plan.h), compiled for the CPU with overflow checks: sizes at which a
GPU test would need hundreds of gigabytes."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include "gemm_plan.h"
using namespace moc;
#define EXPECT(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)
int main() {
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
