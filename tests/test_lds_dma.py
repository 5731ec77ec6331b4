"""The inline assembly of csrc/lds_dma.h in the code the compiler makes around it: the m0 of its own that it may keep there, and the
distance from a vector write of a load's descriptor, which it does not look after inside inline assembly."""
import re
import struct
import subprocess

import pytest

from paper_2511_09323_amd import build

LLVM = "/opt/rocm/llvm/bin/"
WAIT_STATES = 5      # between a vector instruction that writes a scalar register and a vector memory instruction that reads it

PROGRAM = r"""
#include "lds_dma.h"
using namespace moc;
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef const __attribute__((address_space(1))) void* global_ptr;
extern "C" __global__ void probe(const float* a, const void* b, float* out, uint32_t bytes, uint32_t where) {
    extern __shared__ float s[];
    __builtin_amdgcn_global_load_lds((global_ptr)(a + threadIdx.x), (lds_ptr)s, 4, 0, 0);      // the compiler's own: m0 = s
    lds_load16(threadIdx.x * 16u, buffer_desc(b, bytes), where);
    __builtin_amdgcn_global_load_lds((global_ptr)(a + 64 + threadIdx.x), (lds_ptr)s, 4, 0, 0);
    lds_load16<true>(threadIdx.x * 16u, buffer_desc(b, bytes), where);
    __builtin_amdgcn_global_load_lds((global_ptr)(a + 128 + threadIdx.x), (lds_ptr)s, 4, 0, 0);
    wait_counts<0, true>();
    out[threadIdx.x] = s[threadIdx.x];
}
"""


def test_loads_to_lds_leave_the_compiler_its_m0(tmp_path):
    (tmp_path / "probe.hip").write_text(PROGRAM)
    subprocess.run([build.HIPCC] + build.FLAGS + ["--cuda-device-only", "-S", "-I" + build.CSRC, str(tmp_path / "probe.hip"), "-o",
                                                  str(tmp_path / "probe.s")], check=True, capture_output=True)
    own, ours, m0 = 0, 0, None
    for line in (tmp_path / "probe.s").read_text().splitlines():
        line = line.split(";")[0].strip()
        if line.startswith("s_mov_b32 m0, "):
            m0 = line.split(", ")[1]
        elif line.startswith("global_load_lds"):
            own += 1
            assert m0 == "0", "a load of the compiler's own goes where m0 = %s points" % m0
        elif line.startswith("buffer_load_dwordx4") and line.endswith(" lds"):
            ours += 1
            assert re.match(r"s\d+$", m0), m0
    assert (own, ours) == (3, 2)


def scalars(operand):
    """Numbers of the scalar registers that an operand names."""
    m = re.match(r"s\[(\d+):(\d+)\]$|s(\d+)$", operand)
    if not m:
        return set()
    return {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))


def close_writes(lines):
    """The loads to LDS of a kernel and those whose descriptor a vector instruction writes fewer than WAIT_STATES before, on any way that
    leads to them; lines: instructions and, alone on a line, "<label>:"."""
    jumps = {}
    for i, line in enumerate(lines):
        m = re.match(r"s_c?branch\w* (\S+)", line)
        if m:
            jumps.setdefault(m.group(1), []).append(i)

    def reached(i, states, desc):
        """Whether going back from line i, `states` wait states before the load, meets such a write."""
        while i >= 0 and states < WAIT_STATES:
            line = lines[i]
            if line.startswith("<"):
                if any(reached(j - 1, states + 1, desc) for j in jumps.get(line[1:-2], ())):
                    return True
            else:
                if line.startswith(("s_branch", "s_endpgm", "s_setpc")):
                    return False              # (nothing falls through)
                m = re.match(r"v_\w+ (\S+?)(?:, |$)(?:(s\S+?)(?:, |$))?", line)
                if m and (scalars(m.group(1)) & desc or (line.startswith(("v_add_co", "v_sub_co", "v_addc", "v_subb", "v_mad_u64", "v_div_scale"))
                                                         and m.group(2) and scalars(m.group(2)) & desc)):
                    return True
                m = re.match(r"s_nop (\d+)", line)
                states += int(m.group(1)) + 1 if m else 1
            i -= 1
        return False

    loads = [i for i, line in enumerate(lines) if re.match(r"buffer_load_dwordx4 .* lds$", line)]
    return loads, [i for i in loads if reached(i - 1, 0, scalars(re.match(r"\S+ \S+, (s\[\d+:\d+\])", lines[i]).group(1)))]


LOAD = "buffer_load_dwordx4 v14, s[12:15], 0 offen lds"


@pytest.mark.parametrize("code,close", [
    (["v_readlane_b32 s13, v1, 2", "s_mov_b32 m0, s3", "s_nop 0", LOAD], True),
    (["v_readlane_b32 s13, v1, 2", "s_mov_b32 m0, s3", "s_nop 3", LOAD], False),
    (["v_readlane_b32 s11, v1, 2", "s_mov_b32 m0, s3", "s_nop 0", LOAD], False),
    (["v_add_co_u32 v1, s[14:15], v2, v3", "s_mov_b32 m0, s3", "s_nop 0", LOAD], True),
    (["s_nop 7", "<L1>:", "s_mov_b32 m0, s3", "s_nop 0", LOAD, "v_readfirstlane_b32 s12, v0", "s_cbranch_scc1 L1"], True),
    (["v_readfirstlane_b32 s12, v0", "s_branch L1", "s_nop 7", "<L1>:", "s_mov_b32 m0, s3", "s_nop 0", LOAD], True),
    (["v_readfirstlane_b32 s12, v0", "s_branch L2", "<L1>:", "s_mov_b32 m0, s3", "s_nop 0", LOAD], False),
])
def test_the_search_finds_close_writes(code, close):
    loads, bad = close_writes(code)
    assert len(loads) == 1 and bool(bad) == close


def device_code(library):
    """The gfx950 code objects in a library: bundles of (offset, size, name of the target)."""
    blob = open(library, "rb").read()
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        start = m.start()
        at = start + 24
        (n,) = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", blob, at)
            name = blob[at + 24:at + 24 + length]
            at += 24 + length
            if name.endswith(b"gfx950") and size:
                yield blob[start + offset:start + offset + size]


def test_no_load_to_lds_follows_a_vector_write_of_its_descriptor(tmp_path):
    """In every kernel of the built library that uses them."""
    kernels = 0
    for i, code in enumerate(device_code(build.LIB)):
        path = tmp_path / ("unit%d.o" % i)
        path.write_bytes(code)
        text = subprocess.run([LLVM + "llvm-objdump", "-d", "--symbolize-operands", str(path)], capture_output=True, text=True, check=True).stdout
        parts = re.split(r"^[0-9a-f]+ <(_Z\S+)>:$", text, flags=re.M)[1:]
        for name, body in zip(parts[0::2], parts[1::2]):
            if not re.search("gemm_bf16_pp_kernel|decode_gate_stream_kernel", name):
                continue
            lines = [re.sub(r"^[0-9a-f]+ (<L\d+>:)$", r"\1", line.split("//")[0].strip()) for line in body.splitlines() if line.strip()]
            loads, bad = close_writes(lines)
            kernels += 1
            assert loads and not bad, (name, len(bad), len(loads))
    assert kernels > 0
