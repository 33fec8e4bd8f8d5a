"""The direct-to-LDS copy (copy_1k), which is written as an instruction, in the code the compiler
makes around it.

The compiler does not look into the instruction: it cannot pad the hazard of a scalar base that a
vector instruction has just written (five wait states before a vector-memory read), and it knows
that m0 changes only if the copy says so.  A small kernel that provokes both is compiled for the
device and its assembly read.
"""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2510_05421_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCE = """
#include "device.h"
using namespace dvi;
// base from a vector register, right before the copy
__global__ void fresh_base(const uint64_t *p, uint32_t *out) {
    __shared__ __align__(1024) uint4 buf[64];
    const uint64_t v = p[threadIdx.x];
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    copy_1k(lds_addr(buf), 16 * threadIdx.x, (const void *)((uint64_t)hi << 32 | lo));
    __syncthreads();
    out[threadIdx.x] = buf[threadIdx.x].x;
}
// two compiler-made copies to one place, ours to another between them
__global__ void kept_m0(const uint32_t *p, const uint32_t *q, uint32_t *out) {
    __shared__ __align__(1024) uint4 buf[2][64];
    auto *dst = (__attribute__((address_space(3))) uint32_t *)&buf[0][0];
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(p + threadIdx.x), dst, 4, 0, 0);
    copy_1k(lds_addr(&buf[1][0]), 16 * threadIdx.x, q);
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(p + 64 + threadIdx.x), dst, 4, 0, 0);
    __syncthreads();
    out[threadIdx.x] = buf[0][threadIdx.x].x + buf[1][threadIdx.x].x;
}
"""


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    hipcc = HIPCC if os.path.exists(HIPCC) else shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("lds_copy")
    (d / "t.hip").write_text(SOURCE)
    subprocess.run([hipcc, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-S", "--offload-device-only", "-I", CSRC, str(d / "t.hip"), "-o", str(d / "t.s")],
                   check=True, capture_output=True, timeout=300)
    lines = [l.split(";")[0].strip() for l in (d / "t.s").read_text().splitlines()]
    return [l for l in lines if l and not l.startswith((".", "//"))]


def _body(lines, kernel):
    start = next(i for i, l in enumerate(lines) if re.match(r"_Z\w*%s\w*:" % kernel, l))
    end = next(i for i in range(start, len(lines)) if lines[i].startswith("s_endpgm"))
    return lines[start + 1:end]


def test_base_written_by_a_vector_instruction_has_five_wait_states(assembly):
    body = _body(assembly, "fresh_base")
    at = next(i for i, l in enumerate(body) if l.startswith("global_load_lds_dwordx4"))
    base = {int(r) for r in re.search(r"s\[(\d+):(\d+)\]", body[at]).groups()}
    waits = 0
    for l in reversed(body[:at]):
        w = re.match(r"v_readfirstlane_b32 s(\d+)", l)
        if w and int(w.group(1)) in base:
            break
        waits += int(l.split()[1]) + 1 if l.startswith("s_nop") else 1
    else:
        pytest.fail("no vector instruction writes the base: the kernel does not provoke the hazard")
    assert waits >= 5


def test_m0_is_set_again_after_the_copy(assembly):
    body = _body(assembly, "kept_m0")
    loads = [i for i, l in enumerate(body) if l.startswith("global_load_lds_dword")]
    assert len(loads) == 3 and body[loads[1]].startswith("global_load_lds_dwordx4")
    assert any(re.match(r"s_\w+ m0,", l) for l in body[loads[1] + 1:loads[2]])
