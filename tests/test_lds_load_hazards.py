"""The hand-written load into LDS of the GEMM tiles, in the assembly the compiler makes of it for gfx950: it has to be
right whatever instruction stands in front of it, because the compiler does not look for hazards inside."""
import os
import re
import subprocess

import pytest

from paper_2410_18311_amd import build

PROBE = r"""
#include "gemm_tile.hpp"
namespace ci {
// a descriptor whose words come from lane reads right in front of the load
__global__ void probe_descriptor(const char* const* p, float* out) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[1024];
  const uint64_t a = reinterpret_cast<uint64_t>(p[threadIdx.x]);
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)a);
  const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32));
  load_to_lds(smem, threadIdx.x * 16u, rsrc_at(reinterpret_cast<const char*>(hi << 32 | lo)));
  __builtin_amdgcn_s_waitcnt(0);
  out[threadIdx.x] = reinterpret_cast<float*>(smem)[threadIdx.x];
}
// a value that lives in m0 across the load
__global__ void probe_m0(const char* p, int* out) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[1024];
  int v;
  asm volatile("s_mov_b32 %0, 7" : "={m0}"(v));
  load_to_lds(smem, threadIdx.x * 16u, rsrc_at(p));
  __builtin_amdgcn_s_waitcnt(0);
  out[threadIdx.x] = v;
}
}  // namespace ci
"""


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    src = tmp_path_factory.mktemp("asm") / "probe.hip"
    src.write_text(PROBE)
    out = str(src)[:-4] + ".asm"
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", str(src), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0 and os.path.exists(out), r.stderr
    bodies = {}
    for m in re.finditer(r"^_ZN2ci\d+(probe_\w+?)E\w*:[^\n]*\n(.*?)s_endpgm", open(out).read(), flags=re.S | re.M):
        lines = [l.split(";")[0].strip() for l in m.group(2).splitlines()]
        bodies[m.group(1)] = [l for l in lines if l and not l.startswith((".", "#")) and not l.endswith(":")]
    return bodies


def _wait_states(ins):
    return int(ins.split()[1], 0) + 1 if ins.startswith("s_nop") else 1


def test_descriptor_from_lane_reads_has_five_wait_states(assembly):
    code = assembly["probe_descriptor"]
    at = next(i for i, l in enumerate(code) if l.startswith("buffer_load") and l.endswith("lds"))
    first, last = map(int, re.search(r"s\[(\d+):(\d+)\]", code[at]).groups())
    words = {f"s{i}" for i in range(first, last + 1)}
    states = 0
    for l in reversed(code[:at]):
        if re.match(r"v_read(first)?lane_b32 ", l) and l.split()[1].rstrip(",") in words:
            break
        states += _wait_states(l)
    assert states >= 5, code[max(0, at - 10):at + 1]


def test_a_value_in_m0_survives_the_load(assembly):
    code = assembly["probe_m0"]
    at = next(i for i, l in enumerate(code) if l.startswith("buffer_load") and l.endswith("lds"))
    given = next(i for i, l in enumerate(code) if l.startswith("s_mov_b32 m0, 7"))
    assert given < at
    reads = [i for i, l in enumerate(code) if re.search(r"[ ,]m0\b", l) and not l.startswith("s_mov_b32 m0") and i > given]
    assert reads and all(i < at for i in reads), "read from m0 after the load has changed it"
