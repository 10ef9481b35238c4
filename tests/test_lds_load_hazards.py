"""The hand-written load into LDS of the GEMM tiles: what the build looks for in the compiled library, in listings that
have and do not have it, in the library that is built, and in the assembly of a kernel that keeps a value in m0."""
import os
import re
import subprocess

import pytest

from paper_2410_18311_amd import build, isa_check

PROBE = r"""
#include "gemm_tile.hpp"
namespace ci {
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


def _listing(*lines):
    """An objdump listing of one function: instructions four bytes apart."""
    return "0000000000001000 <kernel>:\n" + "".join(
        f"\t{l:<58} // {0x1000 + 4 * i:012X}: 00000000\n" for i, l in enumerate(lines))


LOAD = ("s_mov_b32 m0, s9", "s_nop 0", "buffer_load_dwordx4 v1, s[4:7], 0 offen lds")


@pytest.mark.parametrize("lines,hazard", [
    (("v_readfirstlane_b32 s4, v2", *LOAD), True),
    (("v_readlane_b32 s7, v2, 3", "v_add_u32_e32 v1, v1, v2", *LOAD), True),
    (("v_readfirstlane_b32 s8, v2", *LOAD), False),                              # not the descriptor
    (("v_readfirstlane_b32 s5, v2", "s_nop 2", *LOAD), False),                   # five states: three, the move, the idle one
    (("v_readfirstlane_b32 s5, v2", "s_nop 1", *LOAD), True),                    # four
    (("v_readfirstlane_b32 s5, v2", "v_mov_b32_e32 v3, v4", "v_mov_b32_e32 v3, v4", "s_add_u32 s2, s2, 1", *LOAD), False),
    (("s_add_u32 s4, s4, 0x80", "s_addc_u32 s5, s5, 0", *LOAD), False),          # scalar results: the hardware waits
    (("v_cmp_gt_i32_e64 s[6:7], s0, v1", *LOAD), True),
    (("v_add_co_u32 v1, s[4:5], v1, v2", *LOAD), True),
    (("v_readfirstlane_b32 s4, v2", "s_nop 0", "buffer_load_dwordx4 v[8:11], v1, s[4:7], 0 offen"), False),  # the compiler's
    # into the load by a branch over the instructions that stand in front of it
    (("v_readfirstlane_b32 s4, v2", "s_branch 3", "s_nop 7", "s_nop 7", "s_nop 7", *LOAD), True),
    (("v_readfirstlane_b32 s4, v2", "s_branch 0", "s_endpgm", *LOAD), False),
])
def test_hazards_are_found_on_every_path(lines, hazard):
    assert bool(isa_check.hazards_in(_listing(*lines))) == hazard


PRODUCT = "v_mfma_f32_16x16x32_f16 a[4:7], v[0:3], v[8:11], a[4:7]"


@pytest.mark.parametrize("lines,hazard", [
    (("v_mov_b32_e32 v9, 0", PRODUCT), True),
    (("v_mov_b32_e32 v9, 0", "s_nop 0", PRODUCT), True),
    (("v_mov_b32_e32 v9, 0", "s_nop 1", PRODUCT), False),
    (("v_mov_b64_e32 v[12:13], v[4:5]", PRODUCT), False),                        # not its operands
    (("v_accvgpr_write_b32 a7, v20", PRODUCT), True),
    (("v_permlane32_swap_b32_e32 v20, v3", PRODUCT), True),                      # writes both
    (("ds_read_b128 v[0:3], v40", PRODUCT), False),                              # waited for by its counter
    ((PRODUCT, PRODUCT), False),
    ((PRODUCT, "v_accvgpr_read_b32 v20, a6"), True),
    ((PRODUCT, "s_nop 15", "s_nop 0", "v_accvgpr_read_b32 v20, a6"), True),      # 17
    ((PRODUCT, "s_nop 15", "s_nop 1", "v_accvgpr_read_b32 v20, a6"), False),
    ((PRODUCT, "global_store_dwordx4 v[30:31], a[4:7], off"), True),
    ((PRODUCT, "v_accvgpr_read_b32 v20, a8"), False),
    ((PRODUCT, "s_cbranch_scc1 1", "s_nop 15", "s_nop 1", "v_accvgpr_mov_b32 a12, a4"), True),   # past the first idle states
])
def test_product_hazards_are_found_on_every_path(lines, hazard):
    assert bool(isa_check.product_hazards_in(_listing(*lines))) == hazard


@pytest.mark.parametrize("lines,hazard", [(("s_mov_b32 m0, s9", LOAD[2]), True), (("s_add_i32 m0, s9, s2", "s_nop 0", LOAD[2]), False),
                                          (("s_mov_b32 m0, s9", PRODUCT, LOAD[2]), False)])
def test_a_load_does_not_go_by_m0_at_once(lines, hazard):
    assert bool(isa_check.hazards_in(_listing(*lines))) == hazard


@pytest.mark.parametrize("kernel,looked_at", [("gemm_wide_kernel", True), ("gemm_mid_kernel", True), ("some_kernel", True),
                                              ("gemm_slim_kernel", False)])
def test_the_build_looks_at_every_kernel_that_writes_out_its_products(monkeypatch, kernel, looked_at):
    text = _listing(PRODUCT, "v_accvgpr_read_b32 v20, a6").replace("<kernel>", f"<_ZN2ci{len(kernel)}{kernel}Ev>")
    monkeypatch.setattr(isa_check, "code_objects", lambda path: [kernel.encode()])
    monkeypatch.setattr(isa_check, "listing", lambda code: text)
    assert bool(isa_check.hazards("library")) == looked_at


def test_products_that_are_left_to_the_compiler_are_builtins():
    """The kernels that the build leaves out use no written-out product, and the others are there under the names that it goes by."""
    csrc = {f: open(os.path.join(build.CSRC, f)).read() for f in os.listdir(build.CSRC) if f.endswith((".hip", ".hpp"))}
    assert sorted(f for f, s in csrc.items() if "mfma16_in_place<" in s) == ["gemm_mid.hip", "gemm_wide.hip"]
    names = set(re.findall(r"\b(gemm_\w+_kernel)\(", "".join(s for s in csrc.values() if "mfma" in s)))
    assert {"gemm_mid_kernel", "gemm_wide_kernel"} <= names
    out = {n for n in names if any(f in n for f in isa_check.BY_COMPILER)}
    assert not out & {"gemm_mid_kernel", "gemm_wide_kernel"} and all(any(f in n for n in out) for f in isa_check.BY_COMPILER)


def test_both_families_of_written_out_products_are_in_the_built_library(lib):
    kernels, products = {}, {}
    for code in isa_check.code_objects(build.LIB_PATH):
        if b"gemm_" not in code:
            continue
        for name, ins, _ in isa_check._functions(isa_check.listing(code)):
            m = re.search(r"gemm_(wide|mid)_kernel", name)
            if m and not any(family in name for family in isa_check.BY_COMPILER):
                kernels[m[1]] = kernels.get(m[1], 0) + 1
                products[m[1]] = products.get(m[1], 0) + sum(op.startswith("v_mfma") for op, _, _ in ins)
    # both types of B's four widths, k-major ones too; seven shapes and three of them k-major, some built twice
    assert kernels["wide"] >= 16 and kernels["mid"] >= 20 and min(products.values()) > 1000


def test_the_built_library_has_no_hazard(lib):
    listings = [isa_check.listing(c) for c in isa_check.code_objects(build.LIB_PATH) if b"gemm_" in c]
    loads = sum(1 for text in listings for l in text.splitlines() if "buffer_load" in l and re.search(r"\blds\b", l))
    assert loads > 1000, "the kernels with loads into LDS are not among the code looked at"
    assert not [h for text in listings for h in isa_check.hazards_in(text)]
    products = sum(text.count("v_mfma") for text in listings if "gemm_wide" in text)
    assert products > 1000, "the kernels that write out their products are not among the code looked at"
    assert not isa_check.hazards(build.LIB_PATH)


def test_a_value_in_m0_survives_the_load(assembly):
    code = assembly["probe_m0"]
    at = next(i for i, l in enumerate(code) if l.startswith("buffer_load") and l.endswith("lds"))
    given = next(i for i, l in enumerate(code) if l.startswith("s_mov_b32 m0, 7"))
    assert given < at
    reads = [i for i, l in enumerate(code) if re.search(r"[ ,]m0\b", l) and not l.startswith("s_mov_b32 m0") and i > given]
    assert reads and all(i < at for i in reads), "read from m0 after the load has changed it"
