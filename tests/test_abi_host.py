"""Host-side checks of the C ABI that need no GPU: the library loads, exports
what include/coreinfer.h declares, and rejects bad arguments before touching
the device (validation precedes every HIP call)."""

import ctypes
import os
import re

import pytest

from oracle import coreinfer_oracle as orc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "coreinfer.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(coreinfer_\w+)\s*\(", text)))


def test_library_exports_every_declared_symbol(lib):
    names = _declared_symbols()
    assert len(names) >= 15
    for n in names:
        assert hasattr(lib.raw, n), n
    assert set(names) == set(lib.EXPORTS)
    assert lib.version() >= 2


def test_strerror_names_every_status(lib):
    seen = set()
    for code in (0, -1, -2, -3, -4, -5, -6):
        s = lib.strerror(code)
        assert s and s != "unknown status"
        seen.add(s)
    assert len(seen) == 7
    assert lib.strerror(-99) == "unknown status"


def test_keep_count_agrees_with_the_oracle_rule(lib):
    for n in (0, 1, 2, 3, 7, 10, 30, 1024, 11008, 13824, 16384, 36864):
        for f in (1e-6, 0.01, 0.1, 0.2, 0.25, 0.3, 1 / 3, 0.34, 0.4, 0.5, 0.6, 0.999999, 1.0):
            assert lib.keep_count(f, n) == orc.keep_count(f, n), (f, n)
    assert lib.keep_count(0.4, 16384) == 6554 and lib.keep_count(0.4, 36864) == 14746
    k = ctypes.c_int64(0)
    for bad in (0.0, -0.1, 1.0000001, float("nan"), 1e-9):
        assert lib.raw.coreinfer_keep_count(bad, 10, ctypes.byref(k)) == lib.CI_ERR_INVALID_ARG
    assert lib.raw.coreinfer_keep_count(0.5, -1, ctypes.byref(k)) == lib.CI_ERR_INVALID_ARG
    assert lib.raw.coreinfer_keep_count(0.5, 10, None) == lib.CI_ERR_INVALID_ARG


def test_workspace_sizes(lib):
    assert lib.select_workspace_size(256, 16384) >= 16384 * 4
    assert lib.ffn_decode_workspace_size(1, 6554, 4096) >= 1024 * 4096 * 4
    assert lib.ffn_decode_workspace_size(1, 10, 256) >= 10 * 256 * 4
    assert lib.ffn_decode_workspace_size(8, 14746, 9216) >= 8 * 1024 * 9216 * 4
    import torch
    assert lib.ffn_dense_workspace_size(256, 4096, 16384, torch.float16) >= 256 * 16384 * 2
    b = ctypes.c_size_t(0)
    assert lib.raw.coreinfer_select_workspace_size(0, 10, ctypes.byref(b)) == lib.CI_ERR_INVALID_ARG
    assert lib.raw.coreinfer_select_workspace_size(70000, 10, ctypes.byref(b)) == lib.CI_ERR_INVALID_ARG
    assert lib.raw.coreinfer_select_workspace_size(4, 10, None) == lib.CI_ERR_INVALID_ARG
    assert lib.raw.coreinfer_ffn_decode_workspace_size(0, 10, 64, ctypes.byref(b)) == lib.CI_ERR_INVALID_ARG
    assert lib.raw.coreinfer_ffn_dense_workspace_size(4, 64, 64, 9, ctypes.byref(b)) == lib.CI_ERR_BAD_DTYPE


@pytest.mark.parametrize("B", [1, 2, 8, 64, 65, 300])
@pytest.mark.parametrize("M", [1, 7, 511, 2047, 2048, 3000])
@pytest.mark.parametrize("N", [1, 1025, 12289, 13824, 40960, 40961, 70000])
def test_select_batch_keeps_the_pieces_of_its_workspace_apart(lib, B, M, N):
    """Thresholds, histograms, the counters of all B sentences and the byte counts follow each other inside the
    size that is asked for -- also where the sentences are taken one after the other (M >= 2048 or N > 65536) and
    every one of them writes byte counts while the counters of those before it have to stay."""
    if B * M > 65535 * 64:
        pytest.skip("more tokens than a batch may have")
    at = lib.dev_select_layout(B, M, N)
    size = lib.select_batch_workspace_size(B, M, N)
    assert at["thresholds"] == 0 and at["histograms"] >= B * M * 8
    assert at["counts"] >= at["histograms"] + B * 2048 * 8 * 4
    end = at["counts"] + B * N * 4
    if at["part"] >= 0:
        assert at["part"] >= end and at["part"] % 16 == 0
        end = at["part"] + min(B * M, 512) * -(-N // 4096) * 4096   # a byte per neuron, whole registers of four
    assert size >= end
    if B <= 64 and N <= 40960:
        assert at["part"] >= 0


@pytest.mark.parametrize("B,M,N", [(1, 256, 16384), (1, 4, 10), (8, 512, 36864), (2, 2048, 13824), (65, 9, 40)])
def test_select_refuses_a_workspace_that_ends_before_its_counters(lib, B, M, N):
    """What a selection cannot do without: everything in front of the byte counts."""
    F, at = 0x10000, lib.dev_select_layout(B, M, N)
    least = at["part"] if at["part"] >= 0 else lib.select_batch_workspace_size(B, M, N)
    r = lib.raw
    assert r.coreinfer_select_batch(F, B, M, N, N, 0.2, 0.4, F, F, F, least - 1, None) == lib.CI_ERR_WORKSPACE
    if B == 1:
        assert r.coreinfer_select(F, M, N, N, 0.2, 0.4, F, F, F, least - 1, None) == lib.CI_ERR_WORKSPACE
        assert r.coreinfer_select_hidden(F, 1, 0, M, N, N, 0.2, 0.4, F, F, F, least - 1, None) == lib.CI_ERR_WORKSPACE
        assert r.coreinfer_count_tokens(F, M, N, N, 0.2, F, 0, F, least - 1, None) == lib.CI_ERR_WORKSPACE
        assert r.coreinfer_group_select(F, M, 1, N, 0.2, F, F, F, least - 1, None) == lib.CI_ERR_WORKSPACE


@pytest.mark.parametrize("layout", ["out_major", "neuron_major"])
def test_dense_plan_is_the_same_in_any_workspace_of_the_stated_size(lib, layout):
    """A workspace of just the size that the query states gives the plan, and so the bits, that a larger one gives."""
    import ctypes
    import torch
    sizes = [(17, 896, 3136), (39, 512, 1920), (26, 768, 2688), (50, 448, 1600), (7, 416, 1552), (24, 840, 2688)]
    sizes += [(M, d, N) for M in (5, 16, 33, 61, 77, 100, 128, 129, 200, 577) for d in range(256, 2305, 152)
              for N in (2 * d + 8, 3 * d, 4 * d)]
    for M, d, N in sizes:
        best = lib.dev_dense_plan(M, d, N, torch.float16, "relu", layout)
        hidden = (M * N * 4 + 255) // 256 * 256
        beside = lib.ffn_dense_workspace_size(M, d, N, torch.float16) - hidden
        b = ctypes.c_size_t()
        assert lib.raw.coreinfer_ffn_dense_hidden_workspace_size(M, d, N, lib.CI_F16, ctypes.byref(b)) == 0
        assert best["bytes"] <= min(beside, b.value)
        for room in (beside, b.value, 3 * beside):
            assert lib.dev_dense_plan(M, d, N, torch.float16, "relu", layout, room) == best, (M, d, N, room)
        least = lib.dev_dense_plan(M, d, N, torch.float16, "relu", layout, 256)
        assert least["tail"] == 0 and least["bytes"] == 0   # without room none is split


def test_dense_plans_take_shapes_that_are_built(lib):
    """Every tile shape of a plan is one that the setting for tests accepts, and so has a kernel; those that no size takes have none."""
    import torch
    taken = set()
    for M in (5, 17, 33, 48, 64, 77, 90, 112, 113, 128):
        for d in (8, 64, 256, 456, 1024, 4096, 9216, 32768):
            for N in (8, 136, 1024, 2816, 11008, 16384, 36864, 131072):
                for act in ("relu", "swiglu"):
                    for room in (256, 1 << 20, 1 << 62):
                        plan = lib.dev_dense_plan(M, d, N, torch.bfloat16, act, "out_major", room)
                        taken |= {plan["up"], plan["down"]}
    assert len(taken) > 40
    try:
        for tile in taken:
            lib.dev_set_param("gemm_tile", tile)
    finally:
        lib.dev_set_param("gemm_tile", -1)
    for tm, tn in ((8, 4), (8, 7), (8, 8), (0, 2), (9, 2), (1, 1), (1, 9)):
        assert lib.raw.coreinfer_dev_set_param(b"gemm_tile", 16 + 16 * tm + tn) == lib.CI_ERR_INVALID_ARG
    assert lib.raw.coreinfer_dev_set_param(b"gemm_tile", 15) == lib.CI_ERR_INVALID_ARG


@pytest.mark.parametrize("M,d,N,act,up", [
    (2908, 144, 2400, "swiglu", 4), (1142, 128, 3208, "relu", 0), (3505, 768, 2048, "relu", 1),   # 1 to 5 % are promised by others
    (3962, 504, 1920, "relu", 6), (738, 328, 1872, "swiglu", 8), (2755, 304, 4760, "relu", 5),    # more than 8
    (1024, 5120, 13824, "swiglu", 5)])                                                            # rows that the estimate was fitted to
def test_dense_plan_of_short_rows_takes_odd_widths_where_they_promise_enough(lib, M, d, N, act, up):
    import torch
    assert lib.dev_dense_plan(M, d, N, torch.float16, act, "out_major")["up"] == up


def test_dense_plan_reads_large_weights_once(lib):
    """Where the weights are loaded as data that is not read again: at most 128 tokens, k-contiguous rows of whole cache lines, 80 MB
    of a product, and up to 32 tokens or a layer that the memory-side cache does not hold."""
    import torch
    for M, d, N, act, layout, up, down in [
            (32, 3776, 12736, "relu", "out_major", 1, 1),       # 96 MB a product, 192 MB a layer
            (33, 3776, 12736, "relu", "out_major", 0, 0),
            (32, 3072, 12736, "relu", "out_major", 0, 0),       # 78 MB
            (32, 3008, 10048, "swiglu", "out_major", 1, 0),     # 121 and 60 MB
            (77, 4096, 11008, "swiglu", "out_major", 1, 1),     # 180 and 90 MB: 270 of the cache's 268
            (77, 4096, 10880, "swiglu", "out_major", 0, 0),     # 267 MB
            (77, 4096, 11008, "swiglu", "neuron_major", 1, 0),
            (128, 4096, 16384, "relu", "out_major", 0, 0),      # just the cache's size
            (128, 4096, 16448, "relu", "out_major", 1, 1),
            (129, 5120, 20480, "relu", "out_major", 0, 0),
            (32, 5128, 20488, "relu", "out_major", 0, 0)]:
        plan = lib.dev_dense_plan(M, d, N, torch.float16, act, layout)
        assert (plan["up_once"], plan["down_once"]) == (up, down), (M, d, N, act, layout, plan)


def test_shapes_of_more_than_128_rows_have_no_read_once_loads(lib):
    """Tiles of 256 rows, and those for up projections of more than 128 rows, are never planned where the rule takes such loads, and are
    built without them: no setting asks for them."""
    import torch
    lib.dev_set_param("gemm_once", 2)
    try:
        for tile in range(11):
            lib.dev_set_param("gemm_tile", tile)
            plan = lib.dev_dense_plan(256, 4096, 16384, torch.float16, "relu", "out_major")
            assert plan["up"] == tile and plan["up_once"] == (tile in (0, 1, 3)), tile
    finally:
        lib.dev_set_param("gemm_tile", -1)
        lib.dev_set_param("gemm_once", 1)


def test_hidden_call_makes_no_plans_to_check_its_arguments(lib):
    """A call that is refused for want of a workspace has cost what the same refusal of coreinfer_ffn_dense does, far less
    than the size query, which plans both layouts (fastest of many rounds of each)."""
    import ctypes
    import time
    F, M, d, N = 0x10000, 77, 4096, 11008
    b = ctypes.c_size_t()
    dense = lambda: lib.raw.coreinfer_ffn_dense(F, M, F, None, None, F, None, 0, lib.CI_F16, 0, d, N, F, None, None, 0, None)  # noqa: E731
    hidden = lambda: lib.raw.coreinfer_ffn_dense_hidden(F, M, F, None, None, F, None, 0, lib.CI_F16, 0, d, N, F, F, None, 0, None)  # noqa: E731
    query = lambda: lib.raw.coreinfer_ffn_dense_hidden_workspace_size(M, d, N, lib.CI_F16, ctypes.byref(b))  # noqa: E731
    assert dense() == lib.CI_ERR_WORKSPACE and hidden() == lib.CI_ERR_WORKSPACE and query() == 0
    best = {}
    for _ in range(60):
        for name, f in (("dense", dense), ("hidden", hidden), ("query", query)):
            t = time.perf_counter()
            for _ in range(50):
                f()
            best[name] = min(best.get(name, 1.0), (time.perf_counter() - t) / 50)
    assert best["hidden"] < best["dense"] + 0.4 * best["query"], best


@pytest.mark.parametrize("gathered", [False, True])
def test_decode_slices_leave_few_compute_units_idle(lib, gathered):
    """On 256 compute units: narrow rows keep every slice (two workgroups on a compute unit cost them nothing) but a
    sixth at most; wide ones of several sentences have at most one workgroup per compute unit, a multiple of eight
    where that idles little of the chip; and never more slices than the scratch is sized for."""
    import torch
    for dtype, e in ((torch.float16, 2), (torch.float32, 4)):
        for d in (256, 1024, 2048, 3072, 4096, 9216):
            for K in (5, 410, 14746):
                for B in list(range(1, 70)) + [200, 256, 257, 1000]:
                    bound = min(-(-256 // B), K)
                    n = lib.dev_decode_slices(B, K, d, dtype, gathered)
                    assert 1 <= n <= bound
                    if B == 1 or K < 256 // B:
                        assert n == bound
                    elif d * e < 6144:
                        assert n == bound if gathered or d * e < 4096 else 6 * n >= 5 * bound
                    elif d * e >= 8192 and B <= 256:
                        assert n * B <= 256 and n * B >= (0.72 if gathered else 0.75) * (256 // B * B)
                        assert n == 256 // B or n % 8 == 0


def test_dense_workspace_holds_the_sums_of_split_tiles_only(lib):
    """At most a few rounds of 256 workgroups leave partial sums, whatever the product's size: 4096 x 9216 from 36864
    (576 tiles of 256 x 256, 64 of them split in four) takes 67 MB beside the hidden matrix."""
    import torch
    b = ctypes.c_size_t(0)
    for M, d, N in [(5, 4096, 16384), (77, 4096, 11008), (256, 4096, 16384), (700, 4096, 16384), (1024, 5120, 13824),
                    (2090, 1024, 648), (4096, 9216, 36864), (8000, 9216, 36864), (65535, 8192, 28672)]:
        assert lib.raw.coreinfer_ffn_dense_hidden_workspace_size(M, d, N, lib.CI_F16, ctypes.byref(b)) == lib.CI_OK
        sums = b.value
        assert 256 <= sums <= 8 * 256 * (256 * 256 + 64) * 4 + 256
        if M == 4096:
            assert sums == 64 * 4 * (256 * 256 + 64) * 4 + 256
        hidden = -(-M * N * 4 // 256) * 256
        assert lib.ffn_dense_workspace_size(M, d, N, torch.float16) == hidden + sums
    r, F = lib.raw.coreinfer_ffn_dense, 0x10000
    hidden = 256 * 16384 * 4
    assert r(F, 256, F, None, None, F, None, 0, 1, 0, 4096, 16384, F, None, F, hidden + 255, None) == lib.CI_ERR_WORKSPACE
    r = lib.raw.coreinfer_ffn_dense_hidden
    assert r(F, 256, F, None, None, F, None, 0, 1, 0, 4096, 16384, F, F, F, 255, None) == lib.CI_ERR_WORKSPACE


FAKE = 0x10000  # a non-null, 16-byte aligned address that is never dereferenced on these paths


def test_select_rejects_bad_arguments_without_a_gpu(lib):
    r = lib.raw.coreinfer_select
    ok_ws = 1 << 20
    assert r(None, 4, 64, 64, 0.2, 0.4, FAKE, None, FAKE, ok_ws, None) == lib.CI_ERR_INVALID_ARG
    assert r(FAKE, 4, 64, 64, 0.2, 0.4, None, None, FAKE, ok_ws, None) == lib.CI_ERR_INVALID_ARG
    assert r(FAKE, 0, 64, 64, 0.2, 0.4, FAKE, None, FAKE, ok_ws, None) == lib.CI_ERR_INVALID_ARG
    assert r(FAKE, 4, 64, 64, 0.0, 0.4, FAKE, None, FAKE, ok_ws, None) == lib.CI_ERR_INVALID_ARG
    assert r(FAKE, 4, 64, 64, 0.2, 1.5, FAKE, None, FAKE, ok_ws, None) == lib.CI_ERR_INVALID_ARG
    assert r(FAKE, 4, 64, 32, 0.2, 0.4, FAKE, None, FAKE, ok_ws, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(FAKE + 2, 4, 64, 64, 0.2, 0.4, FAKE, None, FAKE, ok_ws, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(FAKE, 4, 64, 64, 0.2, 0.4, FAKE, None, None, ok_ws, None) == lib.CI_ERR_WORKSPACE
    assert r(FAKE, 4, 64, 64, 0.2, 0.4, FAKE, None, FAKE, 16, None) == lib.CI_ERR_WORKSPACE


def test_compact_rejects_bad_arguments_without_a_gpu(lib):
    r = lib.raw.coreinfer_compact
    F = FAKE
    # (w_up, w_gate, b_up, w_down, layout, dtype, act, d, N, idx, K, up_c, gate_c, b_c, down_c, down_c_layout,
    #  status, stream)
    assert r(F, None, None, F, 0, 7, 0, 64, 128, F, 8, F, None, None, F, 1, None, None) == lib.CI_ERR_BAD_DTYPE
    assert r(F, None, None, F, 0, 1, 5, 64, 128, F, 8, F, None, None, F, 1, None, None) == lib.CI_ERR_BAD_DTYPE
    assert r(F, None, None, F, 3, 1, 0, 64, 128, F, 8, F, None, None, F, 1, None, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(None, None, None, F, 0, 1, 0, 64, 128, F, 8, F, None, None, F, 1, None, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, None, None, F, 0, 1, 0, 64, 128, F, 200, F, None, None, F, 1, None, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, None, None, F, 0, 1, 0, 64, 128, None, 8, F, None, None, F, 1, None, None) == lib.CI_ERR_INVALID_ARG
    # gate given for ReLU / missing for SwiGLU; bias in without bias out
    assert r(F, F, None, F, 0, 1, 0, 64, 128, F, 8, F, F, None, F, 1, None, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, None, None, F, 0, 1, 1, 64, 128, F, 8, F, None, None, F, 1, None, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, None, F, F, 0, 1, 0, 64, 128, F, 8, F, None, None, F, 1, None, None) == lib.CI_ERR_INVALID_ARG
    # d not a multiple of 8 halfs; misaligned pointer
    assert r(F, None, None, F, 0, 1, 0, 60, 128, F, 8, F, None, None, F, 1, None, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F + 8, None, None, F, 0, 1, 0, 64, 128, F, 8, F, None, None, F, 1, None, None) == lib.CI_ERR_BAD_LAYOUT
    # layout of the compact down matrix out of range; up bias with a gated FFN
    assert r(F, None, None, F, 0, 1, 0, 64, 128, F, 8, F, None, None, F, 2, None, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, F, F, F, 0, 1, 1, 64, 128, F, 8, F, F, F, F, 0, None, None) == lib.CI_ERR_INVALID_ARG
    ld = ctypes.c_int64(0)
    assert lib.raw.coreinfer_compact_down_ld(6554, 1, ctypes.byref(ld)) == lib.CI_OK and ld.value == 6560
    assert lib.raw.coreinfer_compact_down_ld(410, 0, ctypes.byref(ld)) == lib.CI_OK and ld.value == 412
    assert lib.raw.coreinfer_compact_down_ld(0, 2, ctypes.byref(ld)) == lib.CI_OK and ld.value == 0
    assert lib.raw.coreinfer_compact_down_ld(8, 5, ctypes.byref(ld)) == lib.CI_ERR_BAD_DTYPE
    assert lib.raw.coreinfer_compact_down_ld(-1, 1, ctypes.byref(ld)) == lib.CI_ERR_INVALID_ARG
    assert lib.raw.coreinfer_compact_down_ld(8, 1, None) == lib.CI_ERR_INVALID_ARG


def test_preferred_compact_layout_and_its_arguments(lib):
    """Pure host function: small layers -> neuron-major, large ones -> output-major, shapes the
    single-launch decode does not take -> neuron-major."""
    import torch
    out = ctypes.c_int(-1)
    r = lib.raw.coreinfer_compact_preferred_layout
    assert r(2765, 5120, lib.CI_BF16, lib.CI_ACT_SWIGLU, ctypes.byref(out)) == lib.CI_OK
    assert out.value == lib.CI_DOWN_NEURON_MAJOR
    assert r(8295, 5120, lib.CI_BF16, lib.CI_ACT_SWIGLU, ctypes.byref(out)) == lib.CI_OK
    assert out.value == lib.CI_DOWN_OUT_MAJOR
    assert r(20000, 32768, lib.CI_F16, lib.CI_ACT_RELU, ctypes.byref(out)) == lib.CI_OK   # d beyond the single launch
    assert out.value == lib.CI_DOWN_NEURON_MAJOR
    assert r(0, 4096, lib.CI_F16, lib.CI_ACT_RELU, ctypes.byref(out)) == lib.CI_OK and out.value == lib.CI_DOWN_NEURON_MAJOR
    assert r(10, 4096, 9, lib.CI_ACT_RELU, ctypes.byref(out)) == lib.CI_ERR_BAD_DTYPE
    assert r(10, 0, lib.CI_F16, lib.CI_ACT_RELU, ctypes.byref(out)) == lib.CI_ERR_INVALID_ARG
    assert r(-1, 64, lib.CI_F16, lib.CI_ACT_RELU, ctypes.byref(out)) == lib.CI_ERR_INVALID_ARG
    assert r(10, 64, lib.CI_F16, lib.CI_ACT_RELU, None) == lib.CI_ERR_INVALID_ARG
    assert lib.compact_preferred_layout(6554, 4096, torch.float16, "relu") in ("neuron_major", "out_major")
    plan = lib.dev_fused_plan(6554, 4096, torch.float16, "relu")
    assert plan["chunks"] >= 2 and plan["chunks"] * plan["chunk_neurons"] >= 6554 and plan["loads_per_row"] == 1
    assert (plan["chunks"] - 1) * plan["chunk_neurons"] < 6554


def test_select_batch_rejects_bad_arguments_without_a_gpu(lib):
    r = lib.raw.coreinfer_select_batch
    ok_ws = 1 << 22
    b = ctypes.c_size_t(0)
    assert lib.raw.coreinfer_select_batch_workspace_size(8, 512, 36864, ctypes.byref(b)) == lib.CI_OK
    assert b.value >= 8 * 36864 * 4 + 8 * 512 * 8
    assert lib.select_batch_workspace_size(1, 256, 16384) == lib.select_workspace_size(256, 16384)
    assert lib.raw.coreinfer_select_batch_workspace_size(0, 4, 64, ctypes.byref(b)) == lib.CI_ERR_INVALID_ARG
    assert lib.raw.coreinfer_select_batch_workspace_size(70000, 4, 64, ctypes.byref(b)) == lib.CI_ERR_INVALID_ARG
    assert lib.raw.coreinfer_select_batch_workspace_size(2, 4, 64, None) == lib.CI_ERR_INVALID_ARG
    # (act, B, M, N, ld, alpha, beta, core_idx, counts, ws, ws_bytes, stream)
    assert r(None, 2, 4, 64, 64, 0.2, 0.4, FAKE, None, FAKE, ok_ws, None) == lib.CI_ERR_INVALID_ARG
    assert r(FAKE, 2, 4, 64, 64, 0.2, 0.4, None, None, FAKE, ok_ws, None) == lib.CI_ERR_INVALID_ARG
    assert r(FAKE, 0, 4, 64, 64, 0.2, 0.4, FAKE, None, FAKE, ok_ws, None) == lib.CI_ERR_INVALID_ARG
    assert r(FAKE, 2, 4, 64, 64, 0.2, 2.0, FAKE, None, FAKE, ok_ws, None) == lib.CI_ERR_INVALID_ARG
    assert r(FAKE, 2, 4, 64, 32, 0.2, 0.4, FAKE, None, FAKE, ok_ws, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(FAKE, 2, 4, 64, 64, 0.2, 0.4, FAKE + 2, None, FAKE, ok_ws, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(FAKE, 2, 4, 64, 64, 0.2, 0.4, FAKE, None, None, ok_ws, None) == lib.CI_ERR_WORKSPACE
    assert r(FAKE, 2, 4, 64, 64, 0.2, 0.4, FAKE, None, FAKE, 16, None) == lib.CI_ERR_WORKSPACE


def test_static_decode_rejects_bad_arguments_without_a_gpu(lib):
    """coreinfer_ffn_decode_static validates like coreinfer_ffn_decode and turns down what its
    scratch cannot hold before any HIP call."""
    r = lib.raw.coreinfer_ffn_decode_static
    F = FAKE
    def desc(K=8, d=64, N=128, layout=1, ld=0, core=None, gate=None, bias=None):
        return lib.ci_ffn_weights(F, gate, bias, F, None, core, K, d, N, ld, layout)
    # (x, B, w, dtype, act, y, status_out, stream)
    assert r(F, 1, None, 1, 0, F, None, None) == lib.CI_ERR_INVALID_ARG
    assert r(None, 1, ctypes.byref(desc()), 1, 0, F, None, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 1, ctypes.byref(desc()), 7, 0, F, None, None) == lib.CI_ERR_BAD_DTYPE
    assert r(F, 1, ctypes.byref(desc(layout=5)), 1, 0, F, None, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, 1, ctypes.byref(desc(gate=F)), 1, 0, F, None, None) == lib.CI_ERR_INVALID_ARG       # gate with ReLU
    assert r(F, 1, ctypes.byref(desc(gate=F, bias=F)), 1, 1, F, None, None) == lib.CI_ERR_INVALID_ARG  # bias with SwiGLU
    assert r(F, 1, ctypes.byref(desc(d=60)), 1, 0, F, None, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, 1, ctypes.byref(desc(layout=0, ld=4)), 1, 0, F, None, None) == lib.CI_ERR_BAD_LAYOUT  # ld < K
    assert r(F, 1, ctypes.byref(desc()), 1, 0, F, F + 2, None) == lib.CI_ERR_BAD_LAYOUT               # status_out misaligned
    assert r(F, 1, ctypes.byref(desc(K=200000, N=200000, layout=0, ld=200000)), 1, 0, F, None, None) == lib.CI_ERR_WORKSPACE
    assert r(F, 8, ctypes.byref(desc(K=4096, d=32768, N=4096)), 1, 0, F, None, None) == lib.CI_ERR_WORKSPACE


def test_compact_update_rejects_bad_arguments_without_a_gpu(lib):
    r = lib.raw.coreinfer_compact_update
    F = FAKE
    big = 1 << 24
    # (w_up, w_gate, b_up, w_down, layout, dtype, act, d, N, new_idx, K, slot_idx, w_up_c, w_gate_c, b_up_c,
    #  w_down_c, down_c_layout, changed, ws, ws_bytes, stream)
    assert r(F, None, None, F, 0, 6, 0, 64, 128, F, 8, F, F, None, None, F, 1, None, F, big, None) == lib.CI_ERR_BAD_DTYPE
    assert r(F, None, None, F, 3, 1, 0, 64, 128, F, 8, F, F, None, None, F, 1, None, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, None, None, F, 0, 1, 0, 64, 128, None, 8, F, F, None, None, F, 1, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, None, None, F, 0, 1, 0, 64, 128, F, 8, None, F, None, None, F, 1, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, None, None, F, 0, 1, 0, 64, 128, F, 200, F, F, None, None, F, 1, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, None, None, F, 0, 1, 1, 64, 128, F, 8, F, F, None, None, F, 1, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, None, F, F, 0, 1, 0, 64, 128, F, 8, F, F, None, None, F, 1, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, None, None, F, 0, 1, 0, 60, 128, F, 8, F, F, None, None, F, 1, None, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, None, None, F, 0, 1, 0, 64, 128, F, 8, F + 2, F, None, None, F, 1, None, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, None, None, F, 0, 1, 0, 64, 128, F, 8, F, F, None, None, F, 1, None, None, big, None) == lib.CI_ERR_WORKSPACE
    assert r(F, None, None, F, 0, 1, 0, 64, 128, F, 8, F, F, None, None, F, 1, None, F, 100, None) == lib.CI_ERR_WORKSPACE
    assert r(F, None, None, F, 0, 1, 0, 64, 128, F, 8, F, F, None, None, F, 7, None, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    n = ctypes.c_size_t(0)
    assert lib.raw.coreinfer_compact_update_workspace_size(128, 8, ctypes.byref(n)) == lib.CI_OK
    assert n.value >= (128 + 3 * 8 + 1) * 4
    assert lib.raw.coreinfer_compact_update_workspace_size(128, 129, ctypes.byref(n)) == lib.CI_ERR_INVALID_ARG


def test_ffn_decode_rejects_bad_arguments_without_a_gpu(lib):
    r = lib.raw.coreinfer_ffn_decode
    F = FAKE
    big = 1 << 30

    def W(**kw):
        base = dict(w_up=F, w_gate=None, b_up=None, w_down=F, b_down=None, core_idx=None, K=16, d=64, N=16,
                    ld_down=0, down_layout=1)
        base.update(kw)
        return ctypes.byref(lib.ci_ffn_weights(**base))

    assert r(F, 1, None, 1, 0, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 1, W(), 9, 0, F, F, big, None) == lib.CI_ERR_BAD_DTYPE
    assert r(F, 1, W(), 1, 2, F, F, big, None) == lib.CI_ERR_BAD_DTYPE
    assert r(None, 1, W(), 1, 0, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 1, W(), 1, 0, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 0, W(), 1, 0, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 1, W(w_up=None), 1, 0, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 1, W(), 1, 1, F, F, big, None) == lib.CI_ERR_INVALID_ARG          # SwiGLU without gate
    assert r(F, 1, W(w_gate=F), 1, 0, F, F, big, None) == lib.CI_ERR_INVALID_ARG   # ReLU with gate
    assert r(F, 1, W(d=60), 1, 0, F, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, 1, W(d=62), 0, 0, F, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F + 4, 1, W(), 1, 0, F, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, 1, W(core_idx=F, N=0), 1, 0, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 1, W(), 1, 0, F, None, big, None) == lib.CI_ERR_WORKSPACE
    assert r(F, 1, W(), 1, 0, F, F, 64, None) == lib.CI_ERR_WORKSPACE
    # up bias with a gated FFN; layout enum; output-major compact matrix: row length, gathered rows
    assert r(F, 1, W(w_gate=F, b_up=F), 1, 1, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 1, W(down_layout=2), 1, 0, F, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, 1, W(down_layout=0, ld_down=8), 1, 0, F, F, big, None) == lib.CI_ERR_BAD_LAYOUT     # shorter than K
    assert r(F, 1, W(down_layout=0, ld_down=20), 1, 0, F, F, big, None) == lib.CI_ERR_BAD_LAYOUT    # not whole vectors
    assert r(F, 1, W(down_layout=0, ld_down=16, core_idx=F), 1, 0, F, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    st = lib.raw.coreinfer_ffn_decode_status
    assert st(None, F, None) == lib.CI_ERR_INVALID_ARG and st(F, None, None) == lib.CI_ERR_INVALID_ARG
    assert st(F + 4, F, None) == lib.CI_ERR_BAD_LAYOUT


def test_ffn_dense_rejects_bad_arguments_without_a_gpu(lib):
    r = lib.raw.coreinfer_ffn_dense
    F = FAKE
    big = 1 << 30
    # (X, M, w_up, w_gate, b_up, w_down, b_down, layout, dtype, act, d, N, Y, A, ws, ws_bytes, stream)
    assert r(F, 8, F, None, None, F, None, 0, 5, 0, 64, 128, F, None, F, big, None) == lib.CI_ERR_BAD_DTYPE
    assert r(F, 8, F, None, None, F, None, 2, 1, 0, 64, 128, F, None, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(None, 8, F, None, None, F, None, 0, 1, 0, 64, 128, F, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 8, F, None, None, F, None, 0, 1, 0, 64, 128, None, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 8, F, None, None, None, None, 0, 1, 0, 64, 128, F, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 8, F, None, None, F, None, 0, 1, 1, 64, 128, F, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 8, F, None, None, F, None, 0, 1, 0, 64, 100, F, None, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, 8, F, None, None, F, None, 0, 1, 0, 64, 128, F, None, None, big, None) == lib.CI_ERR_WORKSPACE
    assert r(F, 8, F, None, None, F, None, 0, 1, 0, 64, 128, F, None, F, 100, None) == lib.CI_ERR_WORKSPACE


def test_next_row_entry_points_reject_bad_arguments_without_a_gpu(lib):
    F = FAKE
    r = lib.raw.coreinfer_count_tokens
    assert r(None, 4, 64, 64, 0.2, F, 0, F, 1 << 20, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 4, 64, 64, 0.2, None, 0, F, 1 << 20, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 4, 64, 64, 1.2, F, 0, F, 1 << 20, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 4, 64, 10, 0.2, F, 0, F, 1 << 20, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, 4, 64, 64, 0.2, F, 0, None, 1 << 20, None) == lib.CI_ERR_WORKSPACE
    assert r(F, 4, 64, 64, 0.2, F, 0, F, 16, None) == lib.CI_ERR_WORKSPACE
    r = lib.raw.coreinfer_count_select
    assert r(None, 64, 10, 0.4, F, F, 256, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 64, 70000, 0.4, F, F, 256, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 64, 10, 0.0, F, F, 256, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 64, 10, 0.4, F, None, 256, None) == lib.CI_ERR_WORKSPACE
    assert r(F, 64, 10, 0.4, F, F, 8, None) == lib.CI_ERR_WORKSPACE
    r = lib.raw.coreinfer_group_select
    big = 1 << 20
    assert r(None, 3, 8, 64, 0.2, F, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 0, 8, 64, 0.2, F, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 3, 80, 64, 0.2, F, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 3, 8, 64, 2.0, F, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 3, 8, 64, 0.2, F, None, F, 16, None) == lib.CI_ERR_WORKSPACE
    r = lib.raw.coreinfer_assign_group
    assert r(F, 4, F, 0, 4, F, F, None) == lib.CI_ERR_INVALID_ARG
    assert r(None, 4, F, 3, 4, F, F, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 4, None, 3, 4, F, F, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 4, F, 3, 4, None, F, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 4, F, 3, 4, F, F + 2, None) == lib.CI_ERR_BAD_LAYOUT
    r = lib.raw.coreinfer_select_hidden
    big = 1 << 22
    assert r(None, 1, 0, 4, 64, 64, 0.2, 0.4, F, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 1, 0, 4, 64, 64, 0.2, 0.4, None, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 9, 0, 4, 64, 64, 0.2, 0.4, F, None, F, big, None) == lib.CI_ERR_BAD_DTYPE
    assert r(F, 1, 7, 4, 64, 64, 0.2, 0.4, F, None, F, big, None) == lib.CI_ERR_BAD_DTYPE
    assert r(F, 1, 0, 0, 64, 64, 0.2, 0.4, F, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 1, 0, 4, 64, 64, 0.0, 0.4, F, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 1, 0, 4, 64, 32, 0.2, 0.4, F, None, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F + 1, 1, 0, 4, 64, 64, 0.2, 0.4, F, None, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F + 2, 0, 0, 4, 64, 64, 0.2, 0.4, F, None, F, big, None) == lib.CI_ERR_BAD_LAYOUT   # fp32 needs 4 bytes
    assert r(F, 1, 0, 4, 64, 64, 0.2, 0.4, F, None, None, big, None) == lib.CI_ERR_WORKSPACE
    assert r(F, 1, 0, 4, 64, 64, 0.2, 0.4, F, None, F, 16, None) == lib.CI_ERR_WORKSPACE
    r = lib.raw.coreinfer_ffn_dense_hidden
    ok = dict(X=F, M=8, up=F, gate=None, bup=None, down=F, bdown=None, layout=0, dt=1, act=0, d=64, N=128, Y=F, H=F,
              ws=F, wsb=big)
    def call(**kw):
        a = dict(ok); a.update(kw)
        return r(a["X"], a["M"], a["up"], a["gate"], a["bup"], a["down"], a["bdown"], a["layout"], a["dt"], a["act"],
                 a["d"], a["N"], a["Y"], a["H"], a["ws"], a["wsb"], None)
    assert call(H=None) == lib.CI_ERR_INVALID_ARG
    assert call(X=None) == lib.CI_ERR_INVALID_ARG
    assert call(down=None) == lib.CI_ERR_INVALID_ARG          # Y wanted without a down matrix
    assert call(act=1) == lib.CI_ERR_INVALID_ARG              # gated FFN without a gate matrix
    assert call(dt=5) == lib.CI_ERR_BAD_DTYPE
    assert call(layout=3) == lib.CI_ERR_BAD_LAYOUT
    assert call(d=60) == lib.CI_ERR_BAD_LAYOUT
    assert call(H=F + 8) == lib.CI_ERR_BAD_LAYOUT
    assert call(ws=None) == lib.CI_ERR_WORKSPACE
    assert call(M=0) == lib.CI_ERR_INVALID_ARG
    r = lib.raw.coreinfer_assign_centroid
    assert r(None, 4, 64, 64, F, 3, F, F, F, 1 << 20, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 4, 64, 64, None, 3, F, F, F, 1 << 20, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 4, 64, 64, F, 3, None, F, F, 1 << 20, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 4, 64, 64, F, 3, F, None, F, 1 << 20, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 0, 64, 64, F, 3, F, F, F, 1 << 20, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 4, 64, 64, F, 0, F, F, F, 1 << 20, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 4, 0, 64, F, 3, F, F, F, 1 << 20, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 4, 64, 32, F, 3, F, F, F, 1 << 20, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, 4, 64, 64, F + 2, 3, F, F, F, 1 << 20, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, 4, 64, 64, F, 3, F, F, None, 1 << 20, None) == lib.CI_ERR_WORKSPACE
    assert r(F, 4, 64, 64, F, 3, F, F, F, 100, None) == lib.CI_ERR_WORKSPACE
    r = lib.raw.coreinfer_core_similarity
    assert r(F, 4, F, 4, None, None) == lib.CI_ERR_INVALID_ARG
    assert r(None, 4, F, 4, F, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, -1, F, 4, F, None) == lib.CI_ERR_INVALID_ARG
    assert r(F + 2, 4, F, 4, F, None) == lib.CI_ERR_BAD_LAYOUT


def test_union_entry_points_reject_bad_arguments_without_a_gpu(lib):
    F = FAKE
    big = 1 << 30
    r = lib.raw.coreinfer_union_build
    # (core_idx, B, K, N, max_rows, union_idx, union_mask, union_count, ws, ws_bytes, stream)
    assert r(None, 2, 8, 64, 16, F, F, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 9, 8, 64, 64, F, F, F, F, big, None) == lib.CI_ERR_INVALID_ARG      # more than 8 sentences
    assert r(F, 0, 8, 64, 64, F, F, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 2, 80, 64, 64, F, F, F, F, big, None) == lib.CI_ERR_INVALID_ARG     # K > N
    assert r(F, 2, 8, 64, 15, F, F, F, F, big, None) == lib.CI_ERR_INVALID_ARG      # max_rows < min(N, B*K)
    assert r(F, 2, 8, 64, 16, None, F, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 2, 8, 64, 16, F, F, None, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F + 2, 2, 8, 64, 16, F, F, F, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, 2, 8, 64, 16, F, F, F, None, big, None) == lib.CI_ERR_WORKSPACE
    assert r(F, 2, 8, 64, 16, F, F, F, F, 64, None) == lib.CI_ERR_WORKSPACE
    n = ctypes.c_size_t(0)
    assert lib.raw.coreinfer_union_workspace_size(36864, ctypes.byref(n)) == lib.CI_OK and n.value >= 36864 * 4
    assert lib.raw.coreinfer_union_workspace_size(0, ctypes.byref(n)) == lib.CI_ERR_INVALID_ARG

    q = lib.raw.coreinfer_ffn_decode_union_workspace_size
    assert q(8, 36864, 9216, 1, 0, ctypes.byref(n)) == lib.CI_OK
    # partial dots [1 chunk][1][36864][8] + partial sums [8][256][9216], fp32
    assert n.value >= (36864 * 8 + 8 * 256 * 9216) * 4
    assert q(9, 64, 64, 1, 0, ctypes.byref(n)) == lib.CI_ERR_INVALID_ARG
    assert q(8, 64, 60, 1, 0, ctypes.byref(n)) == lib.CI_ERR_BAD_LAYOUT
    assert q(8, 64, 64, 7, 0, ctypes.byref(n)) == lib.CI_ERR_BAD_DTYPE

    r = lib.raw.coreinfer_ffn_decode_union

    def W(**kw):
        base = dict(w_up=F, w_gate=None, b_up=None, w_down=F, b_down=None, core_idx=None, K=0, d=64, N=128)
        base.update(kw)
        return ctypes.byref(lib.ci_ffn_weights(**base))

    # (x, B, w, union_idx, union_mask, union_count, max_rows, dtype, act, y, ws, ws_bytes, stream)
    assert r(F, 2, None, F, F, F, 128, 1, 0, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(None, 2, W(), F, F, F, 128, 1, 0, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 2, W(), None, F, F, 128, 1, 0, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 2, W(), F, F, None, 128, 1, 0, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 9, W(), F, F, F, 128, 1, 0, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 2, W(N=0), F, F, F, 128, 1, 0, F, F, big, None) == lib.CI_ERR_INVALID_ARG
    assert r(F, 2, W(), F, F, F, 128, 1, 1, F, F, big, None) == lib.CI_ERR_INVALID_ARG   # SwiGLU without gate
    assert r(F, 2, W(d=60), F, F, F, 128, 1, 0, F, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, 2, W(), F + 2, F, F, 128, 1, 0, F, F, big, None) == lib.CI_ERR_BAD_LAYOUT
    assert r(F, 2, W(), F, F, F, 128, 4, 0, F, F, big, None) == lib.CI_ERR_BAD_DTYPE
    assert r(F, 2, W(), F, F, F, 128, 1, 0, F, None, big, None) == lib.CI_ERR_WORKSPACE
    assert r(F, 2, W(), F, F, F, 128, 1, 0, F, F, 1024, None) == lib.CI_ERR_WORKSPACE


def test_development_hook_validation(lib):
    """csrc/coreinfer_dev.h: launch-shape parameters, not declared in the installed header."""
    r = lib.raw.coreinfer_dev_set_param
    assert r(b"no_such_knob", 1) == lib.CI_ERR_INVALID_ARG
    assert r(b"decode_wgs_per_cu", 0) == lib.CI_ERR_INVALID_ARG
    assert r(None, 1) == lib.CI_ERR_INVALID_ARG
    assert r(b"decode_wgs_per_cu", 2) == lib.CI_OK and r(b"decode_wgs_per_cu", 1) == lib.CI_OK
    # no setting makes a call skip its output: the two that did are gone
    assert r(b"decode_skip_reduce", 1) == lib.CI_ERR_INVALID_ARG
    assert r(b"select_debug", 1) == lib.CI_ERR_INVALID_ARG
    assert "coreinfer_dev_set_param" not in _declared_symbols()


def test_development_probes_validate_before_launching(lib):
    """csrc/coreinfer_dev.h: the load-stream probes reject anything that would read outside the buffer."""
    import ctypes
    vp, i64, ci_ = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int
    sp = lib.raw.coreinfer_dev_stream_probe
    sp.restype = ci_
    sp.argtypes = [vp, i64, i64, ci_, ci_, ci_, ci_, ci_, vp, vp]
    F = 0x100000
    assert sp(None, 1 << 20, 1 << 16, 0, 4, 64, 8, 1, F, None) == lib.CI_ERR_INVALID_ARG
    assert sp(F, 1 << 20, 1 << 16, 1, 17, 64, 8, 1, F, None) == lib.CI_ERR_INVALID_ARG   # 17 windows of 64 KB > 1 MB
    assert sp(F, 1 << 20, 512, 0, 4, 64, 8, 1, F, None) == lib.CI_ERR_INVALID_ARG         # window < 16 * threads
    assert sp(F, 1 << 20, 1 << 16, 0, 4, 96, 8, 1, F, None) == lib.CI_ERR_INVALID_ARG     # threads not whole waves
    assert sp(F, 1 << 20, 1 << 16, 0, 4, 64, 3, 1, F, None) == lib.CI_ERR_INVALID_ARG     # depth
    assert sp(F + 8, 1 << 20, 1 << 16, 0, 4, 64, 8, 1, F, None) == lib.CI_ERR_BAD_LAYOUT
    tp = lib.raw.coreinfer_dev_tile_probe
    tp.restype = ci_
    tp.argtypes = [vp, i64, i64, ci_, ci_, ci_, ci_, ci_, vp, vp]
    # 256 rows of 8 KB per workgroup: two workgroups need 4 MB - 8 KB + 64 * 128 bytes
    assert tp(F, (4 << 20) - 1, 8192, 0, 2, 8, 64, 1, F, None) == lib.CI_ERR_INVALID_ARG
    assert tp(F, 1 << 20, 8192, 1, 2, 8, 64, 1, F, None) == lib.CI_ERR_INVALID_ARG        # shared rows: 2 MB needed
    assert tp(F, 1 << 30, 64, 1, 2, 8, 1, 1, F, None) == lib.CI_ERR_INVALID_ARG           # pitch < 128
    assert tp(F, 1 << 30, 8192, 1, 2, 5, 64, 1, F, None) == lib.CI_ERR_INVALID_ARG        # depth
    assert "coreinfer_dev_stream_probe" not in _declared_symbols()


def test_workloads_module_has_the_five_configurations():
    from paper_2410_18311_amd import workloads as wl
    assert len(wl.WORKLOADS) == 5
    c2 = wl.WORKLOADS["opt6.7b_relu_f16"]
    assert (c2.d, c2.N, c2.L, c2.M, c2.alpha, c2.betas) == (4096, 16384, 32, 256, 0.2, (0.4,))
    t = wl.tiny_relu_f32_numpy()
    assert t["w_up"].shape == (1024, 256) and t["w_down"].shape == (256, 1024)
    assert t["x_prefill"].shape == (32, 256) and t["x_decode"].shape == (16, 256)
    small = c2.scaled(d=64, N=128, M=4, L=1)
    w = wl.layer_weights(small, 0)
    assert w["w_up"].shape == (128, 64) and w["w_down"].shape == (64, 128) and w["w_gate"] is None
    again = wl.layer_weights(small, 0)
    assert (w["w_up"] == again["w_up"]).all()


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0
    assert "ONE GPU" in (r.stdout + r.stderr)


def test_bench_line_fields_are_built_from_the_documented_pieces():
    """The traffic note is only used for the launch size it was measured at."""
    import importlib.util
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(root, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    assert bench.read_traffic_note("opt6.7b_relu_f16", 0.4, 107410228) is not None
    assert bench.read_traffic_note("opt6.7b_relu_f16", 0.4, 2 * 107410228) is None
    assert bench.read_traffic_note("no_such_workload", 0.4, 1) is None


def test_bench_prints_one_short_line_with_every_field_of_its_contract():
    import importlib.util
    import json
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    x = 12345.678901234567

    def record(name, beta):
        return {"metric": "decode_sparse_ffn_tokens_per_s", "value": x, "unit": "tokens/s", "steps": 20, "warmup": 5,
                "ms_per_step": x, "dtype": "bf16",
                "config": {"workload": name, "act": "swiglu", "d_model": 5120, "d_ff": 13824, "layers": 40,
                           "prefill_tokens": 1024, "decode_tokens": 256, "sentences": 1, "alpha": 0.2, "beta": beta,
                           "core_neurons": 13824, "decode_mode": "compacted, w_down_c neuron_major",
                           "decode_launch": "hip_graph_per_token",
                           "value_definition": "decode tokens of a step / GPU time of the step's decode phase (HIP events)"},
                "roofline": {"kernel": "k" * 200, "bound": "hbm", "achieved": x, "peak": 8000.0, "unit": "GB/s", "frac": x / 3e4,
                             "traffic": None, "bytes_per_launch": 1 << 40, "us_per_launch": x, "note": "n" * 400},
                "select_us_per_layer": x, "dense_prefill_tflops": x,
                "parity": {"core_set_bit_exact": True, "decode_max_abs_err_over_rms": x, "layers": list(range(99))},
                "cpu_baseline": {"value": x, "unit": "tokens/s", "cores": 256, "kind": "oracle", "sample": "s" * 300}}
    others = [record(n, 0.2 if b is None else b) for n, b, _, _ in bench.OTHER_WORKLOADS]
    line = json.dumps(bench.printed_line(record(bench.TOP_WORKLOAD, 0.2), others))
    assert "\n" not in line and len(line) < 2000, len(line)
    got = json.loads(line)
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config"):
        assert key in got
    assert got["value"] == x and got["ms_per_step"] == x and len(got["workloads"]) == len(bench.OTHER_WORKLOADS)
    alone = bench.printed_line({**record(bench.TOP_WORKLOAD, 0.2), "parity": None, "cpu_baseline": None}, None)
    assert "workloads" not in alone and "parity" not in alone


def test_per_token_call_of_the_binding_returns_the_status_of_the_c_call(lib):
    """csrc/binding.c hands its arguments on as they are: the same status for every argument that is refused, and no call for arguments
    that are not numbers."""
    import ctypes
    import torch
    w = torch.zeros(4, 8)
    desc = lib.make_weights(w, None, None, w, None)
    good = [w.data_ptr(), 1, ctypes.addressof(desc), lib.CI_F32, lib.CI_ACT_RELU, w.data_ptr(), None, 0, None]
    wrong = {0: (None, 3), 1: (0, -1, 1 << 40), 2: (None,), 3: (7, -1), 4: (9, -1), 5: (None, w.data_ptr() + 2), 6: (None,), 7: (8,)}
    seen = set()
    for at, values in wrong.items():
        for v in values:
            args = good[:at] + [v] + good[at + 1:]
            c_args = list(args)
            c_args[2] = ctypes.cast(args[2], ctypes.POINTER(lib.ci_ffn_weights)) if args[2] else None
            status = lib._binding.ffn_decode(*args)
            assert status == lib.raw.coreinfer_ffn_decode(*c_args) != lib.CI_OK, (at, v)
            seen.add(status)
    assert len(seen) >= 3
    with pytest.raises(TypeError):
        lib._binding.ffn_decode(*good[:-1])
    with pytest.raises(TypeError):
        lib._binding.ffn_decode("x", *good[1:])
    with pytest.raises(OverflowError):
        lib._binding.ffn_decode(good[0], 1 << 70, *good[2:])
    with pytest.raises(TypeError):
        lib.ffn_decode(w, None, "relu", y=w, ws=w)


def test_nothing_in_the_library_throws(lib):
    """No exception crosses the C boundary: the library neither throws nor allocates, and takes no part of the C++ runtime that does
    (random_device throws where the system refuses it)."""
    import subprocess
    from paper_2410_18311_amd import build, isa_check
    out = subprocess.run([isa_check.OBJDUMP, "-T", build.LIB_PATH], check=True, capture_output=True, text=True).stdout
    wanted = [line.split()[-1] for line in out.splitlines() if "*UND*" in line]
    assert any(s.startswith("hip") for s in wanted), "no symbols were read"
    assert not [s for s in wanted if s.startswith(("__cxa_throw", "__cxa_rethrow", "_Znw", "_Zna")) or "random_device" in s]


def test_per_token_call_without_the_c_module(lib, monkeypatch, tmp_path):
    """The C module is for one interpreter and is left out where it cannot be compiled: the package then builds and imports as before,
    and the per-token call gives the same statuses through ctypes."""
    import importlib.util
    import sysconfig
    import torch
    from paper_2410_18311_amd import build
    assert build.BINDING_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    built = tmp_path / "_binding.so"
    built.write_bytes(b"of another library")
    monkeypatch.setattr(build, "BINDING_PATH", str(built))
    monkeypatch.setenv("CC", str(tmp_path / "no compiler"))
    assert build.build_binding() is False and not built.exists()
    spec = importlib.util.spec_from_file_location("paper_2410_18311_amd.coreinfer_without", lib.__file__)
    without = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(without)
    assert without._binding is None
    w = torch.zeros(4, 8)
    for args, kw in (((w, without.make_weights(w, None, None, w, None), "relu"), dict(y=w, ws=w)),
                     ((w, without.make_weights(w, None, None, None, None), "relu"), dict(y=w, ws=w.to(torch.uint8)))):
        mine = without.ci_ffn_weights.from_buffer_copy(args[1])
        theirs = lib.ci_ffn_weights.from_buffer_copy(args[1])
        with pytest.raises(without.CoreInferError) as a:
            without.ffn_decode(args[0], mine, args[2], **kw)
        with pytest.raises(lib.CoreInferError) as b:
            lib.ffn_decode(args[0], theirs, args[2], **kw)
        assert a.value.status == b.value.status != lib.CI_OK
