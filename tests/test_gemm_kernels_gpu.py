"""The dense GEMM kernels at the sizes where a tile, a remainder or a split of the reduction can go
wrong, against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import coreinfer_oracle as orc
from tests._util import assert_close_rms, down_out_major64, f64, rand_weights, score_bound

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check_dense(lib, dtype, act, layout, M, d, N, hidden=False):
    print("dense kernel case", dtype, act, layout, M, d, N, "hidden" if hidden else "scores", flush=True)
    w = rand_weights(d, N, dtype, act, layout, seed=3 * M + d + N, device=DEV)
    X = torch.randn(M, d, generator=torch.Generator().manual_seed(M + 7)).to(dtype).to(DEV)
    args = (X, w["w_up"], w["w_gate"], w["b_up"], w["w_down"], w["b_down"], layout, act)
    if act == "relu":
        A_ref = orc.score_relu(f64(X), f64(w["w_up"]), f64(w["b_up"]))
        y_ref = orc.ffn_relu(f64(X), None, f64(w["w_up"]), f64(w["b_up"]), down_out_major64(w, layout), f64(w["b_down"]))
    else:
        A_ref = orc.score_swiglu(f64(X), f64(w["w_gate"]), f64(w["w_up"]))
        y_ref = orc.ffn_swiglu(f64(X), None, f64(w["w_gate"]), f64(w["w_up"]), down_out_major64(w, layout), f64(w["b_down"]))
    # guard words behind the outputs: a kernel that stores past its last row or column shows
    n = M * N
    S = torch.full((n + 64,), -7.0, dtype=dtype if hidden else torch.float32, device=DEV)
    Y = torch.full((M * d + 64,), -7.0, dtype=dtype, device=DEV)
    if hidden:
        lib.ffn_dense_hidden(*args, Y=Y[:M * d].view(M, d), H=S[:n].view(M, N))
    else:
        lib.ffn_dense(*args, want_y=True, want_a=True, Y=Y[:M * d].view(M, d), A=S[:n].view(M, N))
    torch.cuda.synchronize()
    assert bool((S[n:] == -7.0).all()) and bool((Y[M * d:] == -7.0).all()), "stored past the end"
    got = S[:n].view(M, N)
    if hidden:
        # one rounding of the fp32 value: half a unit in the last place, at most 2^-8 (bf16, 8 bits) or 2^-11
        # (fp16, 11 bits) of it and, for fp16, 2^-25 below its normal range, on top of the scores' own bound
        half_ulp = {torch.bfloat16: 2.0 ** -8, torch.float16: 2.0 ** -11}[dtype]
        bound = half_ulp * A_ref + 2.0 ** -25 + score_bound(dtype, act, A_ref, X, w)
        assert np.all(np.abs(np.abs(f64(got)) - A_ref) <= bound), "hidden values"
    else:
        assert np.max(np.abs(f64(got) - A_ref)) <= score_bound(dtype, act, A_ref, X, w), "scores"
    assert_close_rms(Y[:M * d].view(M, d), y_ref, dtype, "Y")


# 16 x 16 tiles with k split over 1 .. 16 waves (rows, columns and k that end inside a tile, a wave's
# range of zero groups), and the 128 x 128 tiles that take over from 128 of them on
@pytest.mark.parametrize("act,layout", [("relu", "out_major"), ("swiglu", "neuron_major")])
@pytest.mark.parametrize("M,d,N", [(5, 4, 4), (16, 16, 16), (17, 20, 36), (33, 260, 1028), (15, 1100, 68),
                                   (1025, 36, 1924), (2049, 1028, 68)])
def test_dense_f32_tiles(lib, act, layout, M, d, N):
    _check_dense(lib, torch.float32, act, layout, M, d, N)


# The LDS-tiled kernels for 16-bit types, tile shapes forced (0 .. 4: 128x128, 128x256, 256x192, 128x64, 256x256
# rows of A x rows of B), whole and with k split over 3 workgroups per tile: one row and column
# past a tile, k shorter than the ring, k that ends inside a 64-k tile, an odd number of k-tiles, several
# tiles per XCD.
TILE_CASES = [(5, 8, 8), (129, 264, 136), (257, 328, 520), (64, 1608, 776), (300, 1152, 1032)]


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("act,layout,dtype", [("relu", "out_major", torch.float16), ("swiglu", "out_major", torch.bfloat16),
                                              ("relu", "neuron_major", torch.bfloat16)])
@pytest.mark.parametrize("splits", [0, 3])
def test_dense_tile_shapes(lib, tile, act, layout, dtype, splits):
    lib.dev_set_param("gemm_tile", tile)
    lib.dev_set_param("gemm_splits", splits)
    try:
        for M, d, N in TILE_CASES:
            _check_dense(lib, dtype, act, layout, M, d, N)
            _check_dense(lib, dtype, act, layout, M, d, N, hidden=True)
    finally:
        lib.dev_set_param("gemm_tile", -1)
        lib.dev_set_param("gemm_splits", 0)


# 256 rows of A x 192, 256, 224 and 160 of B: blocks that two waves share by halves (224 and 160), one to four k-tiles and a bit (fewer than
# are loaded ahead), columns that end inside a tile and one tile further, a row past a tile
@pytest.mark.parametrize("tile,bn", [(2, 192), (4, 256), (5, 224), (6, 160)])
@pytest.mark.parametrize("act,layout,dtype", [("relu", "out_major", torch.bfloat16), ("swiglu", "out_major", torch.float16),
                                              ("relu", "neuron_major", torch.float16)])
def test_dense_wide_tiles(lib, tile, bn, act, layout, dtype):
    cols = bn // 2 if act == "swiglu" else bn
    try:
        lib.dev_set_param("gemm_tile", tile)
        for splits, M, d, N in [(1, 5, 64, 72), (1, 256, 72, cols), (1, 257, 128, cols + 8), (1, 130, 136, 2 * cols - 8),
                                (2, 300, bn, 520), (3, 257, bn + 8, 840), (1, 513, 192, 200)]:
            lib.dev_set_param("gemm_splits", splits)
            _check_dense(lib, dtype, act, layout, M, d, N, hidden=splits == 2)
    finally:
        lib.dev_set_param("gemm_tile", -1)
        lib.dev_set_param("gemm_splits", 0)


# The shapes for up projections, 192 x 128 and 128 x 96, 160 and 192 (7 .. 10; the down projection behind them falls back to 128 x 128):
# the same edges
@pytest.mark.parametrize("tile,bm,bn", [(7, 192, 128), (8, 128, 96), (9, 128, 160), (10, 128, 192)])
@pytest.mark.parametrize("act,layout,dtype", [("relu", "out_major", torch.bfloat16), ("swiglu", "out_major", torch.float16),
                                              ("relu", "neuron_major", torch.float16)])
def test_dense_mid_tiles(lib, tile, bm, bn, act, layout, dtype):
    cols = bn // 2 if act == "swiglu" else bn
    try:
        lib.dev_set_param("gemm_tile", tile)
        for splits, M, d, N in [(1, 5, 64, 72), (1, bm, 72, cols), (1, bm + 1, 128, cols + 8), (1, bm - 62, 136, 2 * cols - 8),
                                (2, 300, bn, 520), (3, bm + 1, bn + 8, 840), (1, 513, 448, 200)]:
            lib.dev_set_param("gemm_splits", splits)
            _check_dense(lib, dtype, act, layout, M, d, N, hidden=splits == 2)
    finally:
        lib.dev_set_param("gemm_tile", -1)
        lib.dev_set_param("gemm_splits", 0)


# What lies behind the end of k in memory, the start of the next row (of a k-major B: nothing), is loaded and takes no part,
# whatever it is; values that are not finite at the last k reach their own row or column
@pytest.mark.parametrize("tile", [2, 4, 5, 6, 7, 8, 9, 10])
@pytest.mark.parametrize("layout", ["out_major", "neuron_major"])
@pytest.mark.parametrize("splits", [1, 2])
def test_dense_wide_tiles_beside_values_that_are_not_finite(lib, tile, layout, splits):
    M, d, N, dt = 20, 520, 584, torch.float16    # 8 k-tiles and 8, 9 and 8
    g = torch.Generator().manual_seed(tile)
    pos = lambda *s: (torch.rand(*s, generator=g) * 0.02 + 0.001).to(dt).to(DEV)  # noqa: E731
    w_up, down, X = pos(N, d), pos(d, N), pos(M, d)
    X[4, 0], X[9, d - 1], w_up[7, 0], w_up[N - 1, d - 1] = float("inf"), float("inf"), float("inf"), float("inf")
    lib.dev_set_param("gemm_tile", tile)
    lib.dev_set_param("gemm_splits", splits)
    try:
        A = lib.ffn_dense(X, w_up, None, None, down if layout == "out_major" else down.t().contiguous(), None, layout, "relu",
                          want_y=False, want_a=True)[1]
        X, w_up = pos(M, d), pos(N, d)
        down[3, 0], down[d - 1, N - 1], down[11, N - 8] = float("nan"), float("inf"), float("nan")
        Y = lib.ffn_dense(X, w_up, None, None, down if layout == "out_major" else down.t().contiguous(), None, layout, "relu",
                          want_y=True, want_a=False)[0]
    finally:
        lib.dev_set_param("gemm_tile", -1)
        lib.dev_set_param("gemm_splits", 0)
    inf_A = torch.zeros(M, N, dtype=torch.bool, device=DEV)
    inf_A[4], inf_A[9], inf_A[:, 7], inf_A[:, N - 1] = True, True, True, True
    assert torch.equal(torch.isinf(A), inf_A) and not bool(torch.isnan(A).any())
    bad = torch.zeros(M, d, dtype=torch.bool, device=DEV)
    bad[:, 3], bad[:, 11], bad[:, d - 1] = True, True, True
    assert torch.equal(~torch.isfinite(Y), bad) and bool(torch.isinf(Y[:, d - 1]).all())


# Tiles of 16 tm x 16 tn (16 + 16 tm + tn), whole and with k split over 3 workgroups per tile: one row past a tile and one
# short of it, columns that end inside a tile, k of one k-tile (three waves without any), k that ends inside one, k that
# does not divide by the four waves.
@pytest.mark.parametrize("tm,tn", [(tm, tn) for tn in range(2, 9) for tm in range(1, 9) if (tm, tn) not in ((8, 4), (8, 7), (8, 8))])
@pytest.mark.parametrize("act,dtype", [("relu", torch.float16), ("swiglu", torch.bfloat16)])
def test_dense_slim_tiles(lib, tm, tn, act, dtype):
    try:
        lib.dev_set_param("gemm_tile", 16 + 16 * tm + tn)
        for splits in (1, 3):
            lib.dev_set_param("gemm_splits", splits)
            for M, d, N in [(max(5, 16 * tm - 3), 8, 24), (16 * tm + 1, 16 * tn + 8, 840), (16 * tm, 456, 16 * tn * 3)]:
                _check_dense(lib, dtype, act, "out_major", M, d, N, hidden=tm % 2 == 0)
    finally:
        lib.dev_set_param("gemm_tile", -1)
        lib.dev_set_param("gemm_splits", 0)


# Weights loaded as data that is not read again, in every tile shape that can: the bits of the ordinary loads (which the
# tests above hold to the oracle), whole and split, with k that ends inside a k-tile and more k-tiles than a ring holds
@pytest.mark.parametrize("tile", [0, 1, 2, 3] + [16 + 16 * tm + tn for tn in range(2, 9) for tm in range(1, 9)
                                                 if (tm, tn) not in ((8, 4), (8, 7), (8, 8))])
@pytest.mark.parametrize("act,dtype", [("relu", torch.float16), ("relu", torch.bfloat16), ("swiglu", torch.bfloat16)])
def test_dense_read_once_loads(lib, tile, act, dtype):
    M, d, N = 100, 776, 1736
    w = rand_weights(d, N, dtype, act, "out_major", seed=tile, device=DEV)
    X = torch.randn(M, d, generator=torch.Generator().manual_seed(tile)).to(dtype).to(DEV)
    args = (X, w["w_up"], w["w_gate"], w["b_up"], w["w_down"], w["b_down"], "out_major", act)
    lib.dev_set_param("gemm_tile", tile)
    try:
        for splits in (1, 3):
            lib.dev_set_param("gemm_splits", splits)
            out = {}
            for once in (0, 2):
                lib.dev_set_param("gemm_once", once)
                out[once] = lib.ffn_dense(*args, want_y=True, want_a=True)
            assert torch.equal(out[0][0], out[2][0]) and torch.equal(out[0][1], out[2][1])
    finally:
        lib.dev_set_param("gemm_tile", -1)
        lib.dev_set_param("gemm_splits", 0)
        lib.dev_set_param("gemm_once", 1)


# Short prompts over weights of more than 80 MB a product, where the rule takes those loads, and two that keep the ordinary
# ones: a layer that the memory-side cache holds, and rows of no multiple of 128 bytes
@pytest.mark.parametrize("act,dtype,M,d,N,once", [("swiglu", torch.bfloat16, 77, 4096, 11008, (1, 1)), ("relu", torch.float16, 16, 4096, 16384, (1, 1)),
                                                  ("relu", torch.bfloat16, 128, 5120, 13824, (1, 1)), ("swiglu", torch.float16, 31, 3072, 8192, (1, 0)),
                                                  ("swiglu", torch.float16, 33, 3072, 8192, (0, 0)), ("relu", torch.float16, 45, 4104, 12008, (0, 0))])
def test_dense_short_prompts_of_large_layers(lib, act, dtype, M, d, N, once):
    plan = lib.dev_dense_plan(M, d, N, dtype, act, "out_major")
    assert (plan["up_once"], plan["down_once"]) == once
    print("large layer case", act, dtype, M, d, N, lib.dev_dense_plan(M, d, N, dtype, act, "out_major"), flush=True)
    g = torch.Generator(device=DEV).manual_seed(M)
    mat = lambda *s: (torch.randn(*s, generator=g, device=DEV) * 0.02).to(dtype)  # noqa: E731
    up, gate, down = mat(N, d), mat(N, d) if act == "swiglu" else None, mat(d, N)
    X = torch.randn(M, d, generator=g, device=DEV).to(dtype)
    args = (X, up, gate, None, down, None, "out_major", act)
    Y, A = lib.ffn_dense(*args, want_y=True, want_a=True)
    _, H = lib.ffn_dense_hidden(*args)
    cols = torch.randperm(N, generator=torch.Generator().manual_seed(M))[:500].to(DEV)  # sampled neurons, in 64 bits
    z = X.double() @ up[cols].double().t()
    h = torch.nn.functional.silu(X.double() @ gate[cols].double().t()) * z if act == "swiglu" else z.clamp(min=0)
    A_ref = f64(h.abs())
    assert np.abs(f64(A[:, cols]) - A_ref).max() <= score_bound(dtype, act, A_ref), "A"
    assert_close_rms(Y, f64(H.double() @ down.double().t()), dtype, "Y")  # from the rounded hidden matrix itself
    lib.dev_set_param("gemm_once", 0)
    try:
        Y0, A0 = lib.ffn_dense(*args, want_y=True, want_a=True)
    finally:
        lib.dev_set_param("gemm_once", 1)
    assert torch.equal(Y, Y0) and torch.equal(A, A0)


# As planned: token counts on both sides of the slim tiles' range, with a workspace for sums and with the least there is
@pytest.mark.parametrize("M", [5, 16, 17, 64, 77, 128, 129, 256, 257])
@pytest.mark.parametrize("layout", ["out_major", "neuron_major"])
def test_dense_planned_few_rows(lib, M, layout):
    _check_dense(lib, torch.float16, "relu", layout, M, 1032, 3080)
    _check_dense(lib, torch.bfloat16, "swiglu", layout, M, 520, 1400, hidden=True)
    d, N = 1032, 3080
    w = rand_weights(d, N, torch.float16, "relu", layout, seed=M, device=DEV)
    X = torch.randn(M, d, generator=torch.Generator().manual_seed(M)).half().to(DEV)
    args = (X, w["w_up"], w["w_gate"], w["b_up"], w["w_down"], w["b_down"], layout, "relu")
    least = (M * N * 4 + 255) // 256 * 256 + 256
    assert lib.ffn_dense_workspace_size(M, d, N, torch.float16) >= least
    Y0, _ = lib.ffn_dense(*args)
    Y1, _ = lib.ffn_dense(*args, ws=torch.empty(least, dtype=torch.uint8, device=DEV))
    assert_close_rms(Y1, f64(Y0), torch.float16, "Y without room for sums")


@pytest.mark.parametrize("layout", ["out_major", "neuron_major"])
def test_dense_split_last_round_only(lib, layout):
    """A down projection of more than 256 tiles whose last round is split along k: 17 x 16 tiles of
    128x64, whole rounds and split tiles side by side, the last row of tiles ragged."""
    lib.dev_set_param("gemm_tile", 3)
    lib.dev_set_param("gemm_splits", 2)
    try:
        _check_dense(lib, torch.float16, "relu", layout, 2090, 1024, 648)
    finally:
        lib.dev_set_param("gemm_tile", -1)
        lib.dev_set_param("gemm_splits", 0)


# up to four tokens: groups of 4 (8) rows that end inside a group, rows shorter and longer than one pass of 256
# threads, columns that end inside a chunk of 64 vectors, pieces of the neurons that are empty or end inside a batch
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("act,layout", [("relu", "out_major"), ("swiglu", "out_major"), ("relu", "neuron_major"),
                                        ("swiglu", "neuron_major")])
@pytest.mark.parametrize("M", [1, 2, 3, 4])
def test_dense_few_tokens(lib, M, act, layout, dtype):
    for d, N in [(8, 8), (24, 40), (520, 1032), (2056, 2824), (4104, 264)]:
        _check_dense(lib, dtype, act, layout, M, d, N)


def test_dense_few_tokens_infinite_weight(lib):
    """Rows that are loaded again to fill a batch take no part: an infinite weight gives an infinity, not a NaN."""
    d, N, dt = 64, 8 * 19, torch.float16
    X = torch.ones(2, d, dtype=dt, device=DEV)
    w_up = torch.full((N, d), 0.01, dtype=dt, device=DEV)
    w_down = torch.full((N, d), 0.01, dtype=dt, device=DEV)
    w_down[N - 1, 3] = float("inf")
    Y = lib.ffn_dense(X, w_up, None, None, w_down, None, "neuron_major", "relu", want_y=True, want_a=True)[0]
    assert bool(torch.isinf(Y[:, 3]).all()) and int(torch.isfinite(Y).sum()) == 2 * (d - 1)


def _hidden_ws_size(lib, M, d, N):
    b = ctypes.c_size_t(0)
    assert lib.raw.coreinfer_ffn_dense_hidden_workspace_size(M, d, N, lib.CI_F16, ctypes.byref(b)) == lib.CI_OK
    return b.value


def _hidden_layer(M, d, N, dt):
    w = rand_weights(d, N, dt, "relu", "neuron_major", seed=M, device=DEV)
    X = torch.randn(M, d, generator=torch.Generator().manual_seed(d)).to(dt).to(DEV)
    y = orc.ffn_relu(f64(X), None, f64(w["w_up"]), f64(w["b_up"]), down_out_major64(w, "neuron_major"), f64(w["b_down"]))
    return w, X, y


# workspaces with room for all sums of split tiles, for some of a plan of fewer splits, and for none
@pytest.mark.parametrize("M,d,N", [(64, 1608, 1032), (300, 1152, 1032), (129, 264, 2056)])
def test_dense_hidden_takes_what_room_there_is(lib, M, d, N):
    w, X, y_ref = _hidden_layer(M, d, N, torch.float16)
    size = _hidden_ws_size(lib, M, d, N)
    for room in sorted({256, size // 2, size - 256, size, 4 * size}):
        print("dense room case", M, d, N, room, "of", size, flush=True)
        ws = torch.full((max(room, 256) + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
        Y, H = lib.ffn_dense_hidden(X, w["w_up"], None, w["b_up"], w["w_down"], w["b_down"], "neuron_major", "relu",
                                    ws=ws[:max(room, 256)])
        torch.cuda.synchronize()
        assert bool((ws[max(room, 256):] == 0xA5).all()), "stored past the workspace"
        assert_close_rms(Y, y_ref, torch.float16, f"room {room}")


def test_settings_that_change_during_a_call_stay_inside_its_workspace(lib):
    """A development setting may be changed by another thread at any time: the plan a call's workspace was checked
    for is the plan it runs."""
    import threading
    M, d, N = 64, 512, 2056
    w, X, y_ref = _hidden_layer(M, d, N, torch.float16)
    size = _hidden_ws_size(lib, M, d, N)
    ws = torch.full((size + (1 << 20),), 0xA5, dtype=torch.uint8, device=DEV)
    stop = threading.Event()

    def flip():
        i = 0
        while not stop.is_set():
            lib.dev_set_param("gemm_splits", i % 9)
            lib.dev_set_param("gemm_tile", i % 6 - 1)
            i += 1

    t = threading.Thread(target=flip)
    t.start()
    try:
        ys = [lib.ffn_dense_hidden(X, w["w_up"], None, w["b_up"], w["w_down"], w["b_down"], "neuron_major", "relu",
                                   ws=ws[:size])[0] for _ in range(200)]
        torch.cuda.synchronize()
    finally:
        stop.set()
        t.join()
        lib.dev_set_param("gemm_splits", 0)
        lib.dev_set_param("gemm_tile", -1)
    assert bool((ws[size:] == 0xA5).all()), "stored past the workspace"
    for y in ys:
        assert_close_rms(y, y_ref, torch.float16, "while settings change")


# up projections that the second estimate gives to 256 x 256 tiles: rows of no multiple of 64 bytes, last tiles of few
# rows and columns
@pytest.mark.parametrize("act,dtype,M,d,N", [("swiglu", torch.bfloat16, 2400, 1288, 4440), ("relu", torch.float16, 3166, 1832, 5616)])
def test_dense_odd_rows_wide_tiles(lib, act, dtype, M, d, N):
    _check_dense(lib, dtype, act, "out_major", M, d, N)


# Sizes whose up projection has two tile shapes of nearly the same estimated time, up to 128 tokens and above: scores, hidden
# values and outputs are the same bits whichever of them a call asks for.
@pytest.mark.parametrize("act,dtype,M,d,N", [("swiglu", torch.bfloat16, 13, 496, 2624), ("relu", torch.float16, 53, 1000, 2224),
                                             ("relu", torch.bfloat16, 21, 568, 2816), ("swiglu", torch.float16, 21, 560, 2048),
                                             ("relu", torch.float16, 57, 6856, 18768),
                                             # and a plan of 256-row tiles
                                             ("swiglu", torch.float16, 1000, 1160, 8192)])
def test_outputs_asked_for_change_no_bits(lib, act, dtype, M, d, N):
    w = rand_weights(d, N, dtype, act, "out_major", seed=M, device=DEV)
    X = torch.randn(M, d, generator=torch.Generator().manual_seed(M)).to(dtype).to(DEV)
    args = (X, w["w_up"], w["w_gate"], w["b_up"], w["w_down"], w["b_down"], "out_major", act)
    Y, A = lib.ffn_dense(*args, want_y=True, want_a=True)
    _, A_only = lib.ffn_dense(*args, want_y=False, want_a=True)
    Y_only, _ = lib.ffn_dense(*args, want_y=True, want_a=False)
    Y_hidden, H = lib.ffn_dense_hidden(*args)
    assert torch.equal(A_only, A)
    assert torch.equal(Y_only, Y) and torch.equal(Y_hidden, Y)
    assert torch.equal(H.abs(), A.to(dtype))   # one rounding of the same fp32 values


# Slim tiles, as planned, for both projections (the second with k split)
SLIM = [("swiglu", torch.bfloat16, 15, 1280, 4864), ("relu", torch.float16, 32, 2512, 9888)]


def _slim_call(lib, act, dtype, M, d, N):
    plan = lib.dev_dense_plan(M, d, N, dtype, act, "out_major")
    assert plan["up"] >= 32 and plan["down"] >= 32 and plan["splits"] > 1, plan
    w = rand_weights(d, N, dtype, act, "out_major", seed=M, device=DEV)
    X = torch.randn(M, d, generator=torch.Generator().manual_seed(d)).to(dtype).to(DEV)
    ws = torch.empty(lib.ffn_dense_workspace_size(M, d, N, dtype), dtype=torch.uint8, device=DEV)
    Y, A = torch.empty(M, d, dtype=dtype, device=DEV), torch.empty(M, N, device=DEV)

    def call():
        lib.ffn_dense(X, w["w_up"], w["w_gate"], w["b_up"], w["w_down"], w["b_down"], "out_major", act, want_y=True, want_a=True,
                      Y=Y, A=A, ws=ws)
    return X, Y, A, ws, call


@pytest.mark.parametrize("act,dtype,M,d,N", SLIM)
def test_dense_planned_slim(lib, act, dtype, M, d, N):
    _check_dense(lib, dtype, act, "out_major", M, d, N)
    _check_dense(lib, dtype, act, "out_major", M, d, N, hidden=True)


@pytest.mark.parametrize("act,dtype,M,d,N", SLIM)
def test_dense_slim_on_another_stream_and_captured(lib, act, dtype, M, d, N):
    X, Y, A, ws, call = _slim_call(lib, act, dtype, M, d, N)
    call()
    torch.cuda.synchronize()
    first = Y.clone(), A.clone()
    for _ in range(4):   # the same bits whatever the workspace held
        ws.fill_(255)
        call()
        assert torch.equal(Y, first[0]) and torch.equal(A, first[1])
    side = torch.cuda.Stream()
    Y.zero_(), A.zero_(), ws.fill_(255)
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    assert torch.equal(Y, first[0]) and torch.equal(A, first[1])
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for i in range(4):
        X.copy_(torch.randn(M, d, generator=torch.Generator().manual_seed(100 + i)))
        Y.zero_(), A.zero_(), ws.fill_(255)
        g.replay()
        torch.cuda.synchronize()
        replayed = Y.clone(), A.clone()
        call()
        assert torch.equal(replayed[0], Y) and torch.equal(replayed[1], A)


# Infinities and NaN at the last k and at the first of the last, ragged k-tile, which is what chunks past the end are
# loaded from: they reach the rows (or columns) that have them and no others, as sums without those chunks give
@pytest.mark.parametrize("tile", [0, 3, 34, 51, 86, 120])
@pytest.mark.parametrize("splits", [1, 2])
def test_dense_values_that_are_not_finite_in_a_ragged_k_tile(lib, tile, splits):
    M, d, N, dt = 20, 1032, 1096, torch.float16    # 16 k-tiles and 8, 17 and 8
    g = torch.Generator().manual_seed(tile)
    pos = lambda *s: (torch.rand(*s, generator=g) * 0.02 + 0.001).to(dt).to(DEV)  # noqa: E731
    w_up, w_down, X = pos(N, d), pos(d, N), pos(M, d)
    X[3, d - 1], X[5, d - 8], X[7, d - 8] = float("inf"), float("inf"), float("nan")
    w_up[N - 1, d - 1] = float("inf")
    lib.dev_set_param("gemm_tile", tile)
    lib.dev_set_param("gemm_splits", splits)
    try:
        Y, A = lib.ffn_dense(X, w_up, None, None, w_down, None, "out_major", "relu", want_y=True, want_a=True)
        X[3, d - 1], X[5, d - 8], X[7, d - 8], w_up[N - 1, d - 1] = 0.5, 0.5, 0.5, 0.01
        w_down[2, N - 1], w_down[4, N - 8] = float("inf"), float("nan")
        Y2, A2 = lib.ffn_dense(X, w_up, None, None, w_down, None, "out_major", "relu", want_y=True, want_a=True)
    finally:
        lib.dev_set_param("gemm_tile", -1)
        lib.dev_set_param("gemm_splits", 0)
    inf_A = torch.zeros(M, N, dtype=torch.bool, device=DEV)
    inf_A[3], inf_A[5], inf_A[:, N - 1] = True, True, True
    inf_A[7] = False                      # max(NaN, 0) is 0
    assert torch.equal(torch.isinf(A), inf_A)
    assert bool((A[7] == 0).all()) and not bool(torch.isnan(A).any())
    inf_Y = torch.ones(M, d, dtype=torch.bool, device=DEV)
    inf_Y[7] = False
    assert torch.equal(torch.isinf(Y), inf_Y) and bool((Y[7] == 0).all())
    assert bool(torch.isfinite(A2).all())
    assert bool(torch.isinf(Y2[:, 2]).all()) and bool(torch.isnan(Y2[:, 4]).all())
    rest = [c for c in range(d) if c not in (2, 4)]
    assert bool(torch.isfinite(Y2[:, rest]).all())


# What an output's conversion to 16 bits does with ties, the largest and smallest numbers, infinities and NaN, in the kernels for few tokens,
# in slim, middle and wide tiles: hidden values of one and two weights a column, so that the fp32 sum is exact.
@pytest.mark.parametrize("M", [1, 16, 200, 1100])
@pytest.mark.parametrize("layout", ["out_major", "neuron_major"])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_dense_outputs_are_rounded_to_nearest_even(lib, M, layout, dtype):
    d, N = 512, 64
    g = torch.Generator().manual_seed(M)
    fi = torch.finfo(dtype)
    a = torch.randn(d, generator=g).to(dtype)
    b = (a.float() * torch.tensor([0.5, -0.5, 0.25, 1.0])[torch.randint(4, (d,), generator=g)] * fi.eps).to(dtype)   # halfway, and beside it
    a[:8] = torch.tensor([fi.max, -fi.max, float("inf"), -float("inf"), float("nan"), 0.0, fi.tiny, -fi.tiny], dtype=dtype)
    b[:8] = torch.tensor([fi.max * fi.eps / 4, -fi.max * fi.eps / 4, 1.0, 1.0, 1.0, -0.0, fi.tiny / 2, fi.tiny / 2], dtype=dtype)
    down = torch.zeros(d, N, dtype=dtype)
    down[:, 0], down[:, 1] = a, b
    X = torch.zeros(M, d, dtype=dtype, device=DEV)
    w_up, b_up = torch.zeros(N, d, dtype=dtype, device=DEV), torch.ones(N, dtype=dtype, device=DEV)
    w_down = (down if layout == "out_major" else down.t()).contiguous().to(DEV)
    Y, _ = lib.ffn_dense(X, w_up, None, b_up, w_down, None, layout, "relu", want_y=True, want_a=True)
    want = (a.float() + b.float()).to(dtype).expand(M, d)
    got = Y.cpu()
    assert torch.equal(got.isnan(), want.isnan())
    assert torch.equal(got[~got.isnan()], want[~want.isnan()])
