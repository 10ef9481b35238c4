"""Gathered decode of several sentences through the union of their lists: forced at small sizes,
against the oracle and against the kernel that reads every list's rows separately."""
import numpy as np
import pytest
import torch

from oracle import coreinfer_oracle as orc
from tests._util import assert_close_rms, down_out_major64, f64, rand_weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _reference(act, x, S, w):
    Wd = down_out_major64(w, "neuron_major")
    if act == "relu":
        return orc.ffn_relu(f64(x), S, f64(w["w_up"]), f64(w["b_up"]), Wd, f64(w["b_down"]))
    return orc.ffn_swiglu(f64(x), S, f64(w["w_gate"]), f64(w["w_up"]), Wd, f64(w["b_down"]))


# widths around the 64-vector column chunks of the down phase and (16384 fp32 elements = 4096 vectors) rows of
# more than one column chunk in the up phase; row counts around the blocks of 1024 neurons: eight of them, which a
# block counts itself, 8193 neurons, the first that a launch counts ahead, and 65 blocks; slices of fewer rows than 32
@pytest.mark.parametrize("dt,act", [(torch.float16, "relu"), (torch.bfloat16, "swiglu"), (torch.float32, "relu")])
@pytest.mark.parametrize("d,N,K,B", [(512, 2000, 801, 4), (520, 1024, 300, 8), (1016, 1025, 1025, 2), (8, 700, 699, 3),
                                     (64, 8192, 5000, 3), (64, 8193, 5000, 8), (24, 40, 9, 2),
                                     (64, 66000, 30000, 2), (16384, 400, 200, 2)])
def test_gathered_through_the_union(lib, dt, act, d, N, K, B):
    print("gathered union case", dt, act, d, N, K, B, flush=True)
    if d == 16384 and dt != torch.float32:
        pytest.skip("two column chunks need rows of more than 2048 vectors: fp32 only")
    w = rand_weights(d, N, dt, act, "neuron_major", seed=d + N + B, device=DEV)
    rng = np.random.default_rng(K + B)
    sets = np.stack([rng.permutation(N)[:K] for _ in range(B)]).astype(np.int32)   # in no order
    if N - 1 not in sets[B - 1]:
        sets[B - 1, 0] = N - 1      # the last neuron of the last block
    idx = torch.from_numpy(sets).to(DEV)
    x = torch.randn(B, d, generator=torch.Generator().manual_seed(N)).to(dt).to(DEV)
    desc = lib.make_weights(w["w_up"], w["w_gate"], w["b_up"], w["w_down"], w["b_down"], core_idx=idx)
    ys = []
    for mode in (0, 2):
        lib.dev_set_param("gathered_union", mode)
        try:
            ys.append(lib.ffn_decode(x, desc, act))
            if mode == 2:
                y_st = lib.ffn_decode_static(x, desc, act)
            torch.cuda.synchronize()
        finally:
            lib.dev_set_param("gathered_union", 1)
    assert torch.equal(ys[1], y_st), "the library's own scratch gives other results"
    rows = range(B) if N < 10000 else [0]
    for b in rows:
        ref = _reference(act, x[b], np.sort(sets[b]).astype(np.int64), w)
        assert_close_rms(ys[0][b], ref, dt, f"separate rows, sentence {b}")
        assert_close_rms(ys[1][b], ref, dt, f"union, sentence {b}")
    # the same sums in another order, rounded once to the element type
    rms = float(ys[0].float().pow(2).mean().sqrt())
    assert float((ys[1].float() - ys[0].float()).abs().max()) <= {torch.float32: 1e-5, torch.float16: 1e-2,
                                                                    torch.bfloat16: 5e-2}[dt] * rms


def test_repeated_and_invalid_entries_count_as_before(lib):
    """A neuron named r times by a list contributes r times, an entry outside [0, N) nothing -- also when
    another sentence names the same neuron once."""
    d, N, K, B = 256, 3000, 900, 3
    w = rand_weights(d, N, torch.float32, "relu", "neuron_major", seed=5, device=DEV)
    rng = np.random.default_rng(3)
    sets = np.stack([np.sort(rng.choice(N, size=K, replace=False)) for _ in range(B)]).astype(np.int32)
    sets[0, 10:310] = sets[0, 9]          # 301 times the same neuron
    sets[1, [0, 5, 899]] = [-1, N, 2 ** 30]
    sets[2, :9] = sets[0, 9]
    idx = torch.from_numpy(sets).to(DEV)
    x = torch.randn(B, d, generator=torch.Generator().manual_seed(1)).to(DEV)
    desc = lib.make_weights(w["w_up"], None, w["b_up"], w["w_down"], w["b_down"], core_idx=idx)
    out = []
    for mode in (0, 2):
        lib.dev_set_param("gathered_union", mode)
        try:
            out.append(f64(lib.ffn_decode(x, desc, "relu")))
        finally:
            lib.dev_set_param("gathered_union", 1)
    Wu, Wd = f64(w["w_up"]), f64(w["w_down"])
    for b in range(B):
        S = sets[b][(sets[b] >= 0) & (sets[b] < N)]
        ref = np.maximum(f64(x[b]) @ Wu[S].T + f64(w["b_up"])[S], 0.0) @ Wd[S] + f64(w["b_down"])
        rms = np.sqrt(np.mean(ref ** 2))
        for y in out:
            assert np.max(np.abs(y[b] - ref)) <= 1e-5 * rms


@pytest.mark.parametrize("knob,values", [("union_down_wgs_per_cu", (1, 16)), ("gathered_union", (0, 2)), ("decode_wgs", (16, 1024))])
def test_settings_that_change_during_a_call_stay_inside_its_scratch(lib, knob, values):
    """A development setting may be changed by another thread at any time: the slices that a call's scratch was laid
    out or checked for are the slices it runs.  (The library's own scratch turns a call down where they do not fit.)"""
    import threading
    d, N, K, B, dt = 4096, 12000, 6000, 4, torch.float16
    w = rand_weights(d, N, dt, "relu", "neuron_major", seed=9, device=DEV)
    rng = np.random.default_rng(4)
    sets = np.stack([np.sort(rng.permutation(N)[:K]) for _ in range(B)]).astype(np.int32)
    x = torch.randn(B, d, generator=torch.Generator().manual_seed(2)).to(dt).to(DEV)
    idx = torch.from_numpy(sets).to(DEV)     # a descriptor holds addresses only
    desc = lib.make_weights(w["w_up"], None, w["b_up"], w["w_down"], w["b_down"], core_idx=idx)
    size = lib.ffn_decode_workspace_size(B, K, d)
    ws = torch.full((size + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    stop = threading.Event()

    def flip():
        i = 0
        while not stop.is_set():
            lib.dev_set_param(knob, values[i % 2])
            i += 1

    lib.dev_set_param("gathered_union", 0 if knob == "decode_wgs" else 2)
    t = threading.Thread(target=flip)
    t.start()
    ys, refused = [], 0
    try:
        for _ in range(60):
            ys.append(lib.ffn_decode(x, desc, "relu", ws=ws[:size]))
            try:
                ys.append(lib.ffn_decode_static(x, desc, "relu"))
            except lib.CoreInferError as e:
                assert e.status == lib.CI_ERR_WORKSPACE
                refused += 1
        torch.cuda.synchronize()
    finally:
        stop.set()
        t.join()
        for name, default in (("union_down_wgs_per_cu", 1), ("gathered_union", 1), ("decode_wgs", 0)):
            lib.dev_set_param(name, default)
    assert bool((ws[size:] == 0xA5).all()), "stored past the workspace"
    assert refused == 0 or knob == "decode_wgs"
    refs = [_reference("relu", x[b], sets[b].astype(np.int64), w) for b in range(B)]
    for y in ys:
        for b in range(B):
            assert_close_rms(y[b], refs[b], dt, f"sentence {b}")


@pytest.mark.parametrize("dt,act", [(torch.float16, "relu"), (torch.bfloat16, "swiglu")])
def test_gathered_union_graph_replays_match_eager(lib, dt, act):
    """A decode step of several sentences captured once and replayed on other inputs and other core sets (same
    buffers), with eager work and synchronisations in between: every replay against the eager call."""
    d, N, K, B, L = 512, 9000, 3000, 4, 2
    ws_layers = [rand_weights(d, N, dt, act, "neuron_major", seed=70 + l, device=DEV) for l in range(L)]
    idx = torch.zeros(L, B, K, dtype=torch.int32, device=DEV)
    x = torch.zeros(L, B, d, dtype=dt, device=DEV)
    y = torch.zeros_like(x)
    ws = torch.full((lib.ffn_decode_workspace_size(B, K, d),), 0xA5, dtype=torch.uint8, device=DEV)
    descs = [lib.make_weights(w["w_up"], w["w_gate"], w["b_up"], w["w_down"], w["b_down"], core_idx=idx[l])
             for l, w in enumerate(ws_layers)]

    def step(out):
        for l in range(L):
            lib.ffn_decode(x[l], descs[l], act, y=out[l], ws=ws)

    rng = np.random.default_rng(12)

    def refill(i):
        sets = np.stack([[np.sort(rng.permutation(N)[:K]) for _ in range(B)] for _ in range(L)]).astype(np.int32)
        if i == 2:
            sets[:, 1, 5:205] = sets[:, 1, 5:6]      # a neuron named 200 times, in this replay only
        idx.copy_(torch.from_numpy(sets))
        x.copy_(torch.randn(L, B, d, generator=torch.Generator().manual_seed(i)).to(dt))

    lib.dev_set_param("gathered_union", 2)
    try:
        refill(0)
        step(y)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            step(y)
        for i in range(5):
            refill(i)
            y.fill_(-7.0)
            g.replay()
            torch.cuda.synchronize()
            eager = torch.empty_like(y)
            (torch.randn(256, 256, device=DEV) @ torch.randn(256, 256, device=DEV)).sum().item()
            step(eager)
            torch.cuda.synchronize()
            assert torch.equal(eager, y), f"replay {i}"
    finally:
        lib.dev_set_param("gathered_union", 1)
    if act == "relu":
        S = idx[0, 0].cpu().numpy().astype(np.int64)
        assert_close_rms(y[0, 0], _reference(act, x[0, 0], S, ws_layers[0]), dt, "last replay")
