"""The one-launch decode of small layers (every workgroup computes all hidden values, or a part of them that the others read): against the oracle, the same bits as
the two launches in every form of the call, and which of the two a call takes."""
import pytest
import torch

from oracle import coreinfer_oracle as orc
from tests._util import assert_close_rms, f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _layer(dt, act, d, K, seed):
    g = torch.Generator().manual_seed(seed)
    mat = lambda *s: (torch.randn(*s, generator=g) * 0.05).to(dt).to(DEV)  # noqa: E731
    return dict(up=mat(K, d), gate=mat(K, d) if act == "swiglu" else None, b_up=mat(K) if act == "relu" else None,
                down=mat(K, d), b_down=mat(d))


def _reference(w, act, x):
    down = f64(w["down"]).T
    if act == "relu":
        return orc.ffn_relu(f64(x), None, f64(w["up"]), f64(w["b_up"]), down, f64(w["b_down"]))
    return orc.ffn_swiglu(f64(x), None, f64(w["gate"]), f64(w["up"]), down, f64(w["b_down"]))


# rows of one vector, of the lanes of a quarter, half and whole wave, one vector more than each, and of two loads; one
# neuron, one short of and one past a batch of rows, more than the down rows a thread holds (512), the most there can be
@pytest.mark.parametrize("act", ["relu", "swiglu"])
@pytest.mark.parametrize("dt", [torch.float32, torch.float16, torch.bfloat16])
def test_small_decode_shapes(lib, act, dt):
    vec = 4 if dt == torch.float32 else 8
    lib.dev_set_param("decode_small", 2)
    try:
        for vecs in (1, 15, 16, 17, 32, 33, 64, 65, 128):
            d = vecs * vec
            for K, B in ((1, 1), (63, 2), (65, 1), (257, 4), (513, 1), (4096, 1)):
                print("small decode case", dt, act, d, K, B, flush=True)
                w = _layer(dt, act, d, K, d + K)
                x = torch.randn(B, d, generator=torch.Generator().manual_seed(K)).to(dt).to(DEV)
                y = torch.full((B * d + 64,), -7.0, dtype=dt, device=DEV)
                desc = lib.make_weights(w["up"], w["gate"], w["b_up"], w["down"], w["b_down"])
                # a workspace of anything: this path uses none
                ws = torch.full((lib.ffn_decode_workspace_size(B, K, d),), 255, dtype=torch.uint8, device=DEV)
                lib.ffn_decode(x, desc, act, y=y[:B * d].view(B, d), ws=ws)
                torch.cuda.synchronize()
                assert bool((y[B * d:] == -7.0).all()), "stored past the end"
                assert bool((ws == 255).all()), "two launches"
                lib.dev_set_param("decode_small", 0)
                two = lib.ffn_decode(x, desc, act)
                lib.dev_set_param("decode_small", 2)
                assert torch.equal(y[:B * d].view(B, d), two), "other bits than two launches"
                assert_close_rms(y[:B * d].view(B, d), _reference(w, act, x), dt, "y")
    finally:
        lib.dev_set_param("decode_small", 1)


def _one_launch(lib, x, desc, act, y=None):
    """The output of a call and whether it took one launch: two leave partial sums in the workspace."""
    ws = torch.full((lib.ffn_decode_workspace_size(x.shape[0], desc.K, x.shape[1]),), 255, dtype=torch.uint8, device=DEV)
    y = lib.ffn_decode(x, desc, act, y=y, ws=ws)
    return y, bool((ws == 255).all())


# both sides of the rule's lines, with the setting that every program has: elements, vectors of a row, neurons, tokens
@pytest.mark.parametrize("d,K,B,one", [(256, 512, 1, True), (256, 513, 1, False), (512, 256, 4, True), (512, 256, 5, False),
                                       (516, 8, 1, False), (4, 2048, 1, True), (4, 2049, 1, False), (8, 4097, 1, False)])
def test_small_decode_rule(lib, d, K, B, one):
    w = _layer(torch.float32, "relu", d, K, d + K)
    x = torch.randn(B, d, generator=torch.Generator().manual_seed(1)).to(DEV)
    desc = lib.make_weights(w["up"], None, w["b_up"], w["down"], w["b_down"])
    got, took_one = _one_launch(lib, x, desc, "relu")
    assert took_one == one
    assert_close_rms(got, _reference(w, "relu", x), torch.float32, "y")
    static = lib.ffn_decode_static(x, desc, "relu")
    assert torch.equal(static, got)
    # inputs that are not finite reach the output as they do through two launches
    x[0, 0] = float("inf")
    lib.dev_set_param("decode_small", 0)
    try:
        two = lib.ffn_decode(x, desc, "relu")
    finally:
        lib.dev_set_param("decode_small", 1)
    one = lib.ffn_decode(x, desc, "relu")
    assert torch.equal(torch.isnan(one), torch.isnan(two)) and torch.equal(torch.isinf(one), torch.isinf(two))


# layers on both sides of the line for captured calls (64 K elements): the same bits as launched, whichever way either goes
@pytest.mark.parametrize("act,d,K,one", [("swiglu", 128, 256, True), ("swiglu", 128, 300, False), ("relu", 256, 256, True),
                                         ("relu", 256, 257, False)])
def test_small_decode_graph(lib, act, d, K, one):
    w = _layer(torch.float32, act, d, K, 9)
    desc = lib.make_weights(w["up"], w["gate"], w["b_up"], w["down"], w["b_down"])
    x, y = torch.zeros(1, d, device=DEV), torch.empty(1, d, device=DEV)
    ws = lib.decode_workspace(1, K, d, DEV)
    lib.ffn_decode(x, desc, act, y=y, ws=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        lib.ffn_decode(x, desc, act, y=y, ws=ws)
    for i in range(4):
        x.copy_(torch.randn(1, d, generator=torch.Generator().manual_seed(i)))
        ws.fill_(255)
        g.replay()
        torch.cuda.synchronize()
        assert bool((ws == 255).all()) == one
        got, took_one = _one_launch(lib, x, desc, act)
        assert took_one
        assert torch.equal(y, got)


# y over x, whole or in part: two launches, and where they do not lie over one another the same bits from one
@pytest.mark.parametrize("shift", [0, 1, -1, 4, -4])
def test_small_decode_in_place(lib, shift):
    d, K, B = 256, 200, 4
    w = _layer(torch.float32, "relu", d, K, 5)
    desc = lib.make_weights(w["up"], None, w["b_up"], w["down"], w["b_down"])
    x = torch.randn(B, d, generator=torch.Generator().manual_seed(2)).to(DEV)
    apart, took_one = _one_launch(lib, x, desc, "relu")
    assert took_one
    buf = torch.zeros(9 * B * d, device=DEV)
    buf[4 * B * d:5 * B * d].view(B, d).copy_(x)
    o = (4 * B + shift) * d
    got, took_one = _one_launch(lib, buf[4 * B * d:5 * B * d].view(B, d), desc, "relu", y=buf[o:o + B * d].view(B, d))
    assert took_one == (abs(shift) == B)
    assert torch.equal(got, apart)


# Hidden values shared by the workgroups: the bits of two launches, for fewer and more neurons than workgroups and than a thread takes at
# once, one to four tokens; and again without a look at the others' values, when every workgroup computes what it misses itself
@pytest.mark.parametrize("patience", [2000, 0])
@pytest.mark.parametrize("act", ["relu", "swiglu"])
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_small_decode_shared(lib, act, dt, patience):
    vec = 4 if dt == torch.float32 else 8
    calls, alone, gave_up = 20, 0, lib.dev_decode_small_gave_up()   # more calls than rows of words
    lib.dev_set_param("decode_small_patience", patience)
    try:
        for vecs in (1, 16, 33, 64, 128):
            d = vecs * vec
            for K, B in ((1, 4), (9, 1), (257, 3), (513, 1), (2049, 2), (4096, 1)):
                w = _layer(dt, act, d, K, d + K)
                desc = lib.make_weights(w["up"], w["gate"], w["b_up"], w["down"], w["b_down"])
                x = torch.randn(B, d, generator=torch.Generator().manual_seed(K)).to(dt).to(DEV)
                x[0, 0] = float("inf") if K == 9 else x[0, 0]
                lib.dev_set_param("decode_small", 0)
                two = lib.ffn_decode(x, desc, act)
                lib.dev_set_param("decode_small", 3)
                assert lib.dev_decode_small(B, K, d, dt, act) == "shared"
                y = torch.full((B * d + 64,), -7.0, dtype=dt, device=DEV)
                ws = torch.full((lib.ffn_decode_workspace_size(B, K, d),), 255, dtype=torch.uint8, device=DEV)
                for _ in range(calls):
                    y[:B * d] = 0
                    lib.ffn_decode(x, desc, act, y=y[:B * d].view(B, d), ws=ws)
                    assert torch.equal(y[:B * d].view(B, d).nan_to_num(nan=3.0), two.nan_to_num(nan=3.0)), (d, K, B)
                assert bool((y[B * d:] == -7.0).all()), "stored past the end"
                assert bool((ws == 255).all()), "two launches"
                n = -(-vecs // 4)   # workgroups of a token, each of an equal part of the neurons
                alone += calls * B * sum(K * (i + 1) // n - K * i // n < K for i in range(n))
    finally:
        lib.dev_set_param("decode_small", 1)
        lib.dev_set_param("decode_small_patience", 2000)
    gave_up = lib.dev_decode_small_gave_up() - gave_up
    assert gave_up == alone if patience == 0 else gave_up < alone // 2, (gave_up, alone)


# Which way a call takes, with the setting that every program has: both sides of the lines for elements (64 K and 128 K), for batches of
# rows that sharing saves (three) and for workgroups (three), and of a captured stream, whose calls are two launches above 64 K elements
@pytest.mark.parametrize("act,dt,d,K,B,way", [("relu", torch.float32, 256, 256, 1, "all"), ("relu", torch.float32, 256, 257, 1, "shared"),
                                              ("relu", torch.float32, 512, 192, 4, "all"), ("relu", torch.float32, 512, 193, 4, "shared"),
                                              ("relu", torch.float32, 256, 512, 1, "shared"), ("relu", torch.float32, 256, 513, 1, "two launches"),
                                              ("swiglu", torch.float32, 256, 192, 1, "all"), ("swiglu", torch.float32, 256, 193, 1, "shared"),
                                              ("relu", torch.float16, 512, 192, 1, "all"), ("relu", torch.bfloat16, 512, 193, 1, "shared"),
                                              ("relu", torch.float32, 512, 225, 5, "two launches"),
                                              ("relu", torch.float32, 16, 2048, 1, "all"), ("relu", torch.float32, 32, 2048, 4, "all"),
                                              ("relu", torch.float32, 36, 1025, 1, "shared"), ("swiglu", torch.float32, 36, 1024, 1, "all"),
                                              ("relu", torch.float16, 104, 1024, 1, "shared"), ("relu", torch.bfloat16, 96, 1024, 1, "all")])
def test_small_decode_ways(lib, act, dt, d, K, B, way):
    assert lib.dev_decode_small(B, K, d, dt, act) == way
    w = _layer(dt, act, d, K, d + K)
    desc = lib.make_weights(w["up"], w["gate"], w["b_up"], w["down"], w["b_down"])
    x = torch.randn(B, d, generator=torch.Generator().manual_seed(1)).to(dt).to(DEV)
    got, took_one = _one_launch(lib, x, desc, act)
    assert took_one == (way != "two launches")
    assert_close_rms(got, _reference(w, act, x), dt, "y")
    y, ws = torch.empty_like(x), lib.decode_workspace(B, K, d, DEV)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        captured = lib.dev_decode_small(B, K, d, dt, act, torch.cuda.current_stream().cuda_stream)
        lib.ffn_decode(x, desc, act, y=y, ws=ws)
    vec = 4 if dt == torch.float32 else 8
    held = max(16 * vec, 1 << (d - 1).bit_length())   # what the lanes of a row's loads hold
    elements = (2 if act == "swiglu" else 1) * K * held
    assert captured == ("all" if way == "all" and elements <= 65536 else "two launches")
    for _ in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, got)


# Calls of several threads, each on a stream of its own, take the same rows of words in turn
def test_small_decode_shared_by_threads(lib):
    import threading
    d, K = 256, 500
    w = _layer(torch.float32, "relu", d, K, 3)
    desc = lib.make_weights(w["up"], None, w["b_up"], w["down"], w["b_down"])
    xs = torch.randn(6, d, generator=torch.Generator().manual_seed(4)).to(DEV)
    lib.dev_set_param("decode_small", 0)
    want = torch.cat([lib.ffn_decode(xs[i:i + 1], desc, "relu") for i in range(6)])
    lib.dev_set_param("decode_small", 1)
    torch.cuda.synchronize()
    assert lib.dev_decode_small(1, K, d, torch.float32, "relu") == "shared"
    wrong = [None] * 6

    def run(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            ws, y, n = lib.decode_workspace(1, K, d, DEV), torch.empty(1, d, device=DEV), torch.zeros((), dtype=torch.int64, device=DEV)
            for _ in range(200):
                assert lib.dev_decode_small(1, K, d, torch.float32, "relu", s.cuda_stream) == "shared"
                lib.ffn_decode(xs[i:i + 1], desc, "relu", y=y, ws=ws)
                n += (y != want[i:i + 1]).sum()
            s.synchronize()
            wrong[i] = int(n)

    threads = [threading.Thread(target=run, args=(i,)) for i in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert wrong == [0] * 6
