"""The dense GEMM kernels at the sizes where a tile, a remainder or a split of the reduction can go
wrong, against the oracle."""
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
        assert_close_rms(got.abs(), A_ref, dtype, "hidden values")
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
