"""Two-launch decode of many sentences: slice counts that are not a multiple of eight, one workgroup per compute
unit and fewer, narrow and wide rows, compacted and gathered, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import coreinfer_oracle as orc
from tests._util import assert_close_rms, down_out_major64, f64, rand_weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("d,dt", [(512, torch.float16), (3072, torch.bfloat16), (2048, torch.float32)])
@pytest.mark.parametrize("B", [3, 11, 18, 33, 257])
@pytest.mark.parametrize("gathered", [False, True])
def test_decode_of_many_sentences(lib, d, dt, B, gathered):
    N, K = 900, 301
    print("decode slices case", d, dt, B, gathered, "slices", lib.dev_decode_slices(B, K, d, dt, gathered), flush=True)
    w = rand_weights(d, N, dt, "relu", "neuron_major", seed=d + B, device=DEV)
    rng = np.random.default_rng(B)
    x = torch.randn(B, d, generator=torch.Generator().manual_seed(B)).to(dt).to(DEV)
    if gathered:
        sets = np.stack([np.sort(rng.permutation(N)[:K]) for _ in range(B)]).astype(np.int32)
        idx = torch.from_numpy(sets).to(DEV)     # a descriptor holds addresses only
        desc = lib.make_weights(w["w_up"], None, w["b_up"], w["w_down"], w["b_down"], core_idx=idx)
    else:
        sets = np.tile(np.arange(K, dtype=np.int32), (B, 1))
        desc = lib.make_weights(w["w_up"][:K], None, w["b_up"][:K], w["w_down"][:K], w["b_down"])   # the first K rows
    y = lib.ffn_decode(x, desc, "relu")
    torch.cuda.synchronize()
    Wd = down_out_major64(w, "neuron_major")
    for b in sorted({0, B // 2, B - 1}):
        ref = orc.ffn_relu(f64(x[b]), sets[b].astype(np.int64), f64(w["w_up"]), f64(w["b_up"]), Wd, f64(w["b_down"]))
        assert_close_rms(y[b], ref, dt, f"sentence {b}")
