"""The per-token selection kernel at the ends of rows: what lies behind a row is never a key."""
import numpy as np
import pytest
import torch

from oracle import coreinfer_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# rows that end inside, at and one past an item of 1024 keys, one item and an odd number of them, the last of each build
# (4, 8, 16, 24, 40 items); longer strides with larger values, infinities and NaN behind the row
@pytest.mark.parametrize("N", [1, 1023, 1024, 1025, 3072, 4097, 13824, 16384, 16385, 23552, 36865, 40960])
@pytest.mark.parametrize("M", [3, 300])
@pytest.mark.parametrize("dt", [torch.float32, torch.float16, torch.bfloat16])
def test_select_ends_of_rows(lib, N, M, dt):
    if M > 3 and N > 17000:
        M = 20
    print("row end case", N, M, dt, flush=True)
    g = torch.Generator().manual_seed(N + M)
    wide = torch.randn(M, N + 40, generator=g)
    wide[:, N:] = torch.tensor([float("inf"), 60000.0, float("nan"), 9.0]).repeat(10)
    if N > 8:
        wide[0, :4] = torch.tensor([float("inf"), float("nan"), -float("inf"), 0.0])
        wide[1, :] = -wide[1, :].abs()      # nothing positive
        wide[1, N:] = 7.0
        wide[2, :] = 1.5                    # one value
    wide = wide.to(dt)
    act = wide.to(DEV)[:, :N]
    alpha, beta = 0.2, 0.4
    if dt == torch.float32:
        S, counts = lib.select(act, alpha, beta)
    else:
        S, counts = lib.select_hidden(act, "relu", alpha, beta)
    S_ref, c_ref = orc.select(wide[:, :N].float().numpy(), alpha, beta)
    assert np.array_equal(counts.cpu().numpy(), c_ref)
    assert np.array_equal(S.cpu().numpy(), S_ref)


# Values at the ends of the key range: signaling, quiet and negative NaN of the least and the largest payload, both zeros, the least and the
# largest denormal and normal number and infinity, the last as a tie that is cut; few positive ones, so that the threshold is among them
@pytest.mark.parametrize("dt,bits,act", [(torch.float32, 32, "relu"), (torch.float16, 16, "relu"), (torch.float16, 16, "swiglu"),
                                         (torch.bfloat16, 16, "relu"), (torch.bfloat16, 16, "swiglu")])
@pytest.mark.parametrize("N", [40, 2000, 9000])
def test_select_values_at_the_ends_of_the_range(lib, dt, bits, act, N):
    inf = {torch.float32: 0x7f800000, torch.float16: 0x7c00, torch.bfloat16: 0x7f80}[dt]
    sign = 1 << (bits - 1)
    normal = {torch.float32: 0x800000, torch.float16: 0x400, torch.bfloat16: 0x80}[dt]
    special = [inf + 1, inf | (inf >> 1 & ~inf) | 1, sign - 1, sign | (inf + 1), 2 * sign - 1, 0, sign, 1, normal - 1, normal, normal + 1,
               inf - 1, inf, inf, inf, sign | 1, sign | inf, sign | normal]
    M = 12
    v = np.zeros((M, N), dtype=np.int64)
    rng = np.random.default_rng(N)
    for m in range(M):
        at = rng.permutation(N)[:len(special)]
        v[m, at] = special
        if m % 3 == 1:
            v[m] = np.where(v[m] == 0, inf, v[m])      # infinities everywhere: ties at the largest key
        if m % 3 == 2:
            v[m] = np.where(v[m] == 0, rng.integers(1, normal, N), v[m])   # denormals
    kind = {32: (np.uint32, np.int32), 16: (np.uint16, np.int16)}[bits]
    raw = torch.from_numpy(v.astype(kind[0]).view(kind[1])).view(dt)
    alpha, beta = 0.2, 0.4
    if dt == torch.float32:
        S, counts = lib.select(raw.to(DEV), alpha, beta)
    else:
        S, counts = lib.select_hidden(raw.to(DEV), act, alpha, beta)
    A = raw.float().abs() if act == "swiglu" else raw.float()
    S_ref, c_ref = orc.select(A.numpy(), alpha, beta)
    assert np.array_equal(counts.cpu().numpy(), c_ref)
    assert np.array_equal(S.cpu().numpy(), S_ref)


# Def. 2 in parallel with as many workgroups as there are compute units (256) and with more, where its counts are requested
# later; fewer and more than 8192 vectors of counts before a workgroup; counts that do and do not start on 16 bytes
@pytest.mark.parametrize("B,M,N", [(4, 3, 16384), (4, 3, 16385), (5, 2, 13824), (3, 2, 40001), (2, 2, 65536)])
def test_select_batch_workgroups(lib, B, M, N):
    print("batch case", B, M, N, flush=True)
    act = torch.randn(B * M, N, generator=torch.Generator().manual_seed(N)).abs()
    S, counts = lib.select_batch(act.to(DEV), B, 0.2, 0.4)
    for b in range(B):
        S_ref, c_ref = orc.select(act[b * M:(b + 1) * M].numpy(), 0.2, 0.4)
        assert np.array_equal(counts[b].cpu().numpy(), c_ref)
        assert np.array_equal(S[b].cpu().numpy(), S_ref)
