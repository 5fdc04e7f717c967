"""GPU: the general propagation's sums over a row block's entries, whose shares begin and end inside the vectors they are read
as (of four weights and rows from a walk by tiles, of two pairs from a list): numbers of entries that leave every remainder,
below and above a round of a workgroup, in one block and in several.  Against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spp():
    import paper_2305_03152_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("N", [3000, 5 * 16384 + 11])
@pytest.mark.parametrize("M", [1, 2, 4, 5, 6, 7, 8, 9, 1023, 4097, 16385, 16386, 16387, 16388, 33001, 200003])
def test_remainders(spp, N, M):
    print("[case]", N, M, flush=True)
    rng = np.random.default_rng(N * 7 + M)
    row = np.sort(rng.integers(0, N, M))
    rp = np.zeros(N + 1, dtype=np.int64)
    np.cumsum(np.bincount(row, minlength=N), out=rp[1:])
    within = np.arange(M) - rp[row]
    col = (np.repeat(rng.integers(0, N, N), np.diff(rp)) + within) % N   # distinct in a row
    col = col[np.lexsort((col, row))].astype(np.int32)
    p0, t = rng.random(N).astype(np.float32), [rng.random(M).astype(np.float32) for _ in range(2)]
    ref, _ = oracle.vip_general(rp, col, p0, t, 2)
    dev = torch.device("cuda:0")
    ctx = spp.Context(0)                         # its buffers are sized for these entries
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True)
    for shift in (0, 1):                                                 # 1: not aligned for the tiles, from the list
        td = [torch.zeros(M + 4, device=dev)[shift:shift + M].copy_(torch.from_numpy(a)) for a in t]
        got = spp.vip_propagate_general(ctx, G, torch.from_numpy(p0).to(dev), td, 2).cpu().numpy().astype(np.float64)
        # the entry point's bound: fp32 terms of one sign, and a second hop from probabilities rounded to fp32
        assert np.all(np.abs(got - ref) <= 1e-5 * np.asarray(ref) + 1e-37), shift
    G.close()
    ctx.close()
