"""GPU: tiles of the CSR whose rows begin and end where the kernels that walk them change their way: one row over many 64s or
whole tiles, one to sixty-four rows inside 64 edges, rows that end on a 64 or a tile, and row blocks for one to several
wavefronts.  A structure that does not read back as the CSR's edges is refused by its build; the probabilities over it are
compared with the CPU oracle."""
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


@pytest.fixture(scope="module")
def ctx(spp):
    c = spp.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("N", [16384, 64 * 16384, 65 * 16384 + 7, 300 * 16384])          # 1, 64, 66 and 300 row blocks
@pytest.mark.parametrize("lengths", [(1,), (13, 16), (15,), (17, 1, 1, 1), (63, 64, 65), (64,), (4096,), (4095, 1, 8192), (200, 0, 0, 1, 1, 1, 1, 1, 300)],
                         ids=str)
def test_rows_of_a_tile(spp, ctx, N, lengths):
    print("[case]", N, lengths, flush=True)
    rng = np.random.default_rng(N + len(lengths))
    deg = np.zeros(N, dtype=np.int64)
    deg[::max(1, N // 4096)][:4000] = 1          # rows far apart first: tiles with many empty ones
    some = np.resize(np.array(lengths), min(N // 2, 60000 // max(1, int(np.mean(lengths)))))
    deg[N // 2:N // 2 + some.size] = np.minimum(some, N // 2)
    rp = np.zeros(N + 1, dtype=np.int64)
    np.cumsum(deg, out=rp[1:])
    row = np.repeat(np.arange(N), deg)
    step = rng.integers(1, np.maximum(N // np.maximum(deg, 1), 1) + 1)
    col = (np.repeat(rng.integers(0, N, N), deg) + (np.arange(rp[-1]) - rp[row]) * step[row]) % N
    col = col[np.lexsort((col, row))].astype(np.int32)
    dev = torch.device("cuda:0")
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True)
    T = np.flatnonzero(deg)[::3].astype(np.int32)
    fan = (3, 5)
    p = spp.vip_propagate(ctx, G, torch.from_numpy(T).to(dev), max(1, T.size // 4), fan).cpu().numpy()
    ref, _ = oracle.vip(rp, col, T, max(1, T.size // 4), fan)
    assert np.all(np.abs(p.astype(np.float64) - ref) <= 1e-5 * ref + 1e-37)                # the entry point's bound
    p0 = rng.random(N).astype(np.float32)
    t = [rng.random(col.size).astype(np.float32)]
    got = spp.vip_propagate_general(ctx, G, torch.from_numpy(p0).to(dev), [torch.from_numpy(t[0]).to(dev)], 1).cpu().numpy()
    want, _ = oracle.vip_general(rp, col, p0, t, 1)
    assert np.all(np.abs(got.astype(np.float64) - want) <= 1e-5 * np.asarray(want) + 1e-37)
    G.close()
