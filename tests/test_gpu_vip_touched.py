"""GPU: a pushed hop through bins finishes the vertices that it reaches packed 64 lanes and 256 vertices at a time, each
wavefront those of its 1024 rows: numbers of them around those sizes, side by side, spread and at the rows' ends, in the last,
partly filled block too, with a running total from before or none, and at a last hop.  Against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
N = 256 * 16384 + 2000                           # 257 row blocks, the last with one whole wavefront's rows and a part


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


@pytest.mark.parametrize("spread", [False, True])
@pytest.mark.parametrize("hop0,fanouts", [(False, (1, 1)), (True, (1, 1)), (False, (3,)), (True, (2, 5, 1))])
def test_reached_vertices(spp, ctx, spread, hop0, fanouts):
    print("[case]", spread, hop0, fanouts, flush=True)
    rng = np.random.default_rng(7)
    U = []
    for i, n in enumerate((1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 320, 511, 512, 513, 768, 1023, 1024)):
        rows = np.arange(1024) if not spread else rng.permutation(1024)
        U.append((20 + i * 37) * 1024 + rows[1024 - n:])         # up to the last of the 1024
    U.append(N - 1 - np.arange(0, 1900, 1 if not spread else 3))
    U = np.unique(np.concatenate(U))
    T = (3_000_000 + np.arange(U.size) * 7).astype(np.int64)
    col = (np.arange(N) + 5) % N                                 # one edge per vertex
    col[T] = rng.permutation(U)
    rp = np.arange(N + 1, dtype=np.int64)
    T = T.astype(np.int32)
    dev = torch.device("cuda:0")
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col.astype(np.int32)).to(dev), in_lists=True, chunked=True)
    batch = T.size // 2
    for per_hop in (False, True):
        got = spp.vip_propagate(ctx, G, torch.from_numpy(T).to(dev), batch, fanouts, include_hop0=hop0, per_hop=per_hop)
        assert all(spp.vip_last_hops(ctx, len(fanouts))[0])      # pushed, the last one too
        ref_t, ref_h = oracle.vip(rp, col.astype(np.int32), T, batch, fanouts, include_hop0=hop0)
        for g, ref in zip(got if per_hop else (got,), (ref_t, ref_h)):
            # results are rounded to fp32 at every hop: 6e-8 a hop, well below the 1e-5 the entry point states
            assert np.all(np.abs(g.cpu().numpy().astype(np.float64) - ref) <= 1e-6 * np.asarray(ref) + 1e-37)
    G.close()
