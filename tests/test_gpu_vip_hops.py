"""GPU: which hops of a propagation are pushed and which are pulled, decided on the device -- against the rule
computed from the CPU oracle's probabilities, and the probabilities of both forms against the oracle, for
frontiers that are empty, sparse, at the line between the two and dense, one or many source chunks of the
structure, and both ways of listing a frontier (the line is at 2^22 vertices)."""
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


def _ring(N, deg):
    """Vertex v points at v+1 .. v+deg (mod N): `deg * N` edges, a frontier of known size after every hop."""
    col = (np.arange(N, dtype=np.int64)[:, None] + np.arange(1, deg + 1)) % N
    return np.arange(N + 1, dtype=np.int64) * deg, np.sort(col, axis=1).astype(np.int32).ravel()


# deg 8: a frontier of n vertices in a row has 8 n out-edges, the next one n + 7 vertices; pushed up to N / 16 vertices
@pytest.mark.parametrize("N,deg,nT,fanouts,want", [
    (4, 1, 1, (1,), (0,)),                                        # one edge out of M = 4: more than a sixteenth
    (16, 1, 1, (1, 1, 1), (1, 1, 1)),                             # exactly a sixteenth, three times
    (40000, 8, 2486, (8, 8, 8), (1, 1, 1)),                       # 2486, 2493, 2500 = N/16 vertices
    (40000, 8, 2487, (8, 8, 8), (1, 1, 0)),                       # 2501 at the third hop
    (40000, 8, 2501, (8, 8, 8), (0, 0, 0)),                       # pulled from the first
    (600000, 2, 37499, (2, 2, 2, 2), (1, 1, 0, 0)),               # three source chunks
    ((1 << 22) - 1, 1, 1000, (1, 1), (1, 1)),
    (1 << 22, 1, 1 << 18, (1, 1), (1, 1)),
    ((1 << 22) + 5, 1, (1 << 18) + 9, (1, 1), (0, 0))])
def test_the_form_of_each_hop(spp, ctx, N, deg, nT, fanouts, want):
    print("[case]", N, deg, nT, fanouts, flush=True)
    rp, col = _ring(N, deg)
    T = ((np.arange(nT) + N // 3) % N).astype(np.int32)
    dev = torch.device("cuda:0")
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True)
    batch = max(1, nT // 2)
    p, ph = spp.vip_propagate(ctx, G, torch.from_numpy(T).to(dev), batch, fanouts, per_hop=True)
    pushed, edges = spp.vip_last_hops(ctx, len(fanouts))
    assert tuple(int(x) for x in pushed) == want
    for h, e in enumerate(edges):                     # the hop after a pulled one is not looked at
        assert e == (deg * (nT + h * (deg - 1)) if h == 0 or pushed[h - 1] else -1)
    ref_t, ref_h = oracle.vip(rp, col, T, batch, fanouts)
    for got, ref in ((p, ref_t), (ph, ref_h)):
        # results are rounded to fp32 at every hop: 6e-8 a hop, well below the 1e-5 the entry point states
        assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= 1e-6 * np.asarray(ref) + 1e-37)
    G.close()
