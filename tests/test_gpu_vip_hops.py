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


# more row blocks than CUs in the chunked layout: pushes go through bins of the row blocks.  256 blocks, the last with one
# vertex, and 258; frontiers of one vertex, less and more than 64 and 256 vertices for each of 1024 workgroups, in hubs
# whose rows are walked in pieces, at the rim of every block, and all edges into one vertex.
@pytest.mark.parametrize("N,kind,nT", [
    (255 * 16384 + 1, "ring", 1), (255 * 16384 + 1, "ring", 65536), (255 * 16384 + 1, "ring", 65537),
    (257 * 16384 + 77, "ring", 262145), (257 * 16384 + 77, "rim", 257), (257 * 16384 + 77, "hubs", 9), (257 * 16384 + 77, "star", 70000)])
def test_pushes_through_bins(spp, ctx, N, kind, nT):
    print("[case]", N, kind, nT, flush=True)
    rng = np.random.default_rng(N + nT)
    rp, col = _ring(N, 2)
    T = ((np.arange(nT, dtype=np.int64) * 13 + N // 3) % N).astype(np.int32)
    if kind == "rim":                   # the last and the first vertex of the blocks
        T = np.unique(np.r_[np.arange(1, 258) * 16384 - 1, np.arange(1, 258) * 16384 - 2, N - 1]).astype(np.int32)
    if kind == "hubs":
        T = (np.arange(nT) * 400000 + 5).astype(np.int32)
        deg = np.full(N, 2)
        for i, v in enumerate(T):
            deg[v] = (4095, 4096, 4097, 8192, 8193, 30000, 1, 2, 20000)[i]
        rp2 = np.zeros(N + 1, dtype=np.int64)
        np.cumsum(deg, out=rp2[1:])
        col2 = np.empty(rp2[-1], dtype=np.int32)
        own = np.repeat(deg == 2, deg)
        col2[own] = col[np.repeat(deg == 2, 2)]
        for v in T:
            if deg[v] != 2:
                others = rng.choice(N - 1, deg[v], replace=False)
                col2[rp2[v]:rp2[v + 1]] = np.sort(others + (others >= v))
        rp, col = rp2, col2
    if kind == "star":                  # every training vertex points at vertex 7 as well as at its successor
        c = col.reshape(N, 2)
        T = T[(T != 7) & (T + 1 < N)]
        c[T] = np.sort(np.stack([np.full(T.size, 7), np.where(T == 6, 8, T + 1)], 1), axis=1)
        col = c.ravel()
    dev = torch.device("cuda:0")
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True, chunked=True)
    fanouts, batch = (4000, 2, 2), max(1, T.size // 2)
    p, ph = spp.vip_propagate(ctx, G, torch.from_numpy(T).to(dev), batch, fanouts, per_hop=True)
    pushed, edges = spp.vip_last_hops(ctx, len(fanouts))
    ref_t, ref_h = oracle.vip(rp, col, T, batch, fanouts)
    deg = np.diff(rp)
    front = [int(deg[T].sum())] + [int(deg[np.asarray(ref_h[h]) > 0].sum()) for h in range(2)]
    for h in range(3):
        assert pushed[h] == (16 * front[h] <= col.size and (h == 0 or pushed[h - 1]))
        assert edges[h] == (front[h] if h == 0 or pushed[h - 1] else -1)
    assert pushed[0]
    for got, ref in ((p, ref_t), (ph, ref_h)):
        # results are rounded to fp32 at every hop: 6e-8 a hop, well below the 1e-5 the entry point states
        assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= 1e-6 * np.asarray(ref) + 1e-37)
    G.close()


@pytest.mark.parametrize("batch", [1, 300, 599, 600])
def test_probabilities_to_fp32_rounding(spp, ctx, batch):
    """Chains T -> u -> v of which every u and v has one in-edge: p^[1](u) and p^[2](v) are products of two and
    three factors over the whole of (0, 1], the library's fp64 exponentials and logarithms invert each other."""
    nT, deg = 600, np.r_[np.arange(1, 301), np.arange(1, 301) * 40]
    nu = int(deg.sum())
    N = nT + 2 * nu
    rp = np.zeros(N + 1, dtype=np.int64)
    np.cumsum(np.r_[deg, np.ones(nu, int), np.zeros(nu, int)], out=rp[1:])
    col = np.r_[nT + np.arange(nu), nT + nu + np.arange(nu)].astype(np.int32)
    T = np.arange(nT, dtype=np.int32)
    dev = torch.device("cuda:0")
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True)
    for fanouts in ((1, 1), (299, 1), (12000, 2)):
        print("[case]", batch, fanouts, flush=True)
        p, ph = spp.vip_propagate(ctx, G, torch.from_numpy(T).to(dev), batch, fanouts, per_hop=True)
        ref_t, ref_h = oracle.vip(rp, col, T, batch, fanouts)
        # a hop's logarithms are rounded to fp32 (2^-24, which 1 - e^s does not enlarge), and so is the result
        for got, ref, roundings in ((ph[0], ref_h[0], 2), (ph[1], ref_h[1], 3), (p, ref_t, 3)):
            ref = np.asarray(ref)
            assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= (roundings + 0.01) * 2.0**-24 * ref)
    G.close()


# rounds of 8192 edges of a workgroup's portion (64 vertices and more): just below, at and above one round, one
# vertex more than a portion each, more vertices than 1024 for every workgroup, rows longer than a round's share
@pytest.mark.parametrize("N,deg", [(32768, 127), (32768, 128), (32768, 129), (32769, 1), (525000, 2), (7000, 300)])
def test_general_probabilities_in_rounds(spp, ctx, N, deg):
    print("[case]", N, deg, flush=True)
    rng = np.random.default_rng(N + deg)
    rp, col = _ring(N, deg)
    p0 = np.where(rng.random(N) < 0.95, rng.random(N), 0.0).astype(np.float32)
    t = [(rng.random(col.size) * min(1.0, 8 / deg)).astype(np.float32) for _ in range(2)]
    dev = torch.device("cuda:0")
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True)
    p, ph = spp.vip_propagate_general(ctx, G, torch.from_numpy(p0).to(dev), [torch.from_numpy(a).to(dev) for a in t], 2, per_hop=True)
    ref_t, ref_h = oracle.vip_general(rp, col, p0, t, 2)
    for got, ref in ((p, ref_t), (ph, ref_h)):
        # a term's logarithm carries a few units of fp32 (bin_log1p_neg), all terms have one sign, and the second hop
        # starts from probabilities rounded to fp32: the 1e-5 that the entry point states
        assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= 1e-5 * np.asarray(ref) + 1e-37)
    G.close()
