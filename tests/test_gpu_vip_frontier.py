"""GPU: the frontier that a hop's writer lists for the next hop's push -- segments of one and of several rounds of
vertices, ids that the training set names more than once, rows long enough to be walked by all workgroups together (more
than 1024 entries), at the first hop and reached by it -- against the CPU oracle; and that a push takes
no longer for few long rows, or for many of one edge, than for as many edges in ordinary rows."""
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


def _graph(deg):
    """Vertex v points at v+1 .. v+deg[v] (mod N)."""
    N = deg.size
    rp = np.zeros(N + 1, dtype=np.int64)
    np.cumsum(deg, out=rp[1:])
    row = np.repeat(np.arange(N), deg)
    col = (row + 1 + np.arange(rp[-1]) - rp[row]) % N
    wrap = np.flatnonzero(np.arange(N) + deg >= N)
    for v in wrap:
        col[rp[v]:rp[v + 1]].sort()
    return rp, col.astype(np.int32)


def _case(name):
    if name == "giants":                 # the first is in T, the second is reached by vertex 10, the third by the first
        deg = np.full(220_000, 16)
        deg[50], deg[11], deg[20_000], deg[99_000] = 32769, 70_000, 32768, 33_000
        return deg, np.array([10, 50, 150_000, 219_990], np.int32)
    if name == "named_twice":
        deg = np.full(60_000, 9)
        T = np.arange(1500, dtype=np.int32) * 17
        return deg, np.concatenate([T, T[:700], T[:1]])
    if name == "long_twice":             # rows above the limit and below, each named up to three times
        deg = np.full(600_000, 20)
        T = (np.arange(300, dtype=np.int64) * 1700).astype(np.int32)
        deg[T] = 1000 + np.arange(300) % 3 * 20
        return deg, np.concatenate([T, T[::-1], T[100:200]])
    if name == "long_rows":              # 1100 rows above 1024 entries, which a workgroup lays out in two rounds, 1100 below
        deg = np.full(1_200_000, 30)
        T = (np.arange(2200, dtype=np.int64) * 500).astype(np.int32)
        deg[T] = 1025 + np.arange(2200) % 3
        deg[T[::2]] = 1022 + np.arange(1100) % 3
        return deg, T
    if name == "rounds":                 # more training vertices than 2048 workgroups take in a round, all with one edge
        deg = np.full(1_400_000, 14)
        T = (np.arange(600_000, dtype=np.int64) * 2).astype(np.int32)
        deg[T] = 1
        return deg, T
    deg = np.full(300, 20)               # "one": a single training vertex, the last
    return deg, np.array([299], np.int32)


@pytest.mark.parametrize("name", ["giants", "long_rows", "long_twice", "named_twice", "rounds", "one"])
@pytest.mark.parametrize("chunked", [False, True])
def test_listed_frontiers(spp, ctx, name, chunked):
    print("[case]", name, chunked, flush=True)
    deg, T = _case(name)
    rp, col = _graph(deg)
    dev = torch.device("cuda:0")
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True, chunked=chunked)
    fanouts, batch = (3, 40_000, 5), max(1, T.size // 3)
    for _ in range(2):                   # a call leaves its counters and accumulators as the next one expects them
        p, ph = spp.vip_propagate(ctx, G, torch.from_numpy(T).to(dev), batch, fanouts, per_hop=True)
        pushed, edges = spp.vip_last_hops(ctx, len(fanouts))
        assert pushed[0] and edges[0] == int(deg[T].sum())
        ref_t, ref_h = oracle.vip(rp, col, T, batch, fanouts)
        for got, ref in ((p, ref_t), (ph, ref_h)):
            # results are rounded to fp32 at every hop: 6e-8 a hop, well below the 1e-5 the entry point states
            assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= 1e-6 * np.asarray(ref) + 1e-37)
    G.close()


@pytest.mark.parametrize("rows,plain_rows,limit", [(64, 20480, 3.0), (204800, 2048, 1.85)], ids=["long", "short"])
def test_edges_are_shared_out(spp, rows, plain_rows, limit):
    """The same number of edges in rows of two lengths: the same adds, by all CUs either way.  1,024,000 edges in 64 rows took
    eight times as long as in 20480 (241 and 31 us) where one workgroup walked the 64; 204,800 rows of one edge 2.2 times as
    long as 2048 of 100 where a wavefront of 16 walked a workgroup's.  The limits leave room for noise."""
    edges = 1_024_000 if rows == 64 else 204_800
    deg = np.full(1_200_000, 30)
    deg[:rows], deg[rows:rows + plain_rows] = edges // rows, edges // plain_rows
    rp, col = _graph(deg)
    dev = torch.device("cuda:0")
    ctx = spp.Context(0)
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True)
    took = []
    for T in (torch.arange(rows, dtype=torch.int32), torch.arange(rows, rows + plain_rows, dtype=torch.int32)):
        T = T.to(dev)
        spp.vip_propagate(ctx, G, T, max(1, T.numel() // 2), (3,))
        ctx.timing(True)
        for _ in range(8):
            spp.vip_propagate(ctx, G, T, max(1, T.numel() // 2), (3,))
        took.append(ctx.time_stats()[2][1])                 # SPP_T_VIP_HOP_FIRST, the shortest
        assert spp.vip_last_hops(ctx, 1) == ([True], [edges])
        ctx.timing(False)
    ctx.close()
    print("[took]", rows, plain_rows, took)
    assert took[0] < limit * took[1], took
