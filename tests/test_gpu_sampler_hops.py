"""GPU: fanout sampling where the hop kernels can go wrong -- ends of tiles and granules, the fanouts at
which the tile's size changes, no seeds, more seeds than hop 1 sums by itself, hubs that every target
samples, and ids that share the hash bits which name a partition of the id table -- against the CPU oracle,
bit for bit."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
SEED = 0x1234567890ABCDEF


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


def _csr(rows, N):
    """rows: {vertex: ascending distinct neighbours}"""
    rp = np.zeros(N + 1, dtype=np.int64)
    for v, a in rows.items():
        rp[v + 1] = len(a)
    np.cumsum(rp, out=rp)
    col = np.concatenate([rows[v] for v in sorted(rows)]).astype(np.int32) if rows else np.zeros(0, np.int32)
    return rp, col


def _random_graph(N, seed, max_deg):
    rng = np.random.default_rng(seed)
    deg = np.minimum(rng.zipf(1.6, N), max_deg)
    deg[rng.random(N) < 0.1] = 0
    src = np.repeat(np.arange(N, dtype=np.int64), deg)
    dst = rng.integers(0, N, src.size)
    key = np.unique((src << 32 | dst)[src != dst])
    rp = np.zeros(N + 1, dtype=np.int64)
    np.cumsum(np.bincount(key >> 32, minlength=N), out=rp[1:])
    return rp, (key & 0xFFFFFFFF).astype(np.int32)


def _check(spp, ctx, rp, col, batches, fanouts):
    dev = torch.device("cuda:0")
    N = rp.size - 1
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev))
    seeds = [torch.from_numpy(b.astype(np.int32)).to(dev) for b in batches]
    bufs = [spp.MFGBuffers(dev, len(b), fanouts, N) for b in batches]
    for rep in range(2):                                     # the second call meets what the first one left behind
        spp.sample_mfg_multi(ctx, G, [(s, 7 * rep + i, m) for i, (s, m) in enumerate(zip(seeds, bufs))], fanouts, SEED)
        for i, (b, m) in enumerate(zip(batches, bufs)):
            ref = oracle.sample_mfg(rp, col, b.astype(np.int32), fanouts, SEED, 7 * rep + i)
            L = len(fanouts)
            assert m.n == ref.n and m.e == ref.e, (m.n, ref.n, m.e, ref.e)
            assert m.counts.cpu().numpy()[:L + 1].tolist() == list(ref.n)
            assert np.array_equal(m.node_ids[:m.n[L]].cpu().numpy(), ref.node_ids)
            for h in range(L):
                assert np.array_equal(m.indptr[h][:m.n[h] + 1].cpu().numpy(), ref.indptr[h]), (i, h)
                assert np.array_equal(m.src[h][:m.e[h + 1]].cpu().numpy(), ref.src[h]), (i, h)
    G.close()


@pytest.mark.parametrize("fanouts", [(5,), (16, 2), (17, 3), (32, 1), (33, 2), (64, 2), (3, 4, 5)], ids=str)
def test_seed_counts_around_tiles(spp, ctx, fanouts):
    print("[case] fanouts", fanouts, flush=True)
    rp, col = _random_graph(9000, 5, 300)
    rng = np.random.default_rng(1)
    for counts in ([0], [1], [15, 0, 16, 17], [255, 256, 257], [4096], [4097, 300], [9000]):
        _check(spp, ctx, rp, col, [rng.permutation(9000)[:c] for c in counts], fanouts)


def test_many_minibatches_of_unequal_size(spp, ctx):
    print("[case] 64 minibatches", flush=True)
    rp, col = _random_graph(20000, 6, 100)
    rng = np.random.default_rng(2)
    _check(spp, ctx, rp, col, [rng.permutation(20000)[:int(c)] for c in rng.integers(0, 700, 64)], (12, 6, 4))
    _check(spp, ctx, rp, col, [rng.permutation(20000)[:int(c)] for c in rng.integers(0, 90, 13)], (4, 9))


def test_hop_of_more_than_a_million_ids(spp, ctx):
    print("[case] one large minibatch", flush=True)
    rp, col = _random_graph(300000, 7, 40)
    _check(spp, ctx, rp, col, [np.random.default_rng(3).permutation(300000)[:200000]], (15, 10))


def test_hubs_that_every_target_samples(spp, ctx):
    print("[case] hubs", flush=True)
    N = 70000
    rows = {v: [0, 1, 2, 69999] for v in range(10, 60000)}
    rp, col = _csr(rows, N)
    _check(spp, ctx, rp, col, [np.arange(10, 60000)], (4, 3))


def test_ids_that_share_their_partition(spp, ctx):
    # 8192 + 8192 ids whose hash agrees in the top eight bits: more than one table holds, in one partition
    print("[case] shared hash bits", flush=True)
    N = 1 << 22
    ids = np.arange(N, dtype=np.uint64)
    crowd = np.flatnonzero(((ids * 0x9E3779B1) & 0xFFFFFFFF) >> 24 == 77).astype(np.int64)
    assert crowd.size > 16000
    rng = np.random.default_rng(4)
    seeds = rng.permutation(N)[:512]
    rows = {int(v): np.sort(rng.choice(crowd, 40, replace=False)) for v in seeds}
    rows = {v: a[a != v] for v, a in rows.items()}
    rp, col = _csr(rows, N)
    _check(spp, ctx, rp, col, [seeds], (36, 5))
    # the same crowd as seeds: they meet in the table as targets
    _check(spp, ctx, rp, col, [crowd[:12000]], (2,))
