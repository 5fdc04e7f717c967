"""GPU: the transposed edges in row blocks, where the partition of the CSR can go wrong -- ends of tiles of
4096 edges, rows that span tiles, long runs of empty rows, one or many row blocks, graphs on both sides of a
source chunk of 2^18 -- seen through the probabilities that are pulled over them, against the CPU oracle."""
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


def _graph(N, M, rows, seed):
    """About M edges out of the vertices `rows`, the other rows empty."""
    rng = np.random.default_rng(seed)
    src = rng.choice(rows, M)
    dst = rng.integers(0, N, M)
    key = np.unique((src.astype(np.int64) << 32 | dst)[src != dst])
    rp = np.zeros(N + 1, dtype=np.int64)
    np.cumsum(np.bincount(key >> 32, minlength=N), out=rp[1:])
    return rp, (key & 0xFFFFFFFF).astype(np.int32)


def _exactly(rp, col, M):
    """The graph's first M edges."""
    return np.minimum(rp, M), col[:M]


@pytest.mark.parametrize("N,M,kind", [
    (2, 1, "all"), (300, 4095, "all"), (300, 4096, "all"), (300, 4097, "all"), (300, 8193, "all"), (16384, 40000, "all"), (16385, 40000, "all"),
    (70000, 6 * 4096, "ends"), (300000, 500000, "few"), (600000, 900000, "tail"), (1100000, 1500000, "all")])
def test_probabilities_over_row_blocks(spp, ctx, N, M, kind):
    print("[case]", N, M, kind, flush=True)
    rows = {"all": np.arange(N), "ends": np.r_[0:40, N - 40:N], "few": np.arange(0, N, 97),
            "tail": np.arange(N - 20000, N)}[kind]
    rp, col = _graph(N, M + M // 4 + 8, rows, N + M)
    if M < col.size:
        rp, col = _exactly(rp, col, M)
    dev = torch.device("cuda:0")
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True)
    # most vertices in the training set: the first hop is pulled over the structure
    T = np.flatnonzero(np.random.default_rng(1).random(N) < 0.9).astype(np.int32)
    T = T if T.size else np.zeros(1, np.int32)
    p, ph = spp.vip_propagate(ctx, G, torch.from_numpy(T).to(dev), 3 + T.size // 3, (7, 3), per_hop=True)
    ref_t, ref_h = oracle.vip(rp, col, T, 3 + T.size // 3, (7, 3))
    for got, ref in ((p, ref_t), (ph, ref_h)):
        # results are rounded to fp32 at every hop: 6e-8 a hop, well below the 1e-5 the entry point states
        assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= 1e-6 * np.asarray(ref) + 1e-37)
    G.close()
