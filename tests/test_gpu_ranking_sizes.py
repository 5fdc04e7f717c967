"""GPU: rankings whose numbers of keys lie where the sort changes its form or a tile, a wavefront's part of it or a workgroup's run
of scores ends, with many equal scores (their order is by id), against the CPU oracle; and the same sort behind the local order."""
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


def _scores(kind, N, rng):
    if kind == "levels":
        return (rng.integers(1, 12, N) / 16).astype(np.float32)
    return np.exp(rng.normal(-8, 3, N)).astype(np.float32)


@pytest.mark.parametrize("kind", ["spread", "levels"])
@pytest.mark.parametrize("n", [4095, 4096, 4097, 8256, 10241, 40959, 40961, 524287, 524288, 524289, 1048575, 1048576, 1048577])
def test_number_of_keys(spp, ctx, kind, n):
    print("[case]", kind, n, flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n)
    N = n + 1 if kind == "spread" else n + n // 2 + 77       # nearly all kept; ties at the threshold beyond n
    s = _scores(kind, N, rng)
    lo = N // 3
    # of the ids outside [lo, lo + 1) the first n are kept
    cache = spp.build_vip_cache(ctx, torch.from_numpy(s).to(dev), lo, lo + 1, 1, (n + 0.5) / N, torch.zeros((N - 1, 1), device=dev), 1, 4)
    ref = oracle.cache_select(s, lo, lo + 1, 1, (n + 0.5) / N)
    assert ref.size == n and np.array_equal(cache.ids.cpu().numpy(), ref)
    cache.close()


@pytest.mark.parametrize("N", [1, 63, 64, 8191, 8192, 8193, 2097151, 2097153])
def test_where_the_runs_of_scores_end(spp, ctx, N):
    """Every third id a candidate, half of those kept."""
    print("[case]", N, flush=True)
    dev = torch.device("cuda:0")
    s = _scores("spread", N, np.random.default_rng(N))
    s[np.arange(N) % 3 != 0] = 0.0
    cache = spp.build_vip_cache(ctx, torch.from_numpy(s).to(dev), 0, 0, 1, 1 / 6 if N > 6 else 1.0, torch.zeros((N, 1), device=dev), 1, 4)
    assert np.array_equal(cache.ids.cpu().numpy(), oracle.cache_select(s, 0, 0, 1, 1 / 6 if N > 6 else 1.0))
    cache.close()


@pytest.mark.parametrize("n", [2, 64, 2047, 2048, 2049, 524289])
def test_local_order(spp, ctx, n):
    print("[case]", n, flush=True)
    dev = torch.device("cuda:0")
    s = _scores("levels", n, np.random.default_rng(n))
    s[::5] = 0.0
    rows = torch.zeros((n, 1), dtype=torch.float32).pin_memory()
    store = spp.build_local_store(ctx, torch.from_numpy(s).to(dev), 0, n, 1.0, rows)
    rank = store.rank(torch.arange(n, dtype=torch.int32, device=dev)).cpu().numpy()
    order = np.lexsort((np.arange(n), -s))
    want = np.empty(n, np.int64)
    want[order] = np.arange(n)
    assert np.array_equal(rank, want)
    store.close()
