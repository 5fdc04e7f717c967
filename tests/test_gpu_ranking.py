"""GPU: the ranking behind the replica cache where the search for its threshold can go wrong -- ties across the
cut, constant scores, scores that differ in their last bits, denormals, infinities and NaN, too few candidates,
both sizes of the sort -- against the CPU oracle."""
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
    s = np.exp(rng.normal(-8, 3, N)).astype(np.float32)
    if kind == "constant":
        s[:] = 0.25
    elif kind == "few values":
        s = rng.integers(0, 5, N).astype(np.float32)
    elif kind == "last bits":
        s = (np.float32(0.5).view(np.uint32) + rng.integers(0, 700, N).astype(np.uint32)).view(np.float32)
    elif kind == "denormal":
        s = rng.integers(0, 1 << 19, N).astype(np.uint32).view(np.float32)
    elif kind == "odd":
        s[rng.random(N) < 0.01] = np.inf
        s[rng.random(N) < 0.01] = np.nan
        s[rng.random(N) < 0.2] *= -1
    elif kind == "sparse":
        s[rng.random(N) < 0.999] = 0.0
    return s


@pytest.mark.parametrize("kind", ["spread", "constant", "few values", "last bits", "denormal", "odd", "sparse"])
def test_cache_membership(spp, ctx, kind):
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(len(kind))
    for N, lo, hi, K, alpha in [(1, 0, 0, 1, 1.0), (257, 10, 60, 2, 0.3), (4099, 0, 1000, 4, 0.5), (65537, 20000, 30000, 8, 0.9995),
                                (65537, 20000, 30000, 8, 1.01), (300001, 7, 9, 3, 0.5), (1200007, 0, 150000, 8, 0.16), (50021, 0, 100, 1, 5.0)]:
        print("[case]", kind, N, alpha, flush=True)
        s = _scores(kind, N, rng)
        rows = torch.arange(N - (hi - lo), dtype=torch.float32, device=dev)[:, None].repeat(1, 2) if hi - lo < N else torch.zeros((1, 2), device=dev)
        cache = spp.build_vip_cache(ctx, torch.from_numpy(s).to(dev), lo, hi, K, alpha, rows, 2, 4)
        ref = oracle.cache_select(s, lo, hi, K, alpha)
        ids = cache.ids.cpu().numpy()
        assert np.array_equal(ids, ref), (kind, N)
        slot = np.full(N, -1, np.int32)
        slot[ref] = np.arange(ref.size)
        probe = np.r_[0:min(N, 5000), N - min(N, 5000):N].astype(np.int32)
        assert np.array_equal(cache.lookup(torch.from_numpy(probe).to(dev)).cpu().numpy(), slot[probe])
        if ref.size:
            out, st = spp.gather_features(ctx, cache, torch.zeros((max(hi - lo, 1), 2), device=dev), N, lo, hi, None, cache.ids.contiguous())
            assert st["n_cache_hit"] == ref.size
            assert np.array_equal(out[:, 1].cpu().numpy(), np.where(ref < lo, ref, ref - (hi - lo)).astype(np.float32))
        cache.close()
