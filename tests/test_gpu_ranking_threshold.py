"""GPU: a ranking keeps only what reaches its threshold, wherever that lies -- seen through the workspace that the
context keeps, which holds 16 bytes per score that is sorted."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["ordinary", "smallest denormals", "too few"])
def test_what_is_sorted_is_what_can_be_kept(kind):
    import paper_2305_03152_amd as spp
    dev = torch.device("cuda:0")
    N, K, alpha = 1_500_000, 1, 1e-4                                  # 150 are kept
    rng = np.random.default_rng(2)
    if kind == "ordinary":
        s = rng.random(N).astype(np.float32)
    elif kind == "smallest denormals":                                # below 2^20 in their bits: the first digit of all is 0
        s = rng.integers(1, 1 << 20, N).astype(np.uint32).view(np.float32)
    else:
        s = np.zeros(N, np.float32)
        s[rng.integers(0, N, 100)] = 0.5
    ctx = spp.Context(0)
    score = torch.from_numpy(s).to(dev)
    rows = torch.zeros((N, 1), device=dev)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    cache = spp.build_vip_cache(ctx, score, 0, 0, K, alpha, rows, 1, 4)
    kept = free - torch.cuda.mem_get_info()[0]
    assert np.array_equal(cache.ids.cpu().numpy(), oracle.cache_select(s, 0, 0, K, alpha))
    assert kept < 12 << 20, kept                                      # 16 bytes for each of the 1.5M scores would be 24 MB
    cache.close()
    ctx.close()
