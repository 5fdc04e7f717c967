"""GPU: dense hops over row blocks where the stretch of y that 512 consecutive edges need is just short enough for
the window that a wavefront holds in LDS (444 values), just too long for it, or ends at the graph's last vertex
-- against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


# `per` consecutive sources have 512 edges together, so any 512 consecutive edges span per - 1 or per sources: 442 or 443
# (all in the window), 443 or 444 (both sides of the limit), 444 or 445 (none).  One row block: its 131072 k edges are cut
# into whole rounds of 512 for 16 wavefronts of 16 shares, the last of which ends at the last vertex.
@pytest.mark.parametrize("per,first,k", [(443, 0, 2), (444, 0, 2), (444, 1, 2), (444, 2, 1), (444, 3, 3), (445, 1, 2), (40, 2, 1), (512, 0, 1)])
def test_windows_of_y(per, first, k):
    import paper_2305_03152_amd as spp
    print("[case]", per, first, k, flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(per + first)
    deg = np.full(per, 512 // per)
    deg[rng.permutation(per)[:512 - deg.sum()]] += 1
    deg = np.r_[np.zeros(first, int), np.tile(deg, 256 * k)]
    N, M = deg.size, int(deg.sum())
    assert M == 131072 * k and deg.max() <= 16
    rp = np.r_[0, np.cumsum(deg)].astype(np.int64)
    # distinct targets of one source inside the first row block: a random start, then odd steps
    src = np.repeat(np.arange(N), deg)
    rows = min(N, 16384)
    col = (rng.integers(0, rows, N)[src] + (np.arange(M) - rp[src]) * 977) % rows
    col = (np.sort(src * np.int64(1 << 20) + col) & ((1 << 20) - 1)).astype(np.int32)
    T = np.flatnonzero(rng.random(N) < 0.6).astype(np.int32)
    ctx = spp.Context(0)
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True)
    p, ph = spp.vip_propagate(ctx, G, torch.from_numpy(T).to(dev), T.size // 5, (1, 1), per_hop=True)
    assert spp.vip_last_hops(ctx, 2)[0][0] == 0                       # pulled
    ref_t, ref_h = oracle.vip(rp, col, T, T.size // 5, (1, 1))
    for got, ref in ((p, ref_t), (ph, ref_h)):
        # results are rounded to fp32 at every hop: 6e-8 a hop, well below the 1e-5 the entry point states
        assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= 1e-6 * np.asarray(ref) + 1e-37)
    ctx.close()
