"""GPU: the classification and the lists it leaves, at the ends of its chunks of 2048 ids -- lengths around a
chunk, empty lists, device counts below the bound, all ids of one kind, ids outside [0, N), rows of one vector and
of many -- against plain indexing."""
import numpy as np
import pytest
import torch

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


N, LO, HI, K = 40000, 5000, 15000, 4


@pytest.mark.parametrize("D,dtype", [(8, torch.float16), (1, torch.float32), (100, torch.float32), (768, torch.bfloat16)], ids=str)
@pytest.mark.parametrize("lengths", [(1,), (2047,), (2048,), (2049,), (4097, 0, 1, 2048), tuple([37, 2050] * 32)], ids=lambda x: f"{len(x)}x{x[0]}")
def test_gathered_rows_and_counts(spp, ctx, D, dtype, lengths):
    print("[case]", D, dtype, lengths[:4], flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(D + len(lengths))
    table = torch.from_numpy(rng.integers(-30000, 30000, (N, D)).astype(np.int16)).to(dtype)
    local = table[LO:HI].to(dev)
    remote = torch.cat([table[:LO], table[HI:]]).pin_memory()
    score = torch.from_numpy(rng.random(N).astype(np.float32)).to(dev)
    cache = spp.build_vip_cache(ctx, score, LO, HI, K, 0.8, remote, D, table.element_size())
    cached = np.zeros(N, bool)
    cached[cache.ids.cpu().numpy()] = True
    for kind in ("mixed", "local", "missed", "short", "bad"):
        ids, want = [], dict(n_local=0, n_cache_hit=0, n_miss=0)
        for n in lengths:
            x = rng.integers(0, N, n)
            if kind == "local":
                x = rng.integers(LO, HI, n)
            elif kind == "missed":
                x = rng.choice(np.flatnonzero(~cached & ((np.arange(N) < LO) | (np.arange(N) >= HI))), n)
            ids.append(x.astype(np.int32))
        used = [n - n // 3 if kind == "short" else n for n in lengths]
        lists = []
        for x, n, u in zip(ids, lengths, used):
            out = torch.full((max(n, 1), D), 7, dtype=dtype, device=dev)
            lists.append((torch.from_numpy(x).to(dev), n, torch.tensor([u], dtype=torch.int64, device=dev) if kind == "short" else None, out))
        if kind == "bad":
            if lengths[0] < 2:
                continue
            lists[0][0][1] = -5
            lists[0][0][lengths[0] - 1] = N
            with pytest.raises(spp.SppError):
                spp.gather_features_multi(ctx, cache, local, N, LO, HI, remote, lists)
            good = np.ones(lengths[0], bool)
            good[[1, lengths[0] - 1]] = False
            assert torch.equal(lists[0][3].cpu()[good], table[ids[0][good].astype(np.int64)])
            assert torch.all(lists[0][3].cpu()[~good] == 7)
            continue
        ctx.totals(reset=True)
        st = spp.gather_features_multi(ctx, cache, local, N, LO, HI, remote, lists)
        for (_, n, _, out), x, u in zip(lists, ids, used):
            x = x[:u]
            is_local = (x >= LO) & (x < HI)
            want["n_local"] += int(is_local.sum())
            want["n_cache_hit"] += int((cached[x] & ~is_local).sum())
            want["n_miss"] += int((~cached[x] & ~is_local).sum())
            assert torch.equal(out[:u].cpu(), table[x.astype(np.int64)]), kind
            assert torch.all(out[u:].cpu() == 7)
        assert {k: st[k] for k in want} == want, kind
        assert {k: v for k, v in ctx.totals().items() if k in want} == want
    cache.close()
