"""GPU: graphs and caches built from memory that closed ones left behind -- other sizes, several threads with a context
and a stream each -- give what freshly allocated ones give; what is kept serves the next build, stays within its bound
and goes back with the last context or on request."""
import gc
import threading

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


def _ring(N, deg):
    col = (np.arange(N, dtype=np.int64)[:, None] + np.arange(1, deg + 1)) % N
    return np.arange(N + 1, dtype=np.int64) * deg, np.sort(col, axis=1).astype(np.int32).ravel()


def _use(spp, ctx, N, deg, chunked):
    """Builds a graph and a cache, compares both with the oracle, closes both."""
    rp, col = _ring(N, deg)
    T = (np.arange(N // 50) * 3).astype(np.int32)
    g = spp.Graph(ctx, torch.from_numpy(rp).cuda(), torch.from_numpy(col).cuda(), in_lists=True, chunked=chunked)
    p = spp.vip_propagate(ctx, g, torch.from_numpy(T).cuda(), 64, (3, 2))
    ref, _ = oracle.vip(rp, col, T, 64, (3, 2))
    got = p.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= 1e-6 * np.asarray(ref) + 1e-37)      # rounded to fp32 at every hop
    remote = torch.arange((N - N // 4) * 8, dtype=torch.float32).reshape(-1, 8).pin_memory()
    cache = spp.build_vip_cache(ctx, p, 0, N // 4, 4, 0.2, remote, 8, 4)
    ids = oracle.cache_select(p.cpu().numpy(), 0, N // 4, 4, 0.2)
    assert np.array_equal(cache.ids.cpu().numpy(), ids)
    probe = torch.arange(N, dtype=torch.int32, device="cuda")
    slot = np.full(N, -1, np.int32)
    slot[ids] = np.arange(ids.size)
    assert np.array_equal(cache.lookup(probe).cpu().numpy(), slot)
    cache.close()
    g.close()


def test_memory_is_used_again(spp):
    ctx = spp.Context(0)
    for N, deg, chunked in ((40_000, 9, False), (39_000, 9, False), (40_000, 9, True), (90_001, 3, False), (40_000, 9, False)):
        print("[case]", N, deg, chunked, flush=True)
        _use(spp, ctx, N, deg, chunked)
    ctx.close()


def test_threads(spp):
    errors = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                ctx = spp.Context(0)
                for i in range(4):
                    _use(spp, ctx, 20_000 + 3000 * ((i + k) % 3), 7, False)
                ctx.close()
        except Exception as e:                # noqa: BLE001 -- reported by the test's own thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


# What the device reports free is a multiple of 2 MiB: a difference of two readings is off by less than one such step either way,
# and the runtime may hold part of a step from allocations before.  120000000 bytes (57.2 steps) have shown as 57 steps.
STEP = 2 << 20


def _free():
    """Bytes the device reports free, without what torch and handles that nothing refers to any more keep."""
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def test_what_is_kept_serves_the_next_build(spp):
    N, deg = 2_000_000, 30
    rp = torch.arange(N + 1, dtype=torch.int64, device="cuda") * deg
    col = ((torch.arange(N, device="cuda").unsqueeze(1) + torch.arange(1, deg + 1, device="cuda")) % N).sort(1).values.to(torch.int32).reshape(-1)
    ctx = spp.Context(0)
    spp.release_memory(0)
    before = _free()
    g = spp.Graph(ctx, rp, col, in_lists=True)
    built = _free()
    assert before - built >= 4 * N * deg - 2 * STEP                         # a word per edge, and what goes with it
    for _ in range(2):
        g.close()
        assert _free() == built                                             # nothing went back ...
        g = spp.Graph(ctx, rp, col, in_lists=True)
        assert _free() == built                                             # ... and nothing more was taken
    g.close()
    ctx.close()
    assert _free() >= before                                                # the last context's own buffers went with it


def test_what_is_kept_is_bounded(spp):
    ctx = spp.Context(0)
    spp.release_memory(0)
    before = _free()
    for N in (3_000_000, 4_000_000, 5_000_000, 6_000_000, 7_000_000):       # 30 edges a vertex: 360 to 840 MB, 3 GB in all
        rp = torch.arange(N + 1, dtype=torch.int64, device="cuda") * 30
        col = ((torch.arange(N, device="cuda").unsqueeze(1) + torch.arange(1, 31, device="cuda")) % N).sort(1).values.to(torch.int32).reshape(-1)
        g = spp.Graph(ctx, rp, col, in_lists=True)
        g.close()
        del rp, col, g
    assert 360 << 20 < before - _free() < (1 << 30) + (256 << 20)            # something; the bound and what the context's buffers hold
    ctx.close()


def test_what_is_kept_is_given_back_on_request(spp):
    ctx = spp.Context(0)
    N, deg = 1_000_000, 30
    rp = torch.arange(N + 1, dtype=torch.int64, device="cuda") * deg
    col = ((torch.arange(N, device="cuda").unsqueeze(1) + torch.arange(1, deg + 1, device="cuda")) % N).sort(1).values.to(torch.int32).reshape(-1)
    spp.release_memory(0)                                               # else the build may find its memory there, and takes none
    before = _free()
    spp.Graph(ctx, rp, col, in_lists=True).close()
    assert before - _free() > 4 * N * deg - 2 * STEP                    # the edges' words are kept
    spp.release_memory(0)
    assert before - _free() < 2 * N * deg
    ctx.close()
    with pytest.raises(spp.SppError):
        spp.release_memory(-1)
