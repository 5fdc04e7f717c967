"""GPU: the general propagation's hops that walk the whole CSR tile by tile (frontiers with at least half of the edges),
where tiles, rows and row blocks end, against the CPU oracle and against the walk over a listed frontier, which
the same call takes when its probabilities are not aligned for 128-bit loads; and which of the two a call takes."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
TILE = 4096


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


def _graph(rng, N, deg):
    """Rows of the given lengths, their entries ascending and distinct."""
    rp = np.zeros(N + 1, dtype=np.int64)
    np.cumsum(deg, out=rp[1:])
    start = rng.integers(0, N, N)
    step = rng.integers(1, np.maximum(N // np.maximum(deg, 1), 1) + 1)
    within = np.arange(rp[-1]) - np.repeat(rp[:-1], deg)
    col = (np.repeat(start, deg) + within * np.repeat(step, deg)) % N
    order = np.lexsort((col, np.repeat(np.arange(N), deg)))
    return rp, col[order].astype(np.int32)


def _cases():
    for M in (1, 3, 255, TILE - 1, TILE, TILE + 1, 9 * TILE - 5, 9 * TILE, 16 * TILE + 257):
        yield f"spread{M}", 20000, M, None
    yield "hubs", 40000, 0, {5: 20000, 6: 1, 7: 3 * TILE, 8000: TILE, 39999: TILE + 1}
    yield "empty", 60000, 0, {0: 10, 30000: 2000, 59000: 7000}           # tens of thousands of empty rows inside a tile
    yield "gaps", 60000, 0, {0: 3000, 25000: 3000, 50000: 3000}          # fewer, which are looked at one by one
    yield "single", 70 * 16384 + 3, -1, None                             # one edge per row: 4096 rows a tile, 71 row blocks
    yield "most_blocks", 1 << 23, -1, None                               # 512 row blocks


@pytest.mark.parametrize("name,N,M,rows", list(_cases()), ids=lambda x: x if isinstance(x, str) else "")
def test_whole_hops(spp, ctx, name, N, M, rows):
    print("[case]", name, flush=True)
    rng = np.random.default_rng(N + (M or 0))
    deg = np.zeros(N, dtype=np.int64)
    if rows:
        for v, d in rows.items():
            deg[v] = d
    elif M < 0:
        deg[:] = 1
    else:
        deg += np.bincount(rng.integers(0, N, M), minlength=N)
    rp, col = _graph(rng, N, deg)
    p0 = rng.random(N).astype(np.float32)
    p0[rng.random(N) < 0.1] = 0.0
    p0[rng.random(N) < 0.01] = 1.0
    p0[deg >= TILE] = 0.5                                                # the hubs are in the frontier
    t = [(rng.random(col.size) ** 2).astype(np.float32) for _ in range(2)]
    for a in t:
        a[rng.random(a.size) < 0.02] = 1.0
        a[rng.random(a.size) < 0.02] = 0.0
    dev = torch.device("cuda:0")
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True)
    ref_t, ref_h = oracle.vip_general(rp, col, p0, t, 2)
    both = []
    for shift in (0, 1):                                                 # 1: from the list
        td = [torch.zeros(a.size + 4, device=dev)[shift:shift + a.size].copy_(torch.from_numpy(a)) for a in t]
        p, ph = spp.vip_propagate_general(ctx, G, torch.from_numpy(p0).to(dev), td, 2, per_hop=True)
        for got, ref in ((p, ref_t), (ph, ref_h)):
            # a term's logarithm carries a few units of fp32, all terms have one sign, and the second hop starts from
            # probabilities rounded to fp32: the 1e-5 that the entry point states
            assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= 1e-5 * np.asarray(ref) + 1e-37), (name, shift)
        both.append(ph)
    G.close()
    # The two form the same fp32 terms and add them up in fp64 in different orders: the first hop's results are rounded to
    # fp32 from sums that differ by 1e-15 (a unit in the last place at most, 1.2e-7), the second starts from those.
    apart = ((both[0] - both[1]).abs() / both[1].clamp(min=1e-37)).amax(dim=1).tolist()
    assert apart[0] <= 1.2e-7 and apart[1] <= 3.6e-7, (name, apart)


def test_one_term_per_vertex(spp, ctx):
    """A vertex with one in-edge has its term as its sum: the two forms give the same bits, and p = 1 - exp(log(1 - x)) is x
    again.  A term of 2.4 units in the last place (1.4e-7) and the rounding of p below 1/4; above, 1 - x rounded by 3e-8
    and the term again, over x >= 1/4: 6e-7 covers both."""
    N = 1 << 20
    rp, col = np.arange(N + 1, dtype=np.int64), ((np.arange(N) + 7) % N).astype(np.int32)
    rng = np.random.default_rng(3)
    x = np.where(rng.random(N) < 0.5, rng.random(N), np.exp(-60 * rng.random(N))).astype(np.float32)
    x[:4] = 0.25, np.nextafter(np.float32(0.25), np.float32(0)), np.nextafter(np.float32(1), np.float32(0)), 1.0
    dev = torch.device("cuda:0")
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True)
    p0 = torch.ones(N, device=dev)
    got = []
    for shift in (0, 1):
        t = torch.zeros(N + 4, device=dev)[shift:shift + N].copy_(torch.from_numpy(x))
        got.append(spp.vip_propagate_general(ctx, G, p0, t, 1))
    G.close()
    assert torch.equal(got[0], got[1])
    want = np.roll(x.astype(np.float64), 7)
    assert np.all(np.abs(got[0].cpu().numpy() - want) <= 6e-7 * want)


@pytest.mark.parametrize("frontier,shift,form", [(1.0, 0, "tiles"), (0.6, 0, "tiles"), (0.02, 0, "list"), (1.0, 1, "list")])
@pytest.mark.parametrize("N", [500_000, 5_000_000])
def test_which_form_a_call_takes(spp, ctx, N, frontier, shift, form):
    """By the kernels that a call launches and which of them do the work: the walk by tiles fills the bins in the launch that
    lists the frontier otherwise, and the listed fill then leaves at once."""
    dev = torch.device("cuda:0")
    deg = 12
    rp = torch.arange(N + 1, dtype=torch.int64, device=dev) * deg
    col = ((torch.arange(N, device=dev).unsqueeze(1) + torch.arange(1, deg + 1, device=dev) * (N // 13)) % N).sort(1).values.to(torch.int32).reshape(-1)
    G = spp.Graph(ctx, rp, col, in_lists=True)
    p0 = (torch.rand(N, generator=torch.Generator(dev).manual_seed(1), device=dev) < frontier).float()
    t = torch.full((N * deg + 4,), 0.5, device=dev)[shift:shift + N * deg]
    spp.vip_propagate_general(ctx, G, p0, t, 1)
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        spp.vip_propagate_general(ctx, G, p0, t, 1)
        torch.cuda.synchronize()
    G.close()
    took = {name: sum(e.device_time_total for e in prof.key_averages() if name in e.key)
            for name in ("vipg_prepare_kernel", "vip_frontier_list_kernel", "vipg_bin_fill_kernel")}
    print("[took]", N, frontier, shift, took)
    prepare, listing, fill = took.values()
    assert fill > 0 and (prepare > 0) == (shift == 0) and (listing > 0) == (shift == 1), took
    assert fill < prepare / 2 if form == "tiles" else fill > prepare, took


def test_a_probability_that_nothing_uses_is_not_reported(spp, ctx):
    N = 3 * TILE
    rp, col = np.arange(N + 1, dtype=np.int64), ((np.arange(N) + 7) % N).astype(np.int32)
    p0, t = np.full(N, 0.5, np.float32), np.full(N, 0.25, np.float32)
    p0[100], t[100] = 0.0, 2.0
    dev = torch.device("cuda:0")
    G = spp.Graph(ctx, torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev), in_lists=True)
    got = spp.vip_propagate_general(ctx, G, torch.from_numpy(p0).to(dev), torch.from_numpy(t).to(dev), 1).cpu().numpy()
    want = np.where(np.arange(N) == 107, 0.0, 0.125)
    assert np.all(np.abs(got - want) <= 1e-6 * want)       # log1p and expm1 of one term: a few units of fp32
    for wrong in (2.0, -0.5, float("nan")):
        t[200] = wrong
        with pytest.raises(spp.SppError):
            spp.vip_propagate_general(ctx, G, torch.from_numpy(p0).to(dev), torch.from_numpy(t).to(dev), 1)
    G.close()
