"""GPU: propagations recorded into a graph, from a context's first call on: one that is recorded and not run leaves a context
on which the next call is right, and every replay gives what an eager call gives, with eager calls in between."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spp():
    import paper_2305_03152_amd as m
    m.load_library()
    return m


def _leave_dirty_memory():
    """Small blocks of device memory full of ones go back to the runtime, which hands such blocks out again as they are."""
    hip = C.CDLL("libamdhip64.so")
    blocks = []
    for size in (65664, 65920, 66304, 70000, 74250):
        for _ in range(24):
            p = C.c_void_p()
            assert hip.hipMalloc(C.byref(p), C.c_size_t(size)) == 0
            assert hip.hipMemset(p, C.c_int(255), C.c_size_t(size)) == 0
            blocks.append(p)
    assert hip.hipDeviceSynchronize() == 0
    for p in blocks:
        assert hip.hipFree(p) == 0


@pytest.mark.parametrize("kind", ["blocks", "chunked", "general"])
def test_recorded_before_any_call_has_run(spp, kind):
    N, d = 10_000, 10
    rp = torch.arange(N + 1, dtype=torch.int64, device="cuda") * d
    col = ((torch.arange(N, device="cuda").unsqueeze(1) + torch.arange(1, d + 1, device="cuda")) % N).sort(1).values.to(torch.int32).reshape(-1)
    T = torch.arange(300, dtype=torch.int32, device="cuda")
    p0 = torch.linspace(0, 1, N, device="cuda")
    t = torch.linspace(1, 0, N * d, device="cuda")

    def call(ctx, G, sync):
        if kind == "general":
            return spp.vip_propagate_general(ctx, G, p0, t, 2, sync=sync)
        return spp.vip_propagate(ctx, G, T, 64, (3, 2, 4), sync=sync)

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        torch.cuda.synchronize()
        ref_ctx = spp.Context(0)
        want = call(ref_ctx, spp.Graph(ref_ctx, rp, col, in_lists=True, chunked=kind == "chunked"), True)
        _leave_dirty_memory()
        ctx = spp.Context(0)
        G = spp.Graph(ctx, rp, col, in_lists=True, chunked=kind == "chunked")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):     # workspaces are allocated on the way
            recorded = call(ctx, G, False)
        for k in range(4):
            # the sums of a vertex may be added up in another order: the last bit of a result
            print("[case]", kind, k, flush=True)
            assert torch.allclose(call(ctx, G, True), want, rtol=3e-7, atol=0)
            recorded.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.allclose(recorded, want, rtol=3e-7, atol=0)
        ctx.close()
        ref_ctx.close()
