"""GPU: a CSR that does not describe M edges of N vertices is refused, whichever pass validates it (the one of a graph
without lists, the chunked layout's, and the two that build the row blocks), and the next graph is built as ever."""
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


@pytest.mark.parametrize("flags", [dict(in_lists=False), dict(in_lists=True), dict(in_lists=True, chunked=True)], ids=["plain", "blocks", "chunked"])
@pytest.mark.parametrize("N", [5, 9000, 40000])
def test_what_is_refused(spp, ctx, N, flags):
    deg = 3
    rp = np.arange(N + 1, dtype=np.int64) * deg
    col = np.sort((np.arange(N)[:, None] + np.arange(1, deg + 1)) % N, axis=1).astype(np.int32).ravel()
    M = col.size

    def make(rp, col):
        return spp.Graph(ctx, torch.from_numpy(rp).cuda(), torch.from_numpy(col).cuda(), **flags)

    def changed(a, at, value):
        a = a.copy()
        a[at] = value
        return a

    wrong = [(changed(rp, 0, 1), col), (changed(rp, N, M - 1), col), (changed(rp, N, M + 5), col),           # the ends
             (changed(rp, N // 2, 0), col), (changed(rp, N // 2, M + 1), col), (changed(rp, 1, -1), col),      # not monotone
             (rp, changed(col, 0, N)), (rp, changed(col, M - 1, -1)), (rp, changed(col, M // 2, 0x7FFFFFFF))]  # ids
    for i, (r, c) in enumerate(wrong):
        print("[case]", N, flags, i, flush=True)
        with pytest.raises(spp.SppError, match="rowptr"):
            make(r, c)
    make(rp, col).close()
