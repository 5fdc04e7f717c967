"""The device memory pool without a GPU: compiled for the host over an allocator of its own that counts, runs out of
memory and refuses to wait on demand."""
import glob
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2305_03152_amd", "csrc")
SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include "spp_pool.h"
static std::map<void*, size_t> live;
static size_t held = 0, limit = (size_t)1 << 40;
static hipError_t waits = hipSuccess;
static int refuse = 0;                   // allocations that fail although there is room: another thread is about to make it
hipError_t hipMalloc(void** p, size_t n) {
    if (refuse > 0 || held + n > limit) {
        if (refuse > 0) --refuse;
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    *p = malloc(1);
    live[*p] = n;
    held += n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!live.count(p)) { puts("freed twice"); exit(2); }
    held -= live[p];
    live.erase(p);
    free(p);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return waits; }
using namespace spp;
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main(int, char** argv) {
    const size_t MB = (size_t)1 << 20;
    void *a, *b, *c;
    pool_context(0, 1);
    if (!strcmp(argv[1], "kept")) {              // what is retired serves the next request of its size, and no smaller one's
        CHECK(pool_take(0, &a, 100 * MB) == hipSuccess && held == 100 * MB);
        void* const was = a;
        pool_retire(0, {a, nullptr});
        CHECK(held == 100 * MB);
        CHECK(pool_take(0, &b, 50 * MB) == hipSuccess && b != was && held == 150 * MB);
        CHECK(pool_take(0, &c, 100 * MB) == hipSuccess && c == was && held == 150 * MB);
        pool_retire(0, {b, c});
    } else if (!strcmp(argv[1], "refused wait")) {       // memory that may be in use is not kept
        CHECK(pool_take(0, &a, 100 * MB) == hipSuccess && pool_take(0, &b, 10 * MB) == hipSuccess);
        waits = hipErrorStreamCaptureUnsupported;
        pool_retire(0, {a, b});
        CHECK(held == 0);
        waits = hipSuccess;
    } else if (!strcmp(argv[1], "bound")) {
        void* q[20];
        for (void*& p : q) CHECK(pool_take(0, &p, 100 * MB) == hipSuccess);
        for (void* p : q) pool_retire(0, {p});
        CHECK(held == 1000 * MB);                        // ten fit 1 GiB
    } else if (!strcmp(argv[1], "runs out")) {           // the pool gives way to any allocation of the library
        CHECK(pool_take(0, &a, 600 * MB) == hipSuccess);
        pool_retire(0, {a});
        limit = 1000 * MB;
        CHECK(device_malloc(&b, 500 * MB) == hipSuccess && held == 500 * MB);
        CHECK(device_malloc(&c, 600 * MB) == hipErrorOutOfMemory);       // nothing left to give
        CHECK(pool_take(0, &a, 400 * MB) == hipSuccess);
        pool_retire(0, {a});
        CHECK(pool_take(0, &a, 500 * MB) == hipSuccess && held == 1000 * MB);      // also to its own, of another size
        pool_retire(0, {a});
        hipFree(b);
    } else if (!strcmp(argv[1], "emptied by another")) {         // between the allocation that fails and the look at the pool
        refuse = 1;
        CHECK(device_malloc(&a, 500 * MB) == hipSuccess);
        hipFree(a);
    } else if (!strcmp(argv[1], "trimmed")) {
        CHECK(pool_take(0, &a, 600 * MB) == hipSuccess && pool_take(0, &b, 10 * MB) == hipSuccess);
        pool_retire(0, {a});
        pool_trim(0);
        CHECK(held == 10 * MB);                          // what is in use stays
        pool_retire(0, {b});
        CHECK(held == 10 * MB);
    } else {
        return 3;
    }
    pool_context(0, -1);                         // the last context gives everything back
    CHECK(held == 0);
    CHECK(pool_take(0, &a, MB) == hipSuccess);
    pool_retire(0, {a});                         // and what is retired later is not kept
    CHECK(held == 0);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("memory_pool")
    (d / "pool.cpp").write_text(SOURCE)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__=1", "-I", os.path.join(rocm, "include"), "-I", CSRC,
                           "-o", str(d / "pool"), str(d / "pool.cpp"), "-x", "c++", os.path.join(CSRC, "spp_pool.hip"), "-pthread"])
    return str(d / "pool")


@pytest.mark.parametrize("case", ["kept", "refused wait", "bound", "runs out", "emptied by another", "trimmed"])
def test_pool(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_every_allocation_can_empty_the_pool():
    """No file of the library but the pool's own calls hipMalloc, which would fail while the pool holds the memory."""
    for path in glob.glob(os.path.join(CSRC, "*")):
        if os.path.basename(path) != "spp_pool.hip":
            code = re.sub(r"//.*|\"[^\"\n]*\"", "", open(path).read())
            assert not re.search(r"\bhipMalloc\w*\s*\(", code), path
