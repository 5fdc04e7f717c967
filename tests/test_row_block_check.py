"""What the read-back of the row-block layout accepts (no GPU): the functions that it is made of, compiled for the
host, over a small graph's words as they should be and with one mistake planted in them."""
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2305_03152_amd", "csrc")
SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>
#define __device__
#define __forceinline__ inline
#include "spp_edges.h"
using namespace spp;
struct Edge { uint32_t v, u; };
int main(int argc, char** argv) {
    const char* mistake = argv[1];
    const uint32_t N = 300000, rows_per = 1u << kTileRowBits;            // two source chunks, nineteen row blocks
    const uint32_t nrb = (N + rows_per - 1) / rows_per, nch = (N + (1u << kTileSrcLoBits) - 1) >> kTileSrcLoBits;
    srand(7);
    std::vector<Edge> csr;                                               // row by row
    for (uint32_t v = 0; v < N; v += 1 + rand() % 40)
        for (int k = rand() % 6; k > 0; --k) csr.push_back({v, (uint32_t)(((uint64_t)rand() * 2048 + rand() % 2048) % N)});
    unsigned long long want = 0, got = 0;
    for (const Edge& e : csr) edge_mix(want, e.v, e.u);
    // the layout: per block and source chunk the edges' words in CSR order
    std::vector<std::vector<uint32_t>> words(nrb * nch);
    for (const Edge& e : csr)
        words[(e.u >> kTileRowBits) * nch + (e.v >> kTileSrcLoBits)].push_back(
            ((e.v & ((1u << kTileSrcLoBits) - 1)) << kTileRowBits) | (e.u & kTileRowMask));
    std::vector<uint32_t>& w = words[5 * nch];                           // a run with hundreds of edges
    const size_t i = w.size() / 2;
    if (w.size() < 100) return 3;
    size_t j = i + 1;
    while (w[j] >> kTileRowBits == w[i] >> kTileRowBits) ++j;            // the next edge of another source
    if (!strcmp(mistake, "order")) { const uint32_t t = w[i]; w[i] = w[j]; w[j] = t; }
    else if (!strcmp(mistake, "source")) w[i] += 1u << kTileRowBits;     // the neighbouring source, same chunk
    else if (!strcmp(mistake, "one source")) w[i] = (w[j] & ~kTileRowMask) | (w[i] & kTileRowMask);
    else if (!strcmp(mistake, "row")) w[i] ^= 1u;
    else if (!strcmp(mistake, "twice")) w[i] = w[i - 1];
    else if (!strcmp(mistake, "beyond")) words[(nrb - 1) * nch + nch - 1].back() |= kTileRowMask;
    else if (!strcmp(mistake, "chunk")) { words[5 * nch + 1].insert(words[5 * nch + 1].begin(), w.back()); w.pop_back(); }
    else if (strcmp(mistake, "none")) return 4;
    bool ok = true;
    for (uint32_t b = 0; b < nrb; ++b)
        for (uint32_t c = 0; c < nch; ++c) {
            const std::vector<uint32_t>& x = words[b * nch + c];
            const uint32_t rows = N - b * rows_per < rows_per ? N - b * rows_per : rows_per;
            for (size_t p = 0; p < x.size(); ++p) {
                ok = ok && tile_word_ok(x[p], x[p ? p - 1 : p], (int)c, N, rows);
                edge_mix(got, tile_source(x[p], (int)c), b * rows_per + (x[p] & kTileRowMask));
            }
        }
    printf("%d\n", ok && got == want ? 1 : 0);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("check")
    (d / "check.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(d / "check.cpp"), "-o", str(d / "check")], check=True)
    return str(d / "check")


@pytest.mark.parametrize("mistake,accepted", [("none", True), ("order", False), ("source", False), ("one source", False), ("row", False),
                                              ("twice", False), ("beyond", False), ("chunk", False)])
def test_the_read_back(program, mistake, accepted):
    r = subprocess.run([program, mistake], check=True, capture_output=True, text=True)
    assert r.stdout.strip() == ("1" if accepted else "0")


def test_the_sums_come_from_the_csr_and_from_the_words():
    """The pass that places the edges forms neither of the two sums that are compared."""
    parts = re.split(r"__global__ void (?:__launch_bounds__\([^)]*\) )?(\w+)\(", open(os.path.join(CSRC, "spp_graph.hip")).read())
    assert {name for name, body in zip(parts[1::2], parts[2::2]) if "edge_mix(" in body} == {"csr_mix_kernel", "tile_verify_kernel"}
