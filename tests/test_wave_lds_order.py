"""Kernels whose lanes hand counts to the other lanes of their wavefront through LDS, with no barrier between: every such
step has to be ordered for the compiler by a fence at the wavefront's scope (the hardware keeps the order by itself, and no
instruction comes of it).  Counted in the compiler's intermediate code of this repository's own sources."""
import os
import re
import subprocess

import pytest

from paper_2305_03152_amd import build

# per 64 entries: the lanes read a count before one of them stores it anew, and store it before the next 64 are counted
EXPECTED = {
    "spp_radix.hip": {r"radix_mid_scatter_kernelILi2E": 1 + 2 * 2,       # once more: the counts are emptied by other lanes
                      r"radix_mid_scatter_kernelILi4E": 1 + 2 * 4,
                      r"radix_scatter_kernelILi1024E": 2 * 4, r"radix_scatter_kernelILi4096E": 2 * 16},
    "spp_graph.hip": {r"part_place_kernelILi8E": 2 * 4 * 2, r"part_place_kernelILi9E": 2 * 4 * 2},     # full tiles, the last one
    "spp_sample.hip": {r"hop_sample_kernelILi\d+E": 2},                  # in a loop
    "spp_vip.hip": {r"vip_bin_finish_kernelE": 4,                        # around a packed batch's reads, its writes, before the last pass
                    r"vip_hop_kernelE": 2},                              # a window of y is written, and has been read
}


@pytest.mark.parametrize("source", sorted(EXPECTED))
def test_counts_handed_on_in_a_wavefront_are_ordered(source, tmp_path):
    ir = tmp_path / "k.ll"
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", "-emit-llvm", os.path.join(build.CSRC, source), "-o", ir],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    bodies = dict(re.findall(r"^define [^@\n]*amdgpu_kernel[^@\n]*@(\w+)\([^\n]*\n(.*?)^}", ir.read_text(), re.S | re.M))
    for name, least in EXPECTED[source].items():
        found = {k: len(re.findall(r'fence syncscope\("wavefront"\)', body)) for k, body in bodies.items() if re.search(r"\d" + name, k)}
        assert found and all(n >= least for n in found.values()), (name, least, found)
