"""A traffic record is dropped once the sources of the kernels it was taken with change: the list must name all of them."""
import os
import re

import bench


def test_every_gemm_source_counts():
    csrc = "paper_2002_12798_amd/csrc"
    for f in os.listdir(os.path.join(bench.ROOT, csrc)):
        if f.startswith("amap_gemm"):
            assert f"{csrc}/{f}" in bench.GEMM_SOURCES, f
    for files in (bench.GEMM_SOURCES, bench.MAP_SOURCES):
        for f in files:
            text = open(os.path.join(bench.ROOT, f)).read()
            for inc in re.findall(r'#include "(amap_gemm\w*\.hpp)"', text):
                assert f"{csrc}/{inc}" in files, (f, inc)
