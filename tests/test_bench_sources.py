"""bench.py quotes committed profiles only while the kernels' sources are those
they were taken on: its source list and kernel names cover the build's."""
import glob
import os
import re

import bench
from paper_2606_15177_amd import build


def test_layer_sources_cover_the_build():
    layer = {s for s in build.SOURCES if s not in ("place.hip", "window.hip", "moe_abi.hip")}
    assert layer <= set(bench.LAYER_SOURCES)
    for s in bench.LAYER_SOURCES:
        assert os.path.exists(os.path.join(build.CSRC, s)), s


def test_ffn_kernels_have_a_stage():
    names = [n for stage in bench.STAGE_KERNELS.values() for n in stage]
    for path in glob.glob(os.path.join(build.CSRC, "ffn_*.hip")):
        for kernel in re.findall(r"void (\w+_kernel)\(", open(path).read()):
            assert any(n.startswith(kernel) for n in names), kernel
