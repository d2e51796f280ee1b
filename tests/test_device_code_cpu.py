"""Properties of the device code that a run cannot show, read off the unoptimised intermediate code of this
repository's own sources (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2412_20379_amd import build as hip_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _functions(source, tmp_path):
    """{mangled name: text} of a device translation unit before any optimisation"""
    try:
        hipcc = hip_build._hipcc()
        out = str(tmp_path / "unit.ll")
        r = subprocess.run([hipcc, "-x", "hip", "--offload-device-only", "--offload-arch=gfx950", "-std=c++17", "-O1", "-w",
                            "-Xclang", "-disable-llvm-passes", "-emit-llvm", "-S", "-I" + os.path.join(ROOT, "include"),
                            "-I" + hip_build.CSRC, os.path.join(hip_build.CSRC, source), "-o", out], capture_output=True, text=True)
    except (RuntimeError, FileNotFoundError):
        pytest.skip("no hipcc")
    assert r.returncode == 0, r.stderr
    text = open(out).read()
    return {m.group(1): m.group(0) for m in re.finditer(r"^define [^@]*@([\w.$]+)\(.*?^}", text, re.M | re.S)}


def _events(body, **patterns):
    """the calls of interest in program order"""
    found = [(m.start(), name) for name, p in patterns.items() for m in re.finditer(p, body)]
    return [name for _, name in sorted(found)]


def test_lanes_of_a_wavefront_exchange_rows_behind_fences(tmp_path):
    """The transform's wavefronts write rows into LDS in one layout and read them in another, so a lane reads what others
    wrote.  Nothing but a fence tells the compiler to keep the two apart: before the writes (the step before has been
    read) and after them, and where the sums of strip_split_kernel take the place of its last step."""
    fns = _functions("nn_strip_kernels.hip", tmp_path)
    fence = [t for n, t in fns.items() if "lane_exchange_fence" in n]
    assert len(fence) == 1 and re.search(r'fence syncscope\("wavefront"\) acq_rel', fence[0])
    stages = [t for n, t in fns.items() if "RowStage" in n and "5stageE" in n]
    assert stages
    for body in stages:
        seen = _events(body, fence=r"call .*lane_exchange_fence", write=r"call .*store_words")
        assert seen[0] == "fence" and seen[-1] == "fence" and "write" in seen
    splits = [t for n, t in fns.items() if "18strip_split_kernel" in n or "strip_split_kernelI" in n]
    assert splits
    for body in splits:
        seen = _events(body, fence=r"call .*lane_exchange_fence", read=r"call .*RowStage.*4readE", barrier=r"call .*__syncthreads")
        last = len(seen) - 1 - seen[::-1].index("read")
        assert seen[last + 1:][:2] == ["fence", "barrier"]
