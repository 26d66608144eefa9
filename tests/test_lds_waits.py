"""The GEMM kernels that refill LDS with loads from inline assembly write their barriers and waits out by hand
(kernels_gemm.hip, kernels_gemm_mid.hip): one wavefront's loads may overwrite what another has only asked to read.  Their
arguments rest on one rule -- a wavefront's LDS reads have returned before the second barrier after them, i.e. by the end
of the matrix part that follows the memory part they were issued in -- and the order in which the compiler puts its own
waits does not promise it.  The rule is checked here on the assembly of the kernels, as the compiler emits it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2411_00915_amd import build

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


def _kernels(src, name, tmp_path):
    """{symbol: assembly lines} of the kernels of `src` whose symbol holds `name`"""
    out = str(tmp_path / "device.s")
    subprocess.run(["hipcc", "-S", "--offload-device-only", os.path.join(build.CSRC, src), "-o", out] + build.HIP_FLAGS,
                   check=True, capture_output=True)
    kernels, current = {}, None
    with open(out) as f:
        for line in f:
            m = re.match(r"(_Z\w+):", line)
            if m and name in m.group(1):
                current = kernels.setdefault(m.group(1), [])
            elif line.startswith(".Lfunc_end"):
                current = None
            elif current is not None:
                current.append(line.split(";")[0].strip())
    return kernels


def _late_reads(lines):
    """LDS reads that may still be on their way when the second barrier after them is passed.  LDS operations return in
    order, so of those issued the youngest n may be missing after lgkmcnt(n) (scalar loads count, too, and only make the
    wait stricter)."""
    pending, late = [], []                                  # [instruction, barriers passed since]
    for line in lines:
        if line.startswith("ds_"):
            pending.append([line, 0])
        elif line.startswith("s_waitcnt"):
            n = re.search(r"lgkmcnt\((\d+)\)", line)
            if n:
                pending = pending[len(pending) - min(len(pending), int(n.group(1))):]
        elif line.startswith("s_barrier"):
            for p in pending:
                p[1] += 1
            late += [p[0] for p in pending if p[1] == 2 and p[0].startswith("ds_read")]
    return late


@pytest.mark.parametrize("src,name,builds", [("kernels_gemm.hip", "gemm_ring_kernel", 4), ("kernels_gemm_mid.hip", "gemm_mid_kernel", 16)])
def test_lds_reads_return_before_the_second_barrier_after_them(src, name, builds, tmp_path):
    kernels = _kernels(src, name, tmp_path)
    assert len(kernels) == builds
    for symbol, lines in kernels.items():
        assert sum(l.startswith("ds_read") for l in lines) > 20 and sum(l.startswith("s_barrier") for l in lines) > 8, symbol
        late = _late_reads(lines)
        assert not late, f"{symbol}: {len(late)} LDS reads not waited for, first: {late[0]}"


def test_lds_reads_of_the_narrow_tiles_return_before_the_second_barrier_after_them(tmp_path):
    """the tiles of 64 features: one memory part to a stage, so fewer reads and barriers to a kernel"""
    kernels = _kernels("kernels_gemm_mid.hip", "gemm_narrow_kernel", tmp_path)
    assert len(kernels) == 2
    for symbol, lines in kernels.items():
        assert sum(l.startswith("ds_read") for l in lines) >= 12 and sum(l.startswith("s_barrier") for l in lines) > 5, symbol
        late = _late_reads(lines)
        assert not late, f"{symbol}: {len(late)} LDS reads not waited for, first: {late[0]}"
