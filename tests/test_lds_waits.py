"""The GEMM kernels that refill LDS with loads from inline assembly write their barriers and waits out by hand
(kernels_gemm.hip, kernels_gemm_mid.hip): one wavefront's loads may overwrite what another has only asked to read.  Their
arguments rest on one rule -- a wavefront's LDS reads have returned before the second barrier after them, i.e. by the end
of the matrix part that follows the memory part they were issued in; where a stage is one memory and one matrix part (the
medium GEMM with k-steps apart, tiles of 64 features always), before the first, i.e. by the end of that memory part, because
the leading wavefronts refill the stage in the next -- and the order in which the compiler puts its own waits does not promise
it.  The rule is checked here on the assembly of the kernels, as the compiler emits it."""
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


def _late_reads(lines, barriers):
    """LDS reads that may still be on their way when so many barriers after them are passed.  LDS operations return in
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
            late += [p[0] for p in pending if p[1] == barriers and p[0].startswith("ds_read")]
    return late


def test_late_reads_are_found():
    read, wait, other, barrier = "ds_read_b128 v[0:3], v4", "s_waitcnt lgkmcnt(0)", "v_mfma_f32_16x16x32_bf16", "s_barrier"
    for lines, late in (([read, wait, barrier, barrier], (0, 0)), ([read, barrier, wait, other, barrier], (1, 0)),
                        ([read, read, "s_waitcnt lgkmcnt(1)", barrier, wait, barrier], (1, 0)), ([read, barrier, other, barrier], (1, 1)),
                        ([read, "s_waitcnt vmcnt(0)", barrier, barrier, wait], (1, 1)), ([barrier, read, wait, barrier, "ds_write_b128 v4, v[0:3]", barrier], (0, 0))):
        assert tuple(len(_late_reads(lines, n)) for n in (1, 2)) == late, lines


def _check(kernels, barriers, least_reads, least_barriers):
    for symbol, lines in kernels.items():
        assert sum(l.startswith("ds_read") for l in lines) >= least_reads and sum(l.startswith("s_barrier") for l in lines) >= least_barriers, symbol
        late = _late_reads(lines, barriers)
        assert not late, f"{symbol}: {len(late)} LDS reads not waited for, first: {late[0]}"


def test_lds_reads_of_the_ring_return_before_the_second_barrier_after_them(tmp_path):
    kernels = _kernels("kernels_gemm.hip", "gemm_ring_kernel", tmp_path)
    assert len(kernels) == 4
    _check(kernels, 2, 21, 9)


def test_lds_reads_of_the_medium_tiles_return_before_the_barrier_their_loop_allows(tmp_path):
    """Builds of gemm_mid_kernel<WA, deltas, k-steps apart, K tail>: those with k-steps apart have one memory part to a stage"""
    kernels = _kernels("kernels_gemm_mid.hip", "gemm_mid_kernel", tmp_path)
    apart = {s: l for s, l in kernels.items() if re.search(r"row_deltaE\dELb1ELb[01]E", s)}
    assert len(kernels) == 16 and len(apart) == 4
    _check({s: l for s, l in kernels.items() if s not in apart}, 2, 21, 9)
    _check(apart, 1, 21, 9)


def test_lds_reads_of_the_narrow_tiles_return_before_the_first_barrier_after_them(tmp_path):
    """the tiles of 64 features: one memory part to a stage"""
    kernels = _kernels("kernels_gemm_mid.hip", "gemm_narrow_kernel", tmp_path)
    assert len(kernels) == 2
    _check(kernels, 1, 12, 6)


def test_lds_reads_of_the_wide_tiles_return_before_the_barrier_their_loop_allows(tmp_path):
    """the tiles of 256 features: builds <deltas, k-steps apart, K tail>"""
    kernels = _kernels("kernels_gemm_mid.hip", "gemm_wide_kernel", tmp_path)
    apart = {s: l for s, l in kernels.items() if re.search(r"row_deltaE\dELb1ELb[01]E", s)}
    assert len(kernels) == 8 and len(apart) == 2
    _check({s: l for s, l in kernels.items() if s not in apart}, 2, 21, 9)
    _check(apart, 1, 21, 9)
