"""Build the C-ABI library paper_2411_00915_amd/liblora_amd.so for gfx950.

hipcc cross-compiles without a GPU.  The packed-fp32 VALU forms are switched
off for all device code (some of their forms have produced wrong results on the
target machines).
"""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "liblora_amd.so")
# the extension module of the Python calls (no GPU code), named for the interpreter whose ABI it is compiled for
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
OBJ_DIR = os.path.join(HERE, "_build")

SOURCES = ["planner.cpp", "kernels_general.hip", "kernels_tiled.hip", "kernels_stream.hip", "kernels_gemm.hip", "kernels_gemm_small.hip", "kernels_gemm_mid.hip", "kernels_any.hip", "abi.hip", "timing.hip", "probe.hip"]

HIP_FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-Wall", "-Wno-unused-function",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
HOST_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-Wall"]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, src + ".o")
    path = os.path.join(CSRC, src)
    if src.endswith(".hip"):
        cmd = ["hipcc", "-c", path, "-o", obj] + HIP_FLAGS
        if src in NO_SCRATCH:
            cmd.append("-Rpass-analysis=kernel-resource-usage")
    else:
        cmd = ["g++", "-c", path, "-o", obj] + HOST_FLAGS
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{res.stdout}\n{res.stderr}")
    noise = "'-packed-fp32-ops' is not a recognized feature"
    lines = [l for l in res.stderr.splitlines() if noise not in l]
    if src in NO_SCRATCH:
        _check_no_scratch(src, lines, NO_SCRATCH[src])
        lines = _without_remarks(lines)
    err = "\n".join(lines).strip()
    if err:
        sys.stderr.write(err + "\n")
    return obj


# Kernels that count their outstanding loads by hand (s_waitcnt vmcnt(n) written out next to loads issued from
# inline assembly): a register spill would put scratch loads and stores, which the same counter counts, between
# them.  The build fails if the compiler reports scratch use or spills for one of them.
NO_SCRATCH = {"kernels_gemm.hip": ("gemm_ring_kernel",), "kernels_gemm_small.hip": ("gemm_small_kernel", "layer_small_kernel"),
              "kernels_gemm_mid.hip": ("gemm_mid_kernel", "gemm_narrow_kernel", "gemm_wide_kernel"), "kernels_any.hip": ("shrink_rows_kernel",)}
REMARK = "[-Rpass-analysis=kernel-resource-usage]"


def _without_remarks(lines):
    """stderr without the resource remarks and the source lines echoed under them"""
    import re
    return [l for l in lines
            if REMARK not in l and not re.match(r"^\s*(\d+\s*)?\|", l) and not re.match(r"^\d+ remarks? generated", l)]


def _check_no_scratch(src, lines, kernels):
    current, seen = None, set()
    for l in lines:
        if REMARK not in l:
            continue
        text = l.split("remark:", 1)[1].replace(REMARK, "").strip()
        if text.startswith("Function Name:"):
            current = text.split(":", 1)[1].strip()
            continue
        if current is None or not any(k in current for k in kernels):
            continue
        for field in ("ScratchSize [bytes/lane]", "VGPRs Spill", "SGPRs Spill"):
            if text.startswith(field + ":"):
                seen.add(current)
                if int(text.rsplit(":", 1)[1]) != 0:
                    raise RuntimeError(f"{src}: {current} must not use scratch memory, but the compiler reports {text}")
    if not seen:
        raise RuntimeError(f"{src}: no resource report for {kernels}: cannot check that they use no scratch memory")


def _build_calls():
    untagged = os.path.join(HERE, "_calls.so")         # (any interpreter would load it, whatever it was compiled for)
    if os.path.exists(untagged):
        os.remove(untagged)
    subprocess.check_call(["g++", os.path.join(CSRC, "calls.cpp"), "-o", CALLS, "-shared", "-pthread",
                           "-I" + sysconfig.get_paths()["include"]] + HOST_FLAGS)


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        calls = ex.submit(_build_calls)
        objs = list(ex.map(_compile, SOURCES))
        calls.result()
    cmd = ["hipcc", "-shared", "-fPIC", "--offload-arch=gfx950", "-o", OUT] + objs
    subprocess.check_call(cmd)
    if verbose:
        print(OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
