"""Build libmrpie.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import glob
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libmrpie.so")
BUILD = os.path.join(ROOT, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17",
    # no packed-FP32 instructions anywhere in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-munsafe-fp-atomics",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# Per-file flags.  The sweep's single-job kernels take their job as leading
# scalar arguments; preloading them into SGPRs (gfx950) saves the
# kernel-argument fetch at the start of every launch.
FILE_FLAGS = {
    "sweep.hip": ["-mllvm", "-amdgpu-kernarg-preload-count=16"],
    "sweep_sp.hip": ["-mllvm", "-amdgpu-kernarg-preload-count=16"],
    "team.hip": ["-save-temps=obj"],  # its assembly is looked over below
}


def lost_copies(asm: str, functions: str) -> list:
    """Places in the assembly of the functions whose name matches `functions`
    where vector instructions stand at the head of the block that ends a
    divergent branch, before all lanes are switched on again: (function,
    block, instruction).

    The register allocator has put copies of values that are live across such
    a branch there (a long-lived value moved to make room); lanes that did not
    take the branch lose them.  The persistent sweep keeps its phases free of
    divergent branches for that reason, and its wrong results or addresses
    would show on the GPU only, so the build looks for the pattern."""
    found, fn, block, pending = [], "", "", []
    for line in asm.splitlines():
        label = re.match(r"(_Z\S+|\.LBB\S+):|; %bb\.\d+", line)
        if label:
            fn = label.group(1) if line.startswith("_Z") else fn
            block, pending = line.split()[0], []
        elif re.match(r"\s+s_or_b64 exec, exec,", line):
            if re.search(functions, fn):
                found += [(fn, block, i) for i in pending]
            pending = []
        elif re.match(r"\s+(v_(?!readlane|writelane)|(ds|global|scratch|flat|buffer)_)", line):  # (those two take any lane)
            pending.append(line.strip())
    return found


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [HIPCC, *FLAGS, *FILE_FLAGS.get(os.path.basename(src), []), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    if os.path.basename(src) == "team.hip":
        with open(os.path.join(BUILD, "team-hip-amdgcn-amd-amdhsa-gfx950.s")) as f:
            lost = lost_copies(f.read(), r"member_job|6k_team")
        if lost:
            raise RuntimeError("team.hip: copies before the lanes of a divergent branch come back:\n"
                               + "\n".join(map(str, lost[:8])))
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = OUT + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
