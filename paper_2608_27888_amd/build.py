"""Build libntc.so (HIP, gfx950) in-tree.

    python -m paper_2608_27888_amd.build

Every ``csrc/*.hip`` source is compiled to an object of its own, in parallel
(the decode kernels are split by shape family so that no one translation unit
dominates), then the objects are linked into one shared library.  The compiler's
resource report of every kernel goes to libntc.kernels.json beside it: {source:
{mangled kernel name: {"VGPRs", "ScratchSize", "Occupancy", ...}}}.
"""
from __future__ import annotations

import glob
import json
import os
import re
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libntc.so")
KERNELS = os.path.join(HERE, "libntc.kernels.json")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 instructions stay off: plain fp32 arithmetic only
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA results in arch VGPRs: the epilogue reads them without AGPR copies
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
    "-Wall", "-Wno-unused-function",
    "-Rpass-analysis=kernel-resource-usage",
]

# Flags of single sources.  Binning: its LDS atomics come from one lane, at a
# wave-uniform address; the compiler's atomic optimizer would wrap each in a
# wave reduction that costs more than the atomic (512-decoder frame: 74 -> 66 us
# without it).
SOURCE_FLAGS = {
    "ntc_bins.hip": ["-mllvm", "-amdgpu-atomic-optimizer-strategy=None"],
}


def sources():
    return sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))


def jobs() -> int:
    n = os.cpu_count() or 4
    for var in ("MAX_JOBS", "CMAKE_BUILD_PARALLEL_LEVEL"):
        v = os.environ.get(var, "")
        if v.isdigit() and int(v) > 0:
            n = min(n, int(v))
    return max(1, min(n, 16))


def resources(report: str):
    """(resource usage by kernel, the other lines) of a compiler's stderr.  A remark is
    its line, after the include chain, then the source line and a caret line."""
    kernels, rest, includes, cur, quoted = {}, [], [], None, 0
    for line in report.splitlines():
        m = re.search(r" remark: +(.*) \[-Rpass-analysis=kernel-resource-usage\]$", line)
        if m:
            key, _, value = m[1].partition(": ")
            key = key.split(" [")[0].replace(" ", "")
            if key == "FunctionName":
                cur = kernels.setdefault(value, {})
            elif value.isdigit():
                cur[key] = int(value)
            includes, quoted = [], 2
        elif quoted and re.match(r" *\d* \| ", line):
            quoted -= 1
        elif line.startswith("In file included from "):
            includes.append(line)
        else:
            rest += includes + [line]
            includes = []
    return kernels, rest


def build(verbose: bool = False) -> str:
    inc = ["-I", os.path.join(ROOT, "include")]
    objdir = tempfile.mkdtemp(prefix="ntc_build_")
    try:
        def compile_one(src):
            obj = os.path.join(objdir, os.path.basename(src) + ".o")
            extra = SOURCE_FLAGS.get(os.path.basename(src), [])
            cmd = [HIPCC, *FLAGS, *extra, *inc, "-c", "-o", obj, src]
            if verbose:
                print(" ".join(cmd), flush=True)
            r = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
            used, messages = resources(r.stderr)
            if messages:
                print("\n".join(messages), file=sys.stderr, flush=True)
            if r.returncode:
                raise subprocess.CalledProcessError(r.returncode, cmd)
            return obj, used

        srcs = sources()
        # largest sources first: they set the critical path
        srcs.sort(key=lambda s: -os.path.getsize(s))
        with ThreadPoolExecutor(max_workers=jobs()) as pool:
            built = list(pool.map(compile_one, srcs))
        objs = [obj for obj, _ in built]
        tmp = LIB + ".tmp%d" % os.getpid()
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *sorted(objs)]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        with open(tmp + ".json", "w") as f:
            json.dump({os.path.basename(s): used for s, (_, used) in zip(srcs, built)}, f, indent=0)
        os.replace(tmp + ".json", KERNELS)
        os.replace(tmp, LIB)
    finally:
        shutil.rmtree(objdir, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
