"""Build the C-ABI library ``libpod_attn.so`` for gfx950 with hipcc (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpod_attn.so")
SOURCES = ["pod_kernels.hip", "pod_probe.hip", "pod_planner.cpp", "pod_api.cpp"]
# (source, extra flags) of every object: the kernels are compiled once per 16-bit type and head_dim
UNITS = ([("pod_kernels.hip", (f"-DPOD_INSTANCE_DT={dt}", f"-DPOD_INSTANCE_D={d}")) for dt in (0, 1) for d in (128, 256, 64)]
         + [(src, ()) for src in SOURCES])
HEADERS = ["pod_common.h", "pod_launch.h", "pod_planner.h", os.path.join("..", "..", "include", "pod_attn.h")]
# Packed-fp32 instructions are switched off for the device pass (the host pass does not know
# the feature and says so; that message is harmless).  The compiler's rewriting of atomics is
# switched off too: every counter update here is already issued by one lane, so the rewrite would only add
# a lane count and a read-back around each of them.
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
               "-Wall", "-Wno-unused-function", "-Wno-inline-asm"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    built = os.path.getmtime(LIB)
    return any(os.path.getmtime(os.path.join(CSRC, f)) > built for f in SOURCES + HEADERS)


def build(force: bool = True, extra_flags=(), verbose: bool = False) -> str:
    """Compile the library; returns its path.  With force=False only when sources are newer."""
    if not force and not is_stale():
        return LIB
    noise = "is not a recognized feature for this target"

    def run(cmd):
        proc = subprocess.run(cmd, capture_output=True, text=True)
        log = "\n".join(l for l in (proc.stdout + proc.stderr).splitlines() if noise not in l)
        if proc.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + log)
        return log

    with tempfile.TemporaryDirectory() as work, ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
        objects = [os.path.join(work, f"{i}.o") for i in range(len(UNITS))]
        logs = list(pool.map(lambda u: run([hipcc(), *HIPCC_FLAGS, *extra_flags, *u[0][1], "-c",
                                            os.path.join(CSRC, u[0][0]), "-o", u[1]]), zip(UNITS, objects)))
        tmp = LIB + f".tmp{os.getpid()}"
        logs.append(run([hipcc(), "--offload-arch=gfx950", "-shared", *objects, "-o", tmp]))
    log = "\n".join(l for l in logs if l.strip())
    if verbose and log:
        print(log, file=sys.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
