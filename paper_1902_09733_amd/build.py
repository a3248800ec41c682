"""Build libbpstereo.so (HIP, gfx950) in-tree.

Every source under csrc/ is compiled by hipcc for gfx950 with packed-FP32
instructions disabled, then linked into paper_1902_09733_amd/libbpstereo.so.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(ROOT, "_build", "obj")
LIB = os.path.join(HERE, "libbpstereo.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-Wall",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# The half-sweep kernels' minimum operations see no NaN (costs and messages
# are finite or +inf), so they need no NaN-quieting of their operands.
EXTRA = {
    "bp_iter_pm.hip": ["-fno-honor-nans"],
    "bp_iter_pm2_f32.hip": ["-fno-honor-nans"],
    "bp_iter_pm2_f16.hip": ["-fno-honor-nans"],
    "bp_iter_pm2_bf16.hip": ["-fno-honor-nans"],
    "bp_iter_stream_f32.hip": ["-fno-honor-nans"],
    "bp_iter_stream_f16.hip": ["-fno-honor-nans"],
    "bp_iter_stream_bf16.hip": ["-fno-honor-nans"],
}


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    flags = FLAGS + EXTRA.get(os.path.basename(src), [])
    cmd = [HIPCC] + flags + ["-c", src, "-o", obj]
    if src.endswith(".cpp"):
        cmd = [HIPCC] + flags + ["-x", "hip", "-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    if verbose and r.stderr.strip():
        print(r.stderr, file=sys.stderr)
    return obj


def build(verbose: bool = False, jobs: int | None = None) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sources()
    jobs = jobs or min(len(srcs), os.cpu_count() or 4)
    with cf.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
