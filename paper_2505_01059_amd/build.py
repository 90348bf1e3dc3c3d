"""Build libmtp.so (the HIP/C++ engine) in-tree for gfx950 with hipcc."""
import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmtp.so")

SOURCES = ["kernels.hip", "rollout_line.hip", "rollout_quad.hip", "rollout_quad_gen.hip", "rollout_seg.hip",
           "rollout_wide.hip", "rollout_wide_half.hip", "rollout_wide_rest.hip", "pm_replan.hip", "plan.cpp",
           "batch.hip", "batch.cpp", "server.cpp", "plant.cpp", "noalloc.hip", "schedule_cache.cpp"]


def _sched(strategy):
    return ["-mllvm", f"-amdgpu-sched-strategy={strategy}"]


# Most kernels run one wave per SIMD, so the instruction order decides how much of
# a wave's latency shows, and each form has an order that suits it.  Launches in us
# with LLVM's default / iterative-ilp / max-ilp scheduler (values are the same):
# time-sliced 24 links in contact 2910 / 2945 / 2900; one lane, 4 links, 40000
# candidates 80 / 76 / 76, 3 links, 600, 5000 and 40000 candidates 55.3 / 55.9 / 57.0,
# 55.2 / 56.0 / 57.3 and 55.9 / 56.5 / 57.6, 2 links 38.8 / 39.4 / 39.0, 39.7 / 39.7 /
# 38.7 and 40.5 / 40.1 / 38.8; four lanes, 12 links 89 / 92 / 86; eight lanes, 24
# links 121 / 122 / 115; four lanes, 24 links in contact 748 / 760 / 762; four lanes,
# 7 links in contact, three models 168 / 161 / 168; four lanes, 4 links 55.6 / 58.0 /
# 55.9; quad lanes, 7 links 109.5 / 110.8 / 110.6, but as long as their generator
# 200 / 145 / 200 (14000 candidates, a unit of its own).  Whole point-mass replans
# 75.8 / 74.4 / 74.8 us; 256 instances batched 77.1 / 76.7 / 76.9 ms.
EXTRA_FLAGS = {
    "batch.hip": _sched("iterative-ilp"),
    "pm_replan.hip": _sched("iterative-ilp"),
    "rollout_line.hip": _sched("iterative-ilp"),
    "rollout_quad_gen.hip": _sched("iterative-ilp"),
    "rollout_seg.hip": _sched("max-ilp"),
    "rollout_wide.hip": _sched("iterative-ilp"),
    "rollout_wide_half.hip": _sched("max-ilp"),
}
HIP_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed FP32 instructions stay off: plain float code only
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def hipcc():
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def _compile(src):
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [hipcc(), *HIP_FLAGS, *EXTRA_FLAGS.get(src, []), "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile of {src} failed:\n{r.stderr}")
    return obj


def build(verbose=False):
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(6, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
