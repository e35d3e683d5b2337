"""Builds the gfx950 shared library (hipcc) next to this file."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdqn_mi355.so")
SOURCES = ["error.hip", "replay.hip", "net.hip", "envs.hip", "alg1.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
         # the first kernel arguments arrive in scalar registers with the wavefront instead of through a load from cold
         # memory (14 dwords on gfx950; the hot kernels' signatures lead with what they need first)
         "-mllvm", "-amdgpu-kernarg-preload-count=16",
         # every kernel starts on a page of its own: where a small kernel came to lie decided how often it missed the instruction cache (minibatch
         # 45, misses per launch without -> with: fc1's data gradient 84 -> 42, the conv data gradients 281 -> 140, the act head 12 -> 4; counters in
         # profiles/instruction_cache_b45.txt), so the size of one kernel changed the time of the next (250 train steps at minibatch 45 12.89 -> 12.72 ms)
         "-Xarch_device", "-falign-functions=4096"]


def _compile(src: str) -> str:
    obj = os.path.join(CSRC, "_build", os.path.splitext(src)[0] + ".o")
    os.makedirs(os.path.dirname(obj), exist_ok=True)
    cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build() -> str:
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp.%d" % os.getpid()
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
