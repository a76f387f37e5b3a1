"""Builds the HIP library (kernels + C boundary) for gfx950, in-tree: libamp.so, and libamp_strict.so, the same
sources compiled with -DAMP_STRICT_JOIN (joins completed, and messages handed over inside one die, with explicit acquire /
release ordering instead of the fence-free shortcuts; the parity suite runs both so that a mismatch can be attributed).  Every model's persistent kernel
is a source file of its own, compiled side by side."""
from __future__ import annotations

import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(HERE, "libamp.so")
LIB_STRICT = os.path.join(HERE, "libamp_strict.so")
SOURCES = ["amp_tree.hip", "amp_ggnn.hip", "amp_rnn.hip", "amp_mlp.hip", "amp_kernels.hip", "amp_lib.cpp"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc(args) -> str:
    p = subprocess.run(["hipcc"] + FLAGS + args, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if p.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (" ".join(args), p.stdout))
    return p.stdout


def build(verbose: bool = False, strict: bool = True, extra=()) -> str:
    jobs = [(LIB, list(extra))]
    if strict:
        jobs.append((LIB_STRICT, ["-DAMP_STRICT_JOIN"] + list(extra)))
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
        todo = []
        for src in SOURCES:   # the largest first
            for j, (out, flags) in enumerate(jobs):
                obj = os.path.join(tmp, "%s.%d.o" % (src, j))
                todo.append((j, obj, pool.submit(_hipcc, flags + ["-c", os.path.join(HERE, "csrc", src), "-o", obj])))
        logs = [f.result() for _, _, f in todo]
        for j, (out, flags) in enumerate(jobs):
            logs.append(_hipcc(flags + ["-shared"] + [obj for k, obj, _ in todo if k == j] + ["-o", out]))
    if verbose:
        print("".join(logs))
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
