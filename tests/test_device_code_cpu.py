"""Checks of the device code that need the compiler but no GPU: small kernels around the building blocks, compiled for
gfx950, and the instructions they become."""
import os
import re
import subprocess

import pytest

from paper_1705_09786_amd import build

CSRC = os.path.join(build.HERE, "csrc")


def assembly(tmp_path, body, also=""):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text('#include <hip/hip_runtime.h>\n#include "amp_worker.hip.h"\n#include "amp_batch.hip.h"\n' + also + body)
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    p = subprocess.run(["hipcc"] + flags + ["-Werror=inline-asm", "-I" + CSRC, "-S", "--offload-device-only", str(src), "-o", str(out)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout
    return out.read_text()


@pytest.mark.parametrize("times", [1, 2])
def test_transfer_to_lds_leaves_no_stale_m0(tmp_path, times):
    """m0 holds the LDS address of a transfer.  The compiler's own transfers to one address set it once; with global_to_lds in
    between it must be set again, or the second of them goes where global_to_lds did."""
    s = assembly(tmp_path, """
__shared__ float fixed_rows[64];
__global__ void probe(const float* p, float* o) {
  LDSQ float* row = (LDSQ float*)fixed_rows;
  __builtin_amdgcn_global_load_lds((const GQ float*)p + threadIdx.x, row, 4, 0, 0);
%s
  __builtin_amdgcn_global_load_lds((const GQ float*)p + threadIdx.x + 128, row, 4, 0, 0);
  __syncthreads();
  o[threadIdx.x] = fixed_rows[threadIdx.x] + amp_lds[threadIdx.x];
}
""" % "\n".join("  global_to_lds((const GQ float*)p + %d, (LDSQ float*)amp_lds + %d);" % (64 * k, 256 * k) for k in range(times)))
    ops = [(m.group(1), m.group(2).strip()) for m in re.finditer(r"^\s+(s_mov_b32 m0,|global_load_lds_dword(?:x4)?)\s*(.*)$", s, re.M)]
    loads = [(op, prev) for (op, _), prev in zip(ops[1:], ops) if op.startswith("global_load")]
    assert len([op for op, _ in ops if op.startswith("global_load")]) == times + 2, ops
    assert all(prev[0].startswith("s_mov_b32 m0") for _, prev in loads), ops
    assert ops[0][1] == ops[-2][1], ops   # the compiler's two go to the same place


@pytest.mark.parametrize("branch", [False, True])
def test_tree_publication_waits_once_for_each_pair_of_fetches(tmp_path, branch):
    """The arrivals at both of a message's joins, and the parents' arrivals and the rings' reservations, are on their way
    together: no wait for the vector memory between the two atomics of a pair, and no fetch from scratch in front of either."""
    s = assembly(tmp_path, """
__global__ __launch_bounds__(512) void probe(const AmpDev* Dp, const WorkerDev* Wp, int n) {
  const GQ AmpDev* D = (const GQ AmpDev*)Dp;
  const TreeBufs B = tree_bufs(D);
  const WorkerRegs wr = worker_regs(D, (const GQ WorkerDev*)Wp);
  const int lane = threadIdx.x & 63;
  const TreePost tp = tree_post_of(s_M, lane < n ? lane : 0, lane < n, lane < s_M.nF);
  publish_barrier();
  if (threadIdx.x < 64) {
    fence_release();
    tree_publish<%s>(wr, B, tp);
  }
}
""" % ("true" if branch else "false"), also='#include "amp_tree.hip.h"\n')
    body = s[s.index("\n_Z5probe"):]
    ops = re.findall(r"^\s+(global_atomic_add|scratch_load\w*|s_waitcnt vmcnt)", body[:body.index("s_endpgm")], re.M)
    assert not [op for op in ops if op.startswith("scratch")], ops
    first = ops.index("global_atomic_add")
    pairs = [op for op in ops[first:]]
    if branch:   # leaf cells arrive at one join
        assert pairs[:2] == ["global_atomic_add"] * 2, ops
        pairs = pairs[1:]
    assert pairs[1] == "s_waitcnt vmcnt" and pairs[2:5] == ["global_atomic_add"] * 2 + ["s_waitcnt vmcnt"], ops
