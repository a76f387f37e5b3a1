"""Checks of the device code that need the compiler but no GPU: small kernels around the building blocks, compiled for
gfx950, and the instructions they become."""
import os
import re
import subprocess

import pytest

from paper_1705_09786_amd import build

CSRC = os.path.join(build.HERE, "csrc")


def assembly(tmp_path, body):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text('#include <hip/hip_runtime.h>\n#include "amp_worker.hip.h"\n#include "amp_batch.hip.h"\n' + body)
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
