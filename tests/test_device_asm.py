"""AMD assembly of device code that the compiler does not schedule by itself."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2604_15379_amd import build as B

CSRC = os.path.join(os.path.dirname(B.__file__), "csrc")

# The load's offset (its resource, its place in LDS) comes from the vector ALU right in front of it.
PROBE = r"""
#include <hip/hip_runtime.h>
#include "../../include/fleet.h"
#include "graph.hpp"
#include "kernels.hip.inc"
extern __shared__ char probe_lds[];
__device__ __forceinline__ uint32_t sreg(int v) { return (uint32_t)__builtin_amdgcn_readfirstlane(v); }
__global__ void probe(const int* in, float* out, uint32_t lo, uint32_t hi, uint32_t lds, int n) {
  for (int i = 0; i < n; ++i)
    dev::load_to_lds16(lds, threadIdx.x * 16, (u32x4){lo, hi, 1024u, 0x00020000u}, sreg(in[64 * i + threadIdx.x]));
  for (int i = 0; i < n; ++i)
    dev::load_to_lds16(lds, threadIdx.x * 16, (u32x4){lo, hi, sreg(in[64 * i + threadIdx.x]), 0x00020000u}, 0u);
  for (int i = 0; i < n; ++i)
    dev::load_to_lds16(sreg(in[64 * i + threadIdx.x]), threadIdx.x * 16, (u32x4){lo, hi, 1024u, 0x00020000u}, 0u);
  dev::wait_vm<0>();
  out[threadIdx.x] = ((float*)probe_lds)[threadIdx.x];
}
"""


def _regs(text):
    """Scalar registers named in an operand list."""
    out = set()
    for lo, hi, one in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", text):
        out |= {f"s{i}" for i in range(int(lo), int(hi) + 1)} if lo else {f"s{one}"}
    if re.search(r"\bm0\b", text):
        out.add("m0")
    return out


def _wait_states(lines, i, regs):
    """Least wait states between a write by the vector ALU (by the scalar ALU: m0 only) to one of
    `regs` and instruction i, looking back to the label in front of it."""
    least, states = {"valu": 99, "m0": 99}, 0
    for line in reversed(lines[:i]):
        m = re.match(r"\s+([a-z]\w+)\s*(.*)", line)
        if line.endswith(":") or not m:
            break
        name, ops = m.groups()
        dst = _regs(ops.split(",")[0])
        if name.startswith("v_") and dst & regs:
            least["valu"] = min(least["valu"], states)
        if name.startswith("s_") and "m0" in dst:
            least["m0"] = min(least["m0"], states)
        states += 1 + (int(ops, 0) if name == "s_nop" else 0)
    return least


def test_wait_states_in_front_of_loads_to_lds(tmp_path):
    """The hardware does not check the distance between a vector ALU write to a scalar register and a
    vector memory instruction that reads it (five wait states), nor between a write to m0 and a load
    to LDS (one).  The compiler does, but not for an instruction in an assembly statement."""
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc here")
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    res = subprocess.run(["hipcc", *B._FLAGS, f"-I{CSRC}", "--cuda-device-only", "-S", str(src), "-o", str(asm)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    lines = [t for t in (re.split(r";|//", s)[0].rstrip() for s in asm.read_text().splitlines()) if t]
    loads = [i for i, s in enumerate(lines) if re.search(r"buffer_load_dwordx4 .* lds\b", s)]
    assert len(loads) >= 3
    seen = []
    for i in loads:
        w = _wait_states(lines, i, _regs(lines[i]) | {"m0"})
        seen.append(w["valu"])
        assert w["valu"] >= 5 and w["m0"] >= 1, (w, lines[max(0, i - 12):i + 1])
    assert min(seen) < 99                    # the probe does put such a write in front
    assert "inline asm clobber list" not in res.stderr   # (m0 is reserved: what becomes of it there is undefined)
