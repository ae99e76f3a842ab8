"""uniform() (bto_internal.h) moves a step size into scalar registers.  On gfx950
a vector register needs one wait state between the vector instruction that
writes it and the v_readfirstlane that reads it, and the scalar register it
writes two before a vector instruction reads that.  Checked in the listing of a
kernel that puts both next to each other.  No GPU."""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

KERNEL = """
#include "bto_internal.h"
__global__ void k(double* out, const double* in, double s) {
    const double x = bto::uniform(in[threadIdx.x] * s);
    out[threadIdx.x] = in[threadIdx.x + 64] * x;
}
"""


def _regs(text):
    out = set()
    for kind, lo, hi in re.findall(r"\b([vs])\[(\d+):(\d+)\]", text):
        out |= {f"{kind}{i}" for i in range(int(lo), int(hi) + 1)}
    return out | {kind + i for kind, i in re.findall(r"\b([vs])(\d+)\b", text)}


def test_scalar_moves_of_step_sizes_have_their_wait_states(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    (tmp_path / "k.hip").write_text(KERNEL)
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-I", os.path.join(ROOT, "paper_2004_02003_amd", "csrc"), "--cuda-device-only",
                    "-S", "-o", str(tmp_path / "k.s"), str(tmp_path / "k.hip")], check=True, capture_output=True)
    code = [ln.split(";")[0].strip() for ln in open(tmp_path / "k.s")]
    code = [ln for ln in code if re.match(r"[vs]_|global_", ln)]
    moves = 0
    for i, line in enumerate(code):
        op, _, args = line.partition(" ")
        if op != "v_readfirstlane_b32":
            continue
        moves += 1
        dst, src = (_regs(a) for a in args.split(","))
        before = code[i - 1]
        assert not (before.startswith("v_") and src & _regs(before.split(",")[0])), (before, line)
        waited = 0
        for after in code[i + 1:]:
            if waited >= 2:
                break
            name, _, rest = after.partition(" ")
            if name.startswith("v_"):
                assert not dst & _regs(rest.partition(",")[2]), (line, after)
            waited += 1 + int(rest) if name == "s_nop" else 1
    assert moves == 2
