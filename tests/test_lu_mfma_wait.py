"""The wait between the lane swaps and the MFMA instructions of the wavefront LU.

An MFMA that reads the second operand of a v_permlane*_swap one instruction after
it gets the old value, and the compiler keeps no wait states there.  The wait is
part of the source; here the code made from it for gfx950 is looked at: the
operands of every MFMA come out of the wait (so no pass may reorder them), and no
MFMA reads a swap's register within four wait states."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2105_12070_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = """
#include "chem_cell.hpp"
template <int NP, bool FACTORS>
__global__ __launch_bounds__(256, 2) void k_lu(const double* A, int n, double* out, int* info) {
  __shared__ double scr[chem::LU_SCRATCH];
  chem::MatTiles<NP> M;
  chem::load_tiles<NP>(A, n, chem::lane_id(), M);
  double row[NP];
  chem::LuPiv<NP> lu;
  *info = chem::lu_factor<NP, FACTORS>(M, row, n, chem::lane_id(), lu, scr);
  for (int j = 0; j < NP; ++j) out[lu.step * NP + j] = row[j];
}
template __global__ void k_lu<16, false>(const double*, int, double*, int*);
template __global__ void k_lu<56, false>(const double*, int, double*, int*);
template __global__ void k_lu<56, true>(const double*, int, double*, int*);
"""


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    d = tmp_path_factory.mktemp("lu_wait")
    src = d / "lu.hip"
    src.write_text(SOURCE)
    base = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
            "-packed-fp32-ops", "-fno-fast-math", "-ffp-contract=fast", "-w", "-I", CSRC, "--cuda-device-only", "-S"]
    subprocess.run([*base, "-o", str(d / "lu.s"), str(src)], check=True)
    subprocess.run([*base, "-emit-llvm", "-o", str(d / "lu.ll"), str(src)], check=True)
    return (d / "lu.s").read_text(), (d / "lu.ll").read_text()


def test_operands_pass_through_the_wait(code):
    """The multipliers come out of the wait, the rows of U out of a statement that stands before it in the same block
    (volatile statements keep their order)."""
    count = 0
    for fn in re.findall(r"^define .*?^}", code[1], re.M | re.S):
        defs = {}
        for line, text in enumerate(fn.splitlines()):
            m = re.match(r"\s*(%\S+) = (.*)$", text)
            if m:
                defs[m.group(1)] = (line, m.group(2))

        def source(v):
            line, d = defs[v]
            m = re.match(r"extractvalue \{.*\} (%\S+), \d", d)
            return defs[m.group(1)] if m else (line, d)

        for a, b in re.findall(r"@llvm\.amdgcn\.mfma\.f64\.16x16x4f64\(double (%\S+), double (%\S+),", fn):
            count += 1
            (la, da), (lb, db) = source(a), source(b)
            assert 'asm sideeffect ""' in da, da
            assert 'asm sideeffect "s_nop' in db, db
            between = fn.splitlines()[la:lb]
            assert la < lb and not any(t.startswith(("br ", "  br ")) or re.match(r"\S+:", t) for t in between)
    assert count > 50


def regs(op):
    m = re.fullmatch(r"([va])\[(\d+):(\d+)\]", op)
    if m:
        return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    m = re.fullmatch(r"([va])(\d+)", op)
    return {(m.group(1), int(m.group(2)))} if m else set()


def test_no_mfma_close_behind_a_swap(code):
    last, at, count = {}, 0, 0  # register -> wait-state count at which a swap wrote it
    for line in code[0].splitlines():
        line = line.split(";")[0].strip()
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        name, _, rest = line.partition(" ")
        ops = [o.strip() for o in rest.split(",")]
        if name.startswith("v_mfma"):
            count += 1
            for r in set().union(*(regs(o) for o in ops[1:3])):
                assert at - last.get(r, -100) >= 4, line
        at += int(ops[0], 0) + 1 if name == "s_nop" else 1
        if name.startswith("v_permlane") and "swap" in name:
            for r in regs(ops[0]) | regs(ops[1]):
                last[r] = at
    assert count > 50
