"""Wait states that inline assembly owes to the instructions behind it, read
from the assembly that the compiler writes for a kernel made here (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2210_06437_amd import _build

KERNEL = r"""
#include "octohydro_kernels.h"
using namespace octohydro;
// a lane move of a value that monotonise does not touch, or of its result,
// held directly behind it
extern "C" __global__ void probe(const double* a, double* o, const int* u, int* w) {
  const int t = threadIdx.x;
  double l = a[t], r = a[t + 64];
  const double c = a[t + 128];
  int v = u[t];
  asm volatile("" : "+v"(v));
  __builtin_amdgcn_sched_barrier(0);
  PARABOLA(c, l, r);
  asm volatile("" : "+v"(l), "+v"(r));
  __builtin_amdgcn_sched_barrier(0);
  w[t] = MOVE;
  o[t] = l;
  o[t + 64] = r;
}
"""
SHIFT = "__builtin_amdgcn_update_dpp({0}, {0}, 0x111, 0xF, 0xF, false)"


def _assembly(tmp_path, parabola, move):
    src = tmp_path / "probe.hip"
    src.write_text(KERNEL.replace("PARABOLA", parabola).replace("MOVE", move))
    out = tmp_path / "probe.s"
    subprocess.run([_build.HIPCC, *_build.FLAGS, "--offload-device-only", "-S", "-o",
                    str(out), str(src)], check=True, capture_output=True)
    text = out.read_text()
    body = text[text.index("\nprobe:"):]
    return [l.strip() for l in body[:body.index("s_endpgm")].splitlines()
            if re.match(r"\s+[a-z]+_", l)]


def _states_before(lines, first, until):
    """Wait states between the last line that matches `first` and the first
    after it that matches `until`: one per instruction, n + 1 per `s_nop n`."""
    at = max(i for i, l in enumerate(lines) if re.match(first, l))
    n = 0
    for l in lines[at + 1:]:
        if re.search(until, l):
            return n
        nop = re.match(r"s_nop (\d+)", l)
        n += int(nop.group(1)) + 1 if nop else 1
    raise AssertionError("no lane move behind the statement")


@pytest.mark.skipif(not os.path.exists(_build.HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("parabola,move", [
    # the 3D plane task: padded in the parabola
    ("monotonise<true>", SHIFT.format("v")),
    ("monotonise<true>", SHIFT.format("__double2loint(r)")),
    # the node copies: padded in the move
    ("monotonise", "dpp_word<DPP_XOR1>(v)"),
    ("monotonise", "dpp_word<DPP_XOR8>(__double2hiint(l))"),
])
def test_lane_move_behind_the_monotonised_parabola(tmp_path, parabola, move):
    """A DPP operation needs five wait states after a vector instruction has
    written EXEC."""
    lines = _assembly(tmp_path, parabola, move)
    assert _states_before(lines, r"v_cmpx_", r"_dpp\b") >= 5, lines
