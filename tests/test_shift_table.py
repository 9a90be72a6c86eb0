"""The host's table of steps that stands for Algorithm 2's floor(c log2f(M) + P') on the
device (csrc/tables.cpp): every N, precision and moduli table builds, and at each step
and at the maximum before it the shift is the oracle's, up to maxima of 2^31 - 1."""
import subprocess

import pytest

import paper_2602_02549_amd as oz
from oracle.constants import constants
from oracle.ozaki2 import shift
from paper_2602_02549_amd.build import CSRC, hipcc

PROGRAM = r"""
#include <cstdio>
#include "ozaki2_internal.h"
using namespace oz2;
int main() {
  for (int table : {kTablePaper, kTableOptimal})
    for (int b : {64, 32})
      for (int N = 2; N <= (b == 64 ? kMaxModuli : 16); ++N) {
        CrtConsts cc;
        if (!build_consts(N, b, table, &cc)) return 1;
        std::printf("%d %d %d %d", table == kTableOptimal, b, N, cc.shift0);
        for (int s : cc.step) std::printf(" %d", s);
        std::printf("\n");
      }
}
"""
TOP = 2 ** 31 - 1


def test_constants_build_for_every_N():
    for table in (oz.MODULI_PAPER, oz.MODULI_OPTIMAL):
        for prec, top in ((64, 49), (32, 16)):
            for N in range(2, top + 1):
                rc = oz.ozaki2_debug_constants(prec, table, N)[0]
                assert rc == oz.OK, (table, prec, N)


def test_steps(tmp_path):
    try:
        cc = hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    src, exe = tmp_path / "steps.cpp", tmp_path / "steps"
    src.write_text(PROGRAM)
    p = subprocess.run([cc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17",
                        "-ffp-contract=off", "-I", CSRC, f"{CSRC}/tables.cpp", str(src), "-o",
                        str(exe)], capture_output=True, text=True)
    assert p.returncode == 0, p.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0
    lines = [[int(x) for x in line.split()] for line in out.stdout.splitlines()]
    assert len(lines) == 2 * (48 + 15)
    above_2_24 = 0
    for optimal, b, N, shift0, *steps in lines:
        const = constants(N, b, "optimal" if optimal else "paper")
        assert shift(0, 1, const) == shift0
        real = [s for s in steps if s < TOP]
        assert real == sorted(real) and steps[len(real):] == [TOP] * (len(steps) - len(real))
        for j, s in enumerate(real):
            # a repeated step drops the shift by more than one
            below = sum(q < s for q in real)
            assert shift(0, s - 1, const) == shift0 - below, (b, N, s)
            assert shift(0, s, const) == shift0 - sum(q <= s for q in real), (b, N, s)
            above_2_24 += s > 2 ** 24
        assert shift(0, TOP - 1, const) == shift0 - len(real), (b, N)
    assert above_2_24 > 100
