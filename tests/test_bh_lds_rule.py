"""The rule by which the Boys-Handy pair-value kernels keep the next step's ket tables in LDS
(csrc/bh_lds.hpp, compiled for the host): with the LDS that each kernel really takes, both sets
are kept unless that costs a CU one of the workgroups that would run there without."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_17314_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include "bh_lds.hpp"
using namespace xtc;
int main() {
  for (int nn = 1; nn <= BH_MAXNUC; ++nn) {
    printf("split %d %d\n", nn, bh_tables_ahead(BH_PAIRS, nn));
    printf("fp64 %d %d\n", nn, bh_tables_ahead(BH_PAIRS_F64, nn));
  }
}
"""
# bytes beside the tables (two k-steps of half-precision fragments; nothing) and the workgroups
# that the kernels' registers (228 and 164 of a SIMD's 512 a lane, four waves on four SIMDs) allow
KERNELS = {"split": (2 * 4096 * 2, 2), "fp64": (0, 3)}


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_tables_ahead_never_cost_a_workgroup(tmp_path):
    (tmp_path / "rule.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(tmp_path / "rule.cpp"), "-o", str(tmp_path / "rule")],
                   check=True)
    out = subprocess.run([str(tmp_path / "rule")], check=True, capture_output=True, text=True).stdout
    rows = [line.split() for line in out.splitlines()]
    assert len(rows) == 48
    for kernel, nn, ahead in rows:
        nn, (beside, most) = int(nn), KERNELS[kernel]
        ket = 16 * (16 * nn + 2) + 16 * nn            # ket table with its padding, a_I
        size = [8 * (128 * nn + sets * ket + 128) + beside for sets in (1, 2)]
        assert size[1] <= 160 * 1024
        on_cu = [min(most, 160 * 1024 // s) for s in size]
        assert int(ahead) == (on_cu[1] == on_cu[0]), (kernel, nn, ahead, on_cu)
