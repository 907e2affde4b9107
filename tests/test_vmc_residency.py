"""The rule by which two walkers of the e-e local energies share a SIMD (csrc/vmc_residency.hpp,
compiled for the host): only where that saves a round of walkers (256 CUs, 160 KB of LDS, at most
two waves on each of four SIMDs)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_17314_amd", "csrc")
NEED = (1000, 16000, 20480, 23100, 30350, 32768, 33000, 50000, 163840)
WALKERS = (1, 65, 1024, 1025, 1280, 1281, 2048, 2049, 4096, 5120, 8192, 16384, 65536)
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "vmc_residency.hpp"
int main(int argc, char** argv) {
  for (int i = 1; i + 1 < argc; i += 2)
    printf("%ld\n", (long)xtc::vmc_two_per_simd(atol(argv[i]), atol(argv[i + 1])));
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_walkers_share_a_simd_only_to_save_a_round(tmp_path):
    (tmp_path / "r.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(tmp_path / "r.cpp"), "-o", str(tmp_path / "r")], check=True)
    cases = [(n, w) for n in NEED for w in WALKERS]
    out = subprocess.run([str(tmp_path / "r")] + [str(x) for c in cases for x in c], check=True,
                         capture_output=True, text=True).stdout.split()
    assert len(out) == len(cases)
    cu = 160 * 1024
    for (need, walkers), two in zip(cases, map(int, out)):
        on_cu = -(-walkers // 256)
        rounds = lambda resident: -(-on_cu // resident)
        possible = min(8, cu // need)
        assert bool(two) == (rounds(possible) < rounds(min(4, possible))), (need, walkers, two)


@pytest.mark.gpu
def test_energies_do_not_depend_on_the_batch():
    """1,300 walkers run two per SIMD, halves of them one: the same values bit for bit."""
    import torch
    from paper_2607_17314_amd import api
    from workloads import make_config
    wl = make_config("h4")
    sys_ = api.VmcSystem.from_workload(wl)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    centres = torch.as_tensor(wl.atom_xyz).cuda()[torch.arange(sys_.n_el, device="cuda") % len(wl.atom_xyz)]
    R = centres[None] + 0.7 * torch.randn((1300, sys_.n_el, 3), dtype=torch.float64, device="cuda", generator=gen)
    E, dE = api.vmc_local_energy(sys_, wl.corr, R)
    halves = [api.vmc_local_energy(sys_, wl.corr, R[s:s + 650].contiguous()) for s in (0, 650)]
    assert bool(torch.isfinite(E).all())
    assert torch.equal(E, torch.cat([h[0] for h in halves])) and torch.equal(dE, torch.cat([h[1] for h in halves]))
