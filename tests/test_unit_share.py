"""How the fitting kernel's workgroups share the units of a batch: every unit is dealt to a workgroup
or lies with a dealer that some workgroup serves, once, for any number of workgroups and units.  The
rule is host code too, and is asked for here as the kernel asks for it."""
import subprocess

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "svt_units.h"
int main() {
    const int grids[] = {1, 2, 3, 8, 15, 16, 31, 32, 33, 64, 255, 256, 304};
    const long units[] = {0, 1, 15, 16, 17, 31, 33, 128, 129, 400, 511, 512, 513, 4096, 4097, 7500,
                          100003};
    for (int grid : grids)
        for (long nu : units) {
            std::vector<int> owners(nu, 0);
            bool served[svt::kDealers] = {};
            for (int b = 0; b < grid; ++b) {
                const svt::UnitShare s = svt::unit_share(nu, b, grid);
                for (long u = s.lo; u < s.hi; ++u) ++owners[u];
                if (served[s.dealer]) continue;
                served[s.dealer] = true;  // its tickets are drawn until they run past p_hi
                if (s.batch < 1) return 1;
                for (long u = s.p_lo; u < s.p_hi; ++u) ++owners[u];
            }
            long lost = 0, twice = 0;
            for (int n : owners) { lost += n == 0; twice += n > 1; }
            if (lost || twice)
                std::printf("grid %d units %ld: %ld lost, %ld twice\n", grid, nu, lost, twice);
        }
    std::printf("checked\n");
}
"""


def test_every_unit_has_one_owner(tmp_path):
    from paper_1312_0917_amd import build as B
    src, exe = tmp_path / "share.hip", tmp_path / "share"
    src.write_text(PROGRAM)
    r = subprocess.run([B.hipcc(), *B.HIPCC_FLAGS, "-O1", str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60).stdout
    assert out == "checked\n", out
