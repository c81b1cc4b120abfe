"""The grid of the operand preparation (csrc/psi_grid.h), on the host: no launch reaches the runtime's limit of 2^32 threads
whatever number of heads the library accepts, and each is as large as that allows."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "psi_grid.h"
using namespace binattn;

int main() {
    long launches = 0;
    for (int C16 = 1; C16 <= 16; ++C16)
        for (int nblk = 1; nblk <= 32; ++nblk)
            for (PsiKeys keys : {PSI_V_ONLY, PSI_EXPAND, PSI_PHI}) {
                const int nt = psi_threads(nblk), most = psi_heads(C16, nblk, keys);
                const int64_t limit = (int64_t)1 << 32;
                if (most < 1 || psi_workgroups(most, C16, nblk, keys) * nt >= limit || psi_workgroups(2 * most, C16, nblk, keys) * nt < limit) {
                    printf("%d heads: %ld workgroups of %d, d = %d, %d blocks, kind %d\n", most, (long)psi_workgroups(most, C16, nblk, keys), nt, 8 * C16, nblk, (int)keys);
                    return 1;
                }
                ++launches;
            }
    printf("ok %ld\n", launches);
}
"""


def run(tmp_path, edit=lambda header: header):
    header = open(os.path.join(ROOT, "paper_2603_09582_amd", "csrc", "psi_grid.h")).read()
    (tmp_path / "psi_grid.h").write_text(edit(header))
    (tmp_path / "check.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", str(tmp_path), str(tmp_path / "check.cpp"), "-o", exe], check=True)
    return subprocess.run([exe], capture_output=True, text=True, timeout=120)


def test_no_launch_reaches_the_limit_of_threads(tmp_path):
    r = run(tmp_path)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[1]) == 16 * 32 * 3


def test_the_check_sees_one_launch_for_all_heads(tmp_path):
    """All heads that the library accepts in one launch."""
    r = run(tmp_path, lambda s: s.replace("return (int)((((int64_t)1 << 32)", "return (1 << 24) - 1; return (int)((((int64_t)1 << 32)"))
    assert r.returncode == 1
