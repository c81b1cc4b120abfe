"""The index arithmetic of the single launch's V loads (csrc/head_rows.h), run on the host for every head dimension and
both workgroup sizes: every chunk of every token quad belongs to some thread, and the 32-bit offset of a row beyond the
sequence lies behind the end of the buffer descriptor whatever the row pitch."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdint>
#include <cstdio>
#include <initializer_list>
#include "head_rows.h"
using namespace binattn;

int main() {
    long cells = 0, offsets = 0;
    for (int nt : {256, 512})
        for (int c16 = 1; c16 <= 16; ++c16) {
            const int dk = (8 * c16 + 31) / 32, groups = head_v_groups(nt, c16);
            for (int N = 1; N <= 4 * HEAD_QUADS; ++N) {
                static int owners[HEAD_QUADS][16];
                for (auto &r : owners) for (int &x : r) x = 0;
                for (int pass = 0; pass < head_v_passes(nt, dk); ++pass)
                    for (int thread = 0; thread < nt && head_v_pass(pass, groups); ++thread) {
                        const int quad = head_v_quad(head_v_group(thread / c16, nt, dk), pass, groups);
                        if (quad < HEAD_QUADS) ++owners[quad][thread % c16];
                        if (N > 3 && N % 64 != 9 && N % 64 != 0 && N % 128 != 127) continue;
                        for (int64_t pitch : {8, 1 << 10, 1 << 20, (1 << 20) + (1 << 18), 1 << 21, 5 << 19, (3 << 20) + 8, HEAD_FAR_PITCH - 8})
                            for (int t = 0; t < 4; ++t, ++offsets) {
                                const uint32_t bytes = N > 1 ? 2 * (uint32_t)(pitch < 8 * c16 ? 8 * c16 : pitch) : 16 * c16;
                                const uint32_t end = (N - 1) * bytes + 16 * c16, off = (4 * quad + t) * bytes + 16 * (thread % c16);
                                const bool row = 4 * quad + t < N;
                                if (row ? off != (int64_t)(4 * quad + t) * bytes + 16 * (thread % c16) || off + 16 > end : off < end) {
                                    printf("row %d of %d at offset %u, end %u: %d threads, d = %d, pitch %ld\n", 4 * quad + t, N, off, end, nt, 8 * c16, (long)pitch);
                                    return 1;
                                }
                            }
                    }
                for (int quad = 0; 4 * quad < N; ++quad)
                    for (int c = 0; c < c16; ++c, ++cells)
                        if (owners[quad][c] == 0) { printf("nobody loads quad %d chunk %d: %d threads, d = %d\n", quad, c, nt, 8 * c16); return 1; }
            }
        }
    printf("ok %ld %ld\n", cells, offsets);
}
"""


def run(tmp_path, edit=lambda header: header):
    header = open(os.path.join(ROOT, "paper_2603_09582_amd", "csrc", "head_rows.h")).read()
    (tmp_path / "head_rows.h").write_text(edit(header))
    (tmp_path / "check.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", str(tmp_path), str(tmp_path / "check.cpp"), "-o", exe], check=True)
    return subprocess.run([exe], capture_output=True, text=True, timeout=120)


def test_every_chunk_is_loaded_and_no_row_beyond_the_sequence(tmp_path):
    r = run(tmp_path)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[1]) == 2 * 136 * 4 * (64 * 65 // 2)


def test_the_check_sees_a_pass_too_few(tmp_path):
    """Passes counted from nt / (4 dk) groups as if that division left no remainder."""
    r = run(tmp_path, lambda s: s.replace("return (HEAD_QUADS + nt / (4 * dk) - 1) / (nt / (4 * dk));", "return (HEAD_QUADS * 4 * dk + nt - 1) / nt;"))
    assert r.returncode == 1 and "nobody loads quad 63 chunk 4: 256 threads, d = 96" in r.stdout


def test_the_check_sees_an_offset_that_wraps(tmp_path):
    """Rows counted on through all groups: up to 2047 at d = 8."""
    r = run(tmp_path, lambda s: s.replace("|| number < HEAD_QUADS ? number", "|| true ? number"))
    assert r.returncode == 1 and "at offset" in r.stdout and "d = 8," in r.stdout
