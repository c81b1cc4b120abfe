"""The index arithmetic of the dense bias copies (csrc/bias_rows.h), run on the host as the kernel's waves run it: no
copy reads outside the tensor, and every key of every row ends up where the kernel reads it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>
#include "bias_rows.h"
using namespace binattn;
static long cases = 0;

// one wave's tile of one key block; esz: 2 or 4; segs: staged 128-byte segments per row
static void wave_tile(int64_t off, int row0, int N, int64_t sn, int64_t extent, int blk, int esz, int segs) {
    const int EC = 16 / esz, KSEG = 128 / esz;
    std::vector<int64_t> lds(32 * segs * 128 / esz, -1);  // which element of the tensor lies there
    const int klim = bias_key_limit(off, row0, N, sn, extent, blk * 128, EC);
    for (int rg = 0; rg < 4; ++rg)
        for (int seg = 0; seg < segs; ++seg)
            for (int lane = 0; lane < 64; ++lane) {
                const int key0 = blk * 128 + KSEG * seg + EC * bias_copy_chunk(rg, lane);
                if (!(key0 < klim)) continue;
                const int64_t e = off + (int64_t)bias_copy_row(bias_group_row(row0, rg, N), rg, lane, N) * sn + key0;
                if (e < 0 || e + EC > extent) {
                    printf("copy reads [%ld, %ld) of %ld: N=%d row0=%d sn=%ld blk=%d esz=%d\n", (long)e, (long)(e + EC), (long)extent, N, row0, (long)sn, blk, esz);
                    exit(1);
                }
                for (int i = 0; i < EC; ++i) lds[((rg * segs + seg) * 1024 + 16 * lane) / esz + i] = e + i;
            }
    if (klim != N) {
        const int k0 = (N & -EC) - blk * 128;
        for (int ln = 0; ln < 32 && k0 < segs * KSEG; ++ln) {
            const int row = bias_min(row0 + ln, N - 1);
            for (int i = 0; i < (N & (EC - 1)); ++i) {
                const int64_t e = off + (int64_t)row * sn + (N & -EC) + i;
                if (e >= extent) { printf("tail reads element %ld of %ld\n", (long)e, (long)extent); exit(1); }
                lds[bias_lds_chunk(ln, k0 / KSEG, k0 / EC & 7, segs) / esz + i] = e;
            }
        }
    }
    for (int m = 0; m < 32 && row0 + m < N; ++m)
        for (int k = 0; k < segs * KSEG && blk * 128 + k < N; ++k) {
            const int64_t have = lds[bias_lds_chunk(m, k / KSEG, k / EC & 7, segs) / esz + k % EC];
            if (have != off + (int64_t)(row0 + m) * sn + blk * 128 + k) {
                printf("row %d key %d holds %ld: N=%d sn=%ld esz=%d segs=%d\n", row0 + m, blk * 128 + k, (long)have, N, (long)sn, esz, segs);
                exit(1);
            }
        }
    ++cases;
}

int main() {
    const int lengths[] = {1, 2, 3, 5, 7, 8, 9, 15, 31, 33, 63, 64, 65, 95, 97, 100, 121, 127, 128, 129, 131, 160, 191, 197, 250, 255, 256, 257, 391};
    for (int N : lengths)
        for (int extra : {0, 1, 3, 7, 8, 61})
            for (int layout = 0; layout < 5; ++layout)
                for (int B : {1, 2})
                    for (int H : {1, 3}) {
                        const int64_t sn = N == 1 && layout == 4 ? 0 : N + extra;
                        int64_t sh = N * sn, sb = H * sh;
                        if (layout == 1) sb = 0;             // shared over the batch
                        if (layout == 2) sh = sb = 0;        // one matrix for all
                        if (layout == 3) { sb = sn; sh = B * sn; }  // overlapping windows
                        if (layout == 4) { sh = 0; sb = N * sn + 5; }
                        const int64_t extent = bias_extent(B, H, N, sb, sh, sn);
                        for (int b = 0; b < B; ++b)
                            for (int h = 0; h < H; ++h)
                                for (int row0 = 0; row0 < (N + 127) / 128 * 128 + 128; row0 += 32)
                                    for (int blk = 0; blk * 128 < N; ++blk) {
                                        wave_tile(b * sb + h * sh, row0, N, sn, extent, blk, 2, 2);
                                        wave_tile(b * sb + h * sh, row0, N, sn, extent, blk, 4, 2);
                                        wave_tile(b * sb + h * sh, row0, N, sn, extent, blk, 4, 3);
                                    }
                    }
    printf("ok %ld\n", cases);
}
"""


def run(tmp_path, edit=lambda header: header):
    header = open(os.path.join(ROOT, "paper_2603_09582_amd", "csrc", "bias_rows.h")).read()
    (tmp_path / "bias_rows.h").write_text(edit(header))
    (tmp_path / "check.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", str(tmp_path), str(tmp_path / "check.cpp"), "-o", exe], check=True)
    return subprocess.run([exe], capture_output=True, text=True, timeout=120)


def test_copies_stay_inside_the_tensor_and_cover_every_key(tmp_path):
    r = run(tmp_path)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[1]) > 10000


def test_the_check_sees_a_limit_that_is_never_applied(tmp_path):
    """With the key limit always N some copy reads behind the last element."""
    r = run(tmp_path, lambda s: s.replace("> extent ? N - (ec - 1) : N", "> extent ? N : N"))
    assert r.returncode == 1 and "copy reads" in r.stdout
