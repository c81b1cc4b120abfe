"""The split of the single launch's last heads by row blocks (csrc/head_split.h), run on the host for every number of heads: every
row block is taken once, and no chiplet gets more workgroups than its share of the rounds that whole heads would take."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "head_split.h"
using namespace binattn;

static long splits = 0;
static bool check(int heads, int from, int slots) {
    if (from == heads) return true;
    ++splits;
    if (from <= 0 || from > heads || from % 8) { printf("%d heads: split from %d\n", heads, from); return false; }
    std::vector<int> rows(2 * heads, 0);
    int on[8] = {0};
    for (int v = 0; v < split_grid(from, heads); ++v) {
        const int head = split_head(v, from, heads), rb = split_row_block(v, from);
        if (head < 0) { printf("%d heads: workgroup %d takes head %d\n", heads, v, head); return false; }
        if (head >= heads) continue;
        ++on[v % 8];
        if (v < from) ++rows[2 * head], ++rows[2 * head + 1];
        else ++rows[2 * head + rb];
    }
    for (int r : rows)
        if (r != 1) { printf("%d heads from %d: a row block is taken %d times\n", heads, from, r); return false; }
    const int rounds = (heads + slots - 1) / slots;
    for (int x = 0; x < 8; ++x)
        if (on[x] > slots / 8 * rounds) { printf("%d heads from %d: %d workgroups on chiplet %d, %d rounds of %d\n", heads, from, on[x], x, rounds, slots / 8); return false; }
    return true;
}
int main() {
    for (int heads = 257; heads <= 8192; ++heads)
        if (!check(heads, split_last(heads, 512), 512) || !check(heads, split_of_768(heads), 768)) return 1;
    printf("ok %ld\n", splits);
}
"""


def run(tmp_path, edit=lambda header: header):
    header = open(os.path.join(ROOT, "paper_2603_09582_amd", "csrc", "head_split.h")).read()
    edited = edit(header)
    (tmp_path / "head_split.h").write_text(edited)
    (tmp_path / "check.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", str(tmp_path), str(tmp_path / "check.cpp"), "-o", exe], check=True)
    return subprocess.run([exe], capture_output=True, text=True, timeout=120)


def test_every_row_block_once_and_no_chiplet_over_its_share(tmp_path):
    r = run(tmp_path)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[1]) > 4000


def test_the_check_sees_a_share_that_is_counted_over_the_whole_chip(tmp_path):
    """768 slots less the heads, as if heads were dealt out one by one."""
    old = "const int from = SPLIT_XCDS * (2 * eighth - 96 * rounds);"
    r = run(tmp_path, lambda s: s.replace(old, "const int from = (heads - (768 * rounds - heads)) / 8 * 8;"))
    assert r.returncode == 1 and "521 heads from 272: 98 workgroups on chiplet 0, 1 rounds of 96" in r.stdout


def test_the_check_sees_a_row_block_that_is_taken_twice(tmp_path):
    r = run(tmp_path, lambda s: s.replace("((v - from) >> 3) & 1", "((v - from) >> 4) & 1"))
    assert r.returncode == 1 and "is taken" in r.stdout
