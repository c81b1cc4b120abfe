"""Division by one high product (csrc/fast_div.h) against the machine's division, on the host: every quotient's edges."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "fast_div.h"
using namespace binattn;

static long n_checked = 0;
static bool check(int n, int d, FastDiv f) {
    ++n_checked;
    if (fast_div(n, f.m, f.s) == n / d) return true;
    printf("%d / %d = %d, got %d\n", n, d, n / d, fast_div(n, f.m, f.s));
    return false;
}
static bool divisor(int d) {
    const FastDiv f = make_fast_div(d);
    const int top = 0x7fffffff, qmax = top / d;
    // around multiples of d: small quotients, spread ones, the largest
    for (int i = 0; i < 400; ++i) {
        const int64_t q = i < 100 ? i : i < 300 ? (int64_t)qmax * (i - 100) / 200 : (int64_t)qmax - (i - 300);
        for (int64_t n = q * d - 1; n <= q * d + 1; ++n)
            if (n >= 0 && n <= top && !check((int)n, d, f)) return false;
    }
    return check(top, d, f) && check(top - 1, d, f) && check(0, d, f);
}
int main() {
    for (int d = 1; d <= 1 << 17; ++d)  // row blocks of up to 2^24 tokens
        if (!divisor(d)) return 1;
    for (int i = 0, d = 1 << 17; d < 1 << 24; d += 1 + (++i * 2654435761u >> 22))  // batch and heads up to 2^24
        if (!divisor(d)) return 1;
    for (int s = 17; s < 31; ++s)
        for (int o = -3; o <= 3; ++o)
            if (!divisor((1 << s) + o)) return 1;
    if (!divisor(0x7fffffff) || !divisor(0x7ffffffe)) return 1;
    printf("ok %ld\n", n_checked);
}
"""


def run(tmp_path, edit=lambda header: header):
    header = open(os.path.join(ROOT, "paper_2603_09582_amd", "csrc", "fast_div.h")).read()
    (tmp_path / "fast_div.h").write_text(edit(header))
    (tmp_path / "check.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", str(tmp_path), str(tmp_path / "check.cpp"), "-o", exe], check=True)
    return subprocess.run([exe], capture_output=True, text=True, timeout=120)


def test_quotients(tmp_path):
    r = run(tmp_path)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[1]) > 150_000_000


def test_the_check_sees_a_multiplier_that_is_one_too_small(tmp_path):
    assert run(tmp_path, lambda s: s.replace("(uint64_t)d + 1)", "(uint64_t)d)")).returncode == 1
