"""The walk over a row's edges at the largest positions (csrc/rows.h), built for
the host with arrays that check every index."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "rows.h"

static int fail(const char* what, int first, int last, long long at)
{
    printf("%s: row [%d, %d) at %lld\n", what, first, last, at);
    exit(1);
}

template <int U>
static void row(int first, int last, int stop)
{
    std::vector<unsigned> seen;
    auto head = [&](unsigned e) {
        if (e < (unsigned)first || e >= (unsigned)last) fail("position out of the row", first, last, e);
        return (int)(e & 1023);
    };
    auto value = [&](int u) {
        if (u < 0 || u > 1023) fail("head out of range", first, last, u);
        return u * 3;
    };
    ocm::for_row<U>(first, last, head, value, [&](unsigned e, int u, int y) {
        if (u != (int)(e & 1023) || y != u * 3) fail("another edge's head", first, last, e);
        seen.push_back(e);
        return (int)seen.size() == stop;
    });
    const long long len = (long long)last - first, want = stop < 0 || stop > len ? len : stop;
    if ((long long)seen.size() != want) fail("edges walked", first, last, (long long)seen.size());
    for (long long i = 0; i < want; ++i)
        if (seen[i] != (unsigned)first + i) fail("order", first, last, i);
}

int main()
{
    for (int base : {0, 5, INT_MAX - 40})
        for (int a = 0; a < 12; ++a)
            for (int b = a; b <= 40; ++b)
                for (int stop : {-1, 1, 3, 7}) {
                    row<4>(base + a, base + b, stop);
                    row<8>(base + a, base + b, stop);
                }
    return 0;
}
"""


def test_rows_up_to_the_last_position(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(MAIN)
    inc = os.path.join(ROOT, "paper_1111_0627_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wno-unknown-pragmas", "-I", inc, str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout
