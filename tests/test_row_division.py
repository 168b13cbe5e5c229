"""The division of a pair index by the row length that the LSTM kernels do with a multiplication and a
shift (csrc/ktanh_order.h), compiled for the CPU and compared with the division it stands for."""
import os
import subprocess

from paper_1909_07729_amd import build

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "ktanh_order.h"
using namespace ktanh_device;
static unsigned long long tried = 0;
static int check(unsigned p, unsigned d, RowDivision r)
{
    ++tried;
    if (row_of_pair(p, r.mul, r.shift) == p / d) return 0;
    std::printf("%u / %u gives %u\n", p, d, row_of_pair(p, r.mul, r.shift));
    return 1;
}
static int divisor(unsigned d)
{
    const RowDivision r = row_division(d);
    const unsigned top = (1u << 30) - 1;
    int bad = 0;
    // the first and last index of rows near the ends and the middle of the range: where a quotient steps
    for (unsigned long long row : {0ull, 1ull, 2ull, 3ull, (unsigned long long)(top / d / 2), (unsigned long long)(top / d - 1), (unsigned long long)(top / d)})
        for (long long at : {(long long)(row * d) - 1, (long long)(row * d), (long long)(row * d) + d - 1})
            if (at >= 0 && at <= top) bad += check((unsigned)at, d, r);
    return bad + check(top, d, r);
}
int main()
{
    int bad = 0;
    for (unsigned d = 4; d < 70000 && !bad; ++d) bad += divisor(d);
    for (unsigned l = 2; l <= 29; ++l)
        for (int k = -3; k <= 3; ++k) {
            const long long d = (1ll << l) + k;
            if (d >= 4 && d <= (1ll << 30)) bad += divisor((unsigned)d);
        }
    bad += divisor(1u << 30);
    for (unsigned d : {4u, 20u, 1028u, 1536u})   // every index of the first rows
        for (unsigned p = 0; p < 2000000u; ++p) bad += check(p, d, row_division(d));
    std::printf("%llu quotients\n", tried);
    return bad != 0;
}
"""


def test_row_division_equals_the_division(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-fsanitize=undefined", "-fno-sanitize-recover",
                    "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stdout[-2000:] + done.stderr[-2000:]
    assert int(done.stdout.split()[0]) > 8_000_000
