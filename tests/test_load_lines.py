"""Which calls read their input with plain loads (csrc/ktanh_order.h), compiled for the CPU: plain loads are up to 7 % slower
on inputs that come from HBM, so the line has to stand below the size from which they gain less than that."""
import subprocess

from paper_1909_07729_amd import build

PROGRAM = r"""
#include <cstdio>
#include "ktanh_order.h"
using namespace ktanh_device;
int main()
{
    constexpr unsigned long long MiB = 1ull << 20;
    for (unsigned long long moved : {1ull, 13 * MiB, 64 * MiB - 2}) if (!plain_elementwise_loads(moved, true)) return 1;
    for (unsigned long long moved : {64 * MiB, 67 * MiB, 96 * MiB, 100 * MiB, 1ull << 40}) if (plain_elementwise_loads(moved, true)) return 2;
    for (unsigned long long moved : {1ull, 64 * MiB, 96 * MiB}) if (!plain_elementwise_loads(moved, false) || !plain_gradient_loads(moved, false)) return 3;
    for (unsigned long long moved : {96 * MiB + 2, 1ull << 40}) if (plain_elementwise_loads(moved, false) || plain_gradient_loads(moved, false)) return 4;
    for (unsigned long long moved : {1ull, 48 * MiB, 60 * MiB, 96 * MiB, 1ull << 40}) if (plain_gradient_loads(moved, true)) return 5;
    for (unsigned long long moved : {1ull, 13 * MiB - 2}) if (gelu_words_in_turn(moved)) return 6;
    for (unsigned long long moved : {13 * MiB, 144 * MiB, 1ull << 40}) if (!gelu_words_in_turn(moved)) return 7;
    std::puts("ok");
    return 0;
}
"""


def test_plain_loads_only_where_they_pay(tmp_path):
    src, exe = tmp_path / "lines.cpp", tmp_path / "lines"
    src.write_text("#include <initializer_list>\n" + PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0 and done.stdout.strip() == "ok", done.returncode
