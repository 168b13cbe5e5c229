"""The forms in which the kernels evaluate the comparison approximants (csrc/ktanh_approx.h), compiled for
the CPU: rounded to BFloat16 they are the oracle's results on every magnitude of the regions they serve,
and Pade's do not depend on the last two units of the hardware's reciprocal."""
import subprocess

import numpy as np
import pytest

from paper_1909_07729_amd import build

PROGRAM = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "ktanh_approx.h"
using namespace ktanh_device;
static float value(uint32_t u) { float v; std::memcpy(&v, &u, 4); return v; }
static uint32_t bits(float v) { uint32_t u; std::memcpy(&u, &v, 4); return u; }
static uint16_t narrow(float v) { const uint32_t u = bits(v); return (uint16_t)((u + 0x7FFF + ((u >> 16) & 1)) >> 16); }
int main(int, char **argv)
{
    const int which = std::atoi(argv[1]), off = std::atoi(argv[2]);
    auto rcp = [off](float d) { return value(bits((float)(1.0 / (double)d)) + off); };
    for (uint32_t m = 0; m <= 0x7F80; ++m) {
        uint16_t r;
        if (which == 32) r = narrow(pade_of_magnitude<false>(value((m > 0x4080 ? 0x4080 : m) << 16), rcp));
        else if (which == 78) r = narrow(pade_of_magnitude<true>(value((m > 0x40B0 ? 0x40B0 : m) << 16), rcp));
        else if (m < 0x3E80) r = (uint16_t)m;
        else {
            const uint32_t in = m > 0x4080 ? 0x4080 : m, mid = (in & 0x7FF0) | 8;
            const float y = in == 0x4080 ? 1.0f : (float)std::tanh((double)value(mid << 16));
            const float h = value(in << 16) - value(mid << 16);
            r = narrow(which == 2 ? taylor_at<2>(h, y) : taylor_at<3>(h, y));
        }
        std::fwrite(&r, 2, 1, stdout);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    folder = tmp_path_factory.mktemp("approx")
    src, exe = folder / "approx.cpp", folder / "approx"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wall", "-Wextra", "-I", build.CSRC, str(src),
                    "-o", str(exe)], check=True)
    return str(exe)


@pytest.mark.parametrize("which,offsets", [(32, (-2, -1, 0, 1, 2)), (78, (-2, -1, 0, 1, 2)), (2, (0,)), (3, (0,))])
def test_forms_give_the_oracle_s_results(program, oracle, which, offsets):
    x = np.arange(0x7F81, dtype=np.uint16)
    want = {32: oracle.kpade32, 78: oracle.kpade78, 2: oracle.ktaylor2, 3: oracle.ktaylor3}[which](x)
    for off in offsets:
        done = subprocess.run([program, str(which), str(off)], capture_output=True, timeout=60, check=True)
        assert np.array_equal(np.frombuffer(done.stdout, dtype=np.uint16), want), off
