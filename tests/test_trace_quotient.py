"""The tracer's quotients by the majorant, from the library's own header on the host: equal to the division for
every majorant that the walks use (a NaN there would let a ray go on for ever), and majorants below the least
positive float walked as 0."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2404_11894_amd", "csrc", "pg_quotient.h")

PROGRAM = r"""
#include "pg_quotient.h"
#include <cstdio>
#include <cstdlib>
#include <random>
int main(int, char** argv) {
    const double given = std::strtod(argv[1], nullptr), m = pg::walked_majorant(given);
    std::printf("%a\n", m);
    if (!(m > 0.0)) return 0;
    const double y = 1.0 / m;
    std::mt19937_64 rng(7);
    long bad = 0, infinite = 0;
    for (int i = 0; i < 200000; ++i) {
        double u = (double)(rng() >> 11) * 0x1p-53;
        if (i < 64) u = i < 32 ? (double)i * 0x1p-53 : 1.0 - (double)(i - 31) * 0x1p-53;
        const double a = i % 2 ? std::log(1.0 - u) : (double)(float)(u * (m < 3e38 ? m : 3e38));
        const double q = pg::div_by(a, m, y), d = a / m;
        infinite += !std::isfinite(q);
        // a subnormal quotient (majorants above 1e285) only has to be as small
        bad += !(q == d || (std::fabs(d) < 0x1p-1000 && std::fabs(q) < 0x1p-999));
    }
    std::printf("%ld %ld\n", bad, infinite);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("quotient")
    src, exe = d / "quotient.hip", d / "quotient"
    src.write_text(PROGRAM)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "--offload-host-only", "-std=c++17", "-O2", "-ffp-contract=off", "-I", os.path.dirname(HEADER),
                    str(src), "-o", str(exe)], check=True, capture_output=True)
    return str(exe)


def run(program, m):
    return subprocess.run([program, repr(m)], check=True, capture_output=True, text=True).stdout.split()


@pytest.mark.parametrize("m", [2.0 ** -149, 1e-40, 1.1754943508222875e-38, 1e-30, 1e-9, 0.3, 1.0, 8.0, 32.0, 63.7, 1e6,
                               1e30, 3.4028234663852886e38, 1e100, 1e300])
def test_quotients_equal_the_division(program, m):
    walked, bad, infinite = run(program, m)
    assert float.fromhex(walked) == m
    assert (int(bad), int(infinite)) == (0, 0)


@pytest.mark.parametrize("m", [0.0, 5e-324, 2.2250738585072014e-308, 1.2e-307, 1e-300, 1e-46, 2.0 ** -150])
def test_majorants_of_no_float_are_walked_as_zero(program, m):
    assert [float.fromhex(x) for x in run(program, m)] == [0.0]
