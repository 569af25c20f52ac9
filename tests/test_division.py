"""Quotients by a kept reciprocal (csrc/division.hpp), compiled for the CPU, against
quad-precision quotients: the error bounds that the header states, with the
hardware's reciprocal replaced by one that is off by up to 2^-23.  No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#define __device__
#define __forceinline__ inline
static uint64_t s = 88172645463325252ull;
static uint64_t rnd() { s ^= s << 13; s ^= s >> 7; s ^= s << 17; return s; }
static double rcp_off(double d)
{
    return (1.0 / d) * (1.0 + 0x1p-23 * ((double)(int64_t)rnd() * 0x1p-63));
}
#define __builtin_amdgcn_rcp rcp_off
#include "division.hpp"
typedef __float128 Q;
static double ulp(double x)  // unit in the last place of the exact value's binade
{
    int e;
    std::frexp(x, &e);
    return std::ldexp(1.0, e - 53);
}
static double units(double got, Q want) { Q d = ((Q)got - want) / (Q)ulp((double)want); return (double)(d < 0 ? -d : d); }
static double number(int range)
{
    // mantissas at random, and near the ends and the middle of a binade
    const uint64_t k = rnd();
    uint64_t m = rnd() >> 12;
    if (k % 8 == 0) m = rnd() % 64;
    if (k % 8 == 1) m = (1ull << 52) - 1 - rnd() % 64;
    if (k % 8 == 2) m = (1ull << 51) + rnd() % 64 - 32;
    return std::ldexp(1.0 + (double)m * 0x1p-52, (int)(rnd() % (2 * range + 1)) - range);
}
int main(int argc, char **argv)
{
    const long n = atol(argv[1]);
    double wr = 0, wq = 0;
    for (long i = 0; i < n; ++i) {
        const double d = number(200), a = (rnd() & 1 ? 1.0 : -1.0) * number(200), r = ibm::recip(d), q = ibm::quot(a, d, r);
        const double er = units(r, (Q)1 / (Q)d), eq = units(q, (Q)a / (Q)d);
        wr = er > wr ? er : wr;
        wq = eq > wq ? eq : wq;
    }
    printf("%.17g %.17g\n", wr, wq);
    return 0;
}
"""


def test_quotient_and_reciprocal_bounds(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    (tmp_path / "d.cpp").write_text(SRC)
    exe = str(tmp_path / "d")
    r = subprocess.run([gxx, "-std=c++17", "-O2", "-ffp-contract=off", "-I",
                        os.path.join(ROOT, "paper_2605_04335_amd", "csrc"), str(tmp_path / "d.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe, "2000000"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    wr, wq = (float(v) for v in r.stdout.split())
    # (IEEE division: 1/2; more needs a quotient that close to halfway between two numbers)
    assert wr <= 0.5 + 2.0 ** -35 and wq <= 0.5 + 2.0 ** -50
