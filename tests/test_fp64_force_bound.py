"""The stated error of the FP64 force's polynomial: the coefficients of the kernels, the same
sequence of fused multiply-adds, against 113-bit arithmetic (no GPU needed)."""
from __future__ import annotations

import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1409_4923_amd", "csrc")

SRC = r"""
#include <math.h>
#include <quadmath.h>
#include <stdint.h>
#include <stdio.h>
@CONSTANTS@
static double quarter(double x) { return 0.25 - fabs(x - rint(x)); }
static double cos_turns(double x)
{
    const double s = quarter(x), z = s * s;
    double q = SIN_C[7];
    for (int k = 6; k >= 0; --k) q = fma(q, z, SIN_C[k]);
    return fma(s, SIN_C0, s * fma(z, q, SIN_C0_LO));
}
static double force(double x, double A)
{
    const double s = quarter(x), z = s * s;
    double q = FORCE_C[7];
    for (int k = 6; k >= 0; --k) q = fma(q, z, FORCE_C[k]);
    return fma(s, FORCE_C0, fma(s, fma(z, q, FORCE_C0_LO), A));
}
static double cos_err, force_err;
static void look(double x)
{
    const __float128 r = fabsq((__float128)x - rintq(x)), two_pi = 2 * M_PIq;
    const __float128 c = r <= 0.125Q ? cosq(two_pi * r) : sinq(two_pi * (0.25Q - r));
    const double a = fabs((double)(cos_turns(x) - c)), b = fabs((double)(force(x, 0.0) + two_pi * c));
    if (a > cos_err) cos_err = a;
    if (b > force_err) force_err = b;
}
int main(void)
{
    uint64_t u = 88172645463325252ull;
    for (int i = 0; i < @POINTS@; ++i) {
        u ^= u << 13; u ^= u >> 7; u ^= u << 17;
        look((double)(u >> 11) * 0x1p-53 * 3.0 - 1.0);
        look(0.5 + ((double)(u & 0xFFFFFF) - 0x800000) * 0x1p-32);      /* where it is largest */
    }
    printf("%.4g %.4g\n", cos_err, force_err);
    return 0;
}
"""


def constants():
    with open(os.path.join(CSRC, "paths.hpp")) as f:
        text = f.read()
    found = re.findall(r"constexpr double ((?:SIN|FORCE)_C[^;]*);", text)
    assert len(found) == 4
    return "\n".join("static const double " + c + ";" for c in found)


@pytest.mark.parametrize("points", [400_000])
def test_stated_error(tmp_path, points):
    src, exe = str(tmp_path / "t.c"), str(tmp_path / "t")
    with open(src, "w") as f:
        f.write(SRC.replace("@CONSTANTS@", constants()).replace("@POINTS@", str(points)))
    subprocess.check_call(["gcc", "-O2", "-std=gnu11", "-ffp-contract=off", src, "-o", exe, "-lquadmath", "-lm"])
    cos_err, force_err = map(float, subprocess.run([exe], capture_output=True, text=True).stdout.split())
    print(cos_err, force_err)
    # the largest errors found over 100 times these points (the roundings of s, z, the last
    # Horner steps, the product and the result add up to at most 4e-16 and 2 pi times that)
    assert cos_err <= 2.73e-16
    assert force_err <= 1.44e-15
