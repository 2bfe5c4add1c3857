"""Host check of cos(pi a) alone (fd_elem.hpp), the third Gaussian component of every
FP64 pair: compiled for the host and compared with long-double libm over [0, 2], at the
multiples of 2^-32 that the draws use, and close to the ends, the zeros and the extremes.
One polynomial of eleven terms in r^2 <= 1/4, largest 3.14 |r|, each rounded to 2^-53 of
partial sums below 2: a few units of 2^-53 (the bar of the other sine and cosine, 8)."""
import os
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1707_04232_amd", "csrc")

PROGRAM = r"""
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_rcp(x) (1.0 / (x))
#define __builtin_amdgcn_rsq(x) (1.0 / sqrt(x))
#define __ballot(p) ((unsigned long long)((p) ? 1 : 0))
#include "fd_elem.hpp"
static uint64_t s = 0x9E3779B97F4A7C15ull;
static uint64_t rnd() { s ^= s << 13; s ^= s >> 7; s ^= s << 17; return s; }
static double worst = 0.0;
static void check(double a) {
    if (!(a >= 0.0 && a <= 2.0)) return;
    const long double pl = 3.14159265358979323846264338327950288L;
    const long double want = cosl(pl * (long double)a);
    const double e = (double)fabsl((long double)sdpd::fd_cospi(a) - want) / 0x1p-53;
    if (!(e <= worst)) worst = e;   // (a NaN stays)
}
int main() {
    for (int k = 0; k < 2000000; ++k) {
        check((double)(rnd() >> 11) * 0x1p-52);                             // any double
        check(2.0 * fma((double)(uint32_t)(rnd() >> 16), 0x1p-32, 0x1p-33)); // of a draw
    }
    const double at[] = {0.0, 0.25, 0.5, 0.75, 1.0, 1.25, 1.5, 1.75, 2.0};
    for (double c : at)
        for (int e = 0; e <= 60; ++e) {
            check(c + ldexp(1.0, -e));
            check(c - ldexp(1.0, -e));
            check(c);
            check(nextafter(c, 4.0));
            check(nextafter(c, -4.0));
        }
    printf("%g\n", worst);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_cospi_within_a_few_units():
    with tempfile.TemporaryDirectory() as d:
        src, exe = os.path.join(d, "cospi.cpp"), os.path.join(d, "cospi")
        with open(src, "w") as f:
            f.write(PROGRAM)
        subprocess.run(["g++", "-O2", "-ffp-contract=off", "-std=c++17", "-I", CSRC, src, "-o",
                        exe, "-lm"], check=True)
        out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
    print("max error of cos(pi a) in 2^-53:", out.strip())
    assert float(out) <= 8.0
