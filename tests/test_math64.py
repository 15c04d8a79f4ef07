"""The FP64 reciprocal, reciprocal square root and exponential of the anchors'
kernels (rj_math64.h) against 80-bit extended precision on the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <random>
#include "rj_math64.h"
int main() {
    std::mt19937_64 g(1);
    std::uniform_real_distribution<double> u(0.0, 1.0), s(-1.0, 1.0);
    long double rcp = 0, rsq = 0, ex = 0, deep = 0;
    auto rel = [](double got, long double want) { return std::fabs((long double)got / want - 1.0L) * 0x1p53L; };
    for (int i = 0; i < 4000000; ++i) {
        const double x = std::ldexp(1.0 + u(g), (int)(600 * s(g)));
        // a starting value as far off as the hardware's may be, at most 2^-24
        const double d = 1.0 + 0x1p-24 * s(g);
        rcp = std::fmax(rcp, rel(rj::rcp_from(x, (double)(1.0L / x) * d), 1.0L / x));
        rsq = std::fmax(rsq, rel(rj::rsq_from(x, (double)(1.0L / sqrtl(x)) * d), 1.0L / sqrtl(x)));
        double k;
        const double y = i % 2 ? -700.0 * u(g) : 0.3 * s(g);
        const double p = rj::exp_series(y, k);
        ex = std::fmax(ex, rel(std::ldexp(p, (int)k), expl(y)));
        const double z = -745.0 - 1e4 * u(g);
        const double q = rj::exp_series(z, k);
        deep = std::fmax(deep, (long double)std::ldexp(q, (int)std::fmax(k, -3000.0)));
    }
    std::printf("%.6Lf %.6Lf %.6Lf %Lg\n", rcp, rsq, ex, deep);
}
"""


def test_errors_against_extended_precision(tmp_path):
    """In units of 2^-53, relative to the value: the reciprocal's last rounding
    alone (1), the root's with the rounding of x y, which the series halves
    (1.5), the exponential's last rounding, the reduced argument's (0.25), the
    last but one of the series (0.35, and 0.1 for those before) and the series'
    rest (0.04): below 2.  Beyond the smallest number: 0 or that number."""
    (tmp_path / "m.cpp").write_text(SRC)
    subprocess.run(["g++", "-O2", "-std=c++17", "-mfma", "-ffp-contract=off", "-I",
                    os.path.join(ROOT, "paper_1811_04156_amd", "csrc"), "-o", str(tmp_path / "m"),
                    str(tmp_path / "m.cpp")], check=True)
    rcp, rsq, ex, deep = (float(x) for x in subprocess.run([str(tmp_path / "m")], check=True, capture_output=True,
                                                           text=True).stdout.split())
    print(rcp, rsq, ex, deep)
    assert rcp <= 1.0 + 1e-4 and rsq <= 1.5 + 1e-4 and ex <= 2.0
    assert deep <= 5e-324
