"""Rounding of the kernels' reciprocals, roots and fast speed (csrc/physics.h
compiled for the host, the hardware's estimates stood in by values off by up to
2^-24, their measured bound), against 113-bit arithmetic (CPU only).

Bounds in ulps.  After two Newton steps on an estimate off by e = 2^-24 (sqrt_pos;
their residuals carry no rounding of the iterate) or one third-order step (e^3 is
left) what counts is roundings: the last operation's, 1/2, and for sqrt_ratio_pos
half of those of g and a g, together 2^-53 of the result, another ulp at most.
The fast speed is to be no further off than in the form with the squared speeds
divided by the density, from correctly rounded parts."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = r"""
#pragma once
#include <cmath>
#include <quadmath.h>
#define __device__
#define __forceinline__ inline
double off();                                     // relative error of the next estimate
inline double __builtin_amdgcn_rsq(double x) { return (double)((1 + (__float128)off()) / sqrtq((__float128)x)); }
inline double __builtin_amdgcn_rcp(double x) { return (double)((1 + (__float128)off()) / (__float128)x); }
using std::fma; using std::fmax; using std::fmin; using std::sqrt; using std::fabs;
"""

MAIN = r"""
#include <cstdio>
#include <random>
#include "physics.h"
typedef __float128 Q;
std::mt19937_64 gen(5);
double U() { return std::uniform_real_distribution<double>(0.0, 1.0)(gen); }
double off() { const int k = gen() % 4; return k == 0 ? 0x1p-24 : k == 1 ? -0x1p-24 : 0x1p-24 * (2 * U() - 1); }
double err(double got, Q want)
{
    const double w = std::fabs((double)want);
    return std::fabs((double)((got - want) / (Q)(std::nextafter(w, INFINITY) - w)));
}
struct Stat {
    double max = 0, sum = 0; long n = 0;
    void add(double e) { max = e > max ? e : max; sum += e; ++n; }
    void put(const char *name) { std::printf("%s %.6f %.6f\n", name, max, sum / n); }
};
double any(int span) { return std::ldexp(1 + U(), (int)(U() * 2 * span) - span); }
int main()
{
    Stat rcp, root, ratio;
    for (int i = 0; i < 400000; ++i) {
        const double x = any(300), a = any(200), y = any(200);
        rcp.add(err(rcp_pos(x), 1 / (Q)x));
        root.add(err(sqrt_pos(x), sqrtq((Q)x)));
        ratio.add(err(sqrt_ratio_pos(y, a), sqrtq((Q)y / a)));
    }
    rcp.put("rcp");
    root.put("sqrt");
    ratio.put("ratio");
    for (int wide = 0; wide < 2; ++wide) {
        Stat now, squared;
        for (int i = 0; i < 400000; ++i) {
            const double g = 1.5, rho = 1e-3 * std::pow(1e5, U()), p = 1e-4 * std::pow(1e6, U());
            const double beta = wide ? 1e-2 * std::pow(1e4, U()) : 0.3 * std::pow(100.0, U());
            const double B = std::sqrt(2 * p / beta), c = 2 * U() - 1, s = std::sqrt(1 - c * c), h = 6.28 * U();
            const double b0 = B * c, b1 = B * s * std::cos(h), b2 = B * s * std::sin(h);
            const Q A = (Q)g * p + (Q)b0 * b0 + (Q)b1 * b1 + (Q)b2 * b2, d = A * A - 4 * (Q)g * p * b0 * b0;
            const Q want = sqrtq((A + sqrtq(d > 0 ? d : 0)) / (2 * (Q)rho));
            const double bb = b0 * b0 + b1 * b1 + b2 * b2;
            now.add(err(fast_speed_of(fma(g, p, bb), 4.0 * g * p, b0, rho + rho), want));
            const double ir = 1.0 / rho, gp = g * p, a = (gp + bb) * ir, q = a * a - 4.0 * gp * b0 * b0 * ir * ir;
            squared.add(err(std::sqrt(0.5 * (a + std::sqrt(q > 0.0 ? q : 0.0))), want));
        }
        now.put(wide ? "speed_wide" : "speed");
        squared.put(wide ? "squared_wide" : "squared");
    }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_roots_and_fast_speed(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(STUB)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "roots")
    subprocess.check_call(["g++", "-O2", "-std=gnu++17", "-mfma", "-ffp-contract=off", "-I", str(tmp_path), "-I",
                           os.path.join(ROOT, "paper_2211_12867_amd", "csrc"), str(tmp_path / "main.cpp"), "-o", exe,
                           "-lquadmath"])
    r = {k: (float(a), float(b)) for k, a, b in
         (line.split() for line in subprocess.check_output([exe], text=True).splitlines())}
    print(r)
    assert r["rcp"][0] < 0.51 and r["sqrt"][0] < 0.51 and r["ratio"][0] < 1.51
    for k in ("", "_wide"):
        assert r["speed" + k][1] <= r["squared" + k][1]
