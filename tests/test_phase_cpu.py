"""The phase of the per-point potential factor (csrc/phase.hpp), compiled for the host and
checked against exp(-i theta) in long double.

Tolerance: the reduction's three fused steps round at the size of what they leave, at most
pi plus 2 pi - 6.28125 = 0.0019 per turn (half an ulp each), then the two series and their
sum round below 1 three times: 3 ulp(pi) / 2 + 3 ulp(1) + 2^-53 * 0.0019 |theta| / pi.
CPU only: this runs no GPU code."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_1903_02581_amd", "csrc", "phase.hpp")

SHIM = """
#pragma once
#include <cmath>
#define __device__
#define __host__
#define __forceinline__ inline
struct double2 { double x, y; };
inline double2 make_double2(double a, double b) { return {a, b}; }
using std::fma; using std::rint; using std::fabs;
"""

DRIVER = r"""
#include "HEADER"
#include <cstdio>
#include <random>
using namespace hom4d_impl::dev;
int main() {
    std::mt19937_64 g(7);
    const double size[] = {1e-9, 0.1, 1.0, 4.0, 100.0, 1e4, 1e8};
    for (double a : size) {
        std::uniform_real_distribution<double> u(-a, a);
        double err = 0.0;
        for (int i = 0; i < 200000; ++i) {
            double th = u(g);
            if (i % 4 == 0) th = std::rint(th / 0.7853981633974483) * 0.7853981633974483;  // the seams
            const double2 f = expmi(th);
            err = std::fmax(err, std::hypot((double)(f.x - cosl((long double)th)), (double)(f.y + sinl((long double)th))));
        }
        std::printf("%.17g %.3e\n", a, err);
    }
    const double far[] = {1e15, -3e20, 1e300};
    for (double th : far) { const double2 f = expmi(th); std::printf("far %.17g\n", std::hypot(f.x, f.y)); }
    return 0;
}
"""


def test_expmi(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    os.makedirs(tmp_path / "hip")
    (tmp_path / "hip" / "hip_runtime.h").write_text(SHIM)
    (tmp_path / "t.cpp").write_text(DRIVER.replace("HEADER", HEADER))
    exe = str(tmp_path / "t")
    res = subprocess.run([gxx, "-O2", "-std=c++17", "-I", str(tmp_path), str(tmp_path / "t.cpp"), "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
    near = 0
    for line in out.split("\n"):
        if line.startswith("far"):
            assert abs(float(line.split()[1]) - 1.0) <= 1e-15, line
        elif line.strip():
            a, err = map(float, line.split())
            assert err <= 1.5 * 2.0 ** -51 + 3.0 * 2.0 ** -53 + 2.0 ** -53 * 0.0019 * a / 3.0, line
            near += 1
    assert near == 7
