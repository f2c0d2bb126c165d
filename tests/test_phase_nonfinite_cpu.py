"""The phase of the per-point potential factor at infinite and NaN angles (NaN, so that the
state's norm shows it) and at the ends of the finite range (a unit number), compiled for the
host.  CPU only: this runs no GPU code."""
import os
import shutil
import subprocess

import pytest

from tests.test_phase_cpu import HEADER, SHIM

DRIVER = r"""
#include "HEADER"
#include <cstdio>
#include <initializer_list>
#include <limits>
using namespace hom4d_impl::dev;
int main() {
    const double inf = std::numeric_limits<double>::infinity(), nan = std::numeric_limits<double>::quiet_NaN();
    for (double th : {inf, -inf, nan, -nan}) {
        const double2 f = expmi(th);
        std::printf("none %d\n", f.x != f.x && f.y != f.y);
    }
    const double least = std::numeric_limits<double>::denorm_min();
    for (double th : {0.0, -0.0, least, -least, 1e-300, 1e14, -1e15, 1e200}) {
        const double2 f = expmi(th);
        std::printf("unit %.17g\n", std::hypot(f.x, f.y));
    }
    return 0;
}
"""


def test_expmi_out_of_range(tmp_path):
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
    out = [line.split() for line in subprocess.run([exe], capture_output=True, text=True,
                                                   check=True).stdout.splitlines()]
    assert [float(v) for k, v in out if k == "none"] == [1.0] * 4
    unit = [float(v) for k, v in out if k == "unit"]
    assert len(unit) == 8 and all(abs(u - 1.0) <= 1e-15 for u in unit)
