"""The small-angle polynomials of the kernels' phase and damping (csrc/phase.h)
against extended precision, on the CPU: the host pass of the header is built
with hipcc and the same coefficients are evaluated in 80-bit arithmetic, whose
own rounding (1e-19 per operation, 5e-19 allowed) is far below what is
checked, so the bounds below are those that the header states for its
coefficients."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

DRIVER = r"""
#include <cmath>
#include <cstdio>
#include "phase.h"
using namespace bemtx;
typedef long double L;
template <bool SHORT> void run(L top)
{
    L es = 0, ec = 0, ee = 0;
    for (int i = -4000; i <= 4000; ++i) {
        const L t = top * i / 4000;
        L s, c;
        small_sincos<SHORT>(t, s, c);
        if (i) es = std::fmax(es, std::fabs((s - std::sin(t)) / t));
        ec = std::fmax(ec, std::fabs(c - std::cos(t)));
        ee = std::fmax(ee, std::fabs(small_exp<SHORT>(t) - std::exp(t)));
    }
    std::printf("%.3Le %.3Le %.3Le\n", es, ec, ee);
}
int main()
{
    run<false>(1);
    run<true>(kShortPhase);
    double es = 0, ec = 0;
    for (int i = -4000; i <= 4000; ++i) {
        const double t = i / 4000.0;
        double s, c;
        small_sincos_f32(t, s, c);
        if (i) es = std::fmax(es, std::fabs((s - std::sin(t)) / t));
        ec = std::fmax(ec, std::fabs(c - std::cos(t)));
    }
    std::printf("%.3e %.3e 0\n", es, ec);
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
def test_small_angle_polynomials(tmp_path):
    src = tmp_path / "driver.cpp"
    src.write_text(DRIVER)
    exe = str(tmp_path / "driver")
    subprocess.check_call([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-x", "hip",
                           "-I", os.path.join(ROOT, "paper_2206_00708_amd", "csrc"), str(src), "-o", exe])
    got = [[float(v) for v in line.split()]
           for line in subprocess.check_output([exe], text=True).splitlines()]
    rounding = 5e-19
    # sin(t)/t, cos t and exp(t): |t| <= 1, the short range, FP32
    bounds = [(2e-19, 3e-18, 5e-18), (2e-18, 1e-20, 1e-18), (4e-10, 2e-9, 0)]
    for g, b in zip(got, bounds):
        assert all(x <= y + rounding for x, y in zip(g, b)), (g, b)
