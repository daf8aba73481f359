"""The host's plan of the steps to an orthogonal polar factor (polar_plan.hpp): it ends for whatever sums the device returns, and the
steps take every singular value to where the last one leaves X X^T - I as small as stated."""
import os
import subprocess

import numpy as np
import pytest

from paper_2510_24273_amd import build

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "polar_plan.hpp"
int main(int argc, char** argv)
{
    for (int i = 1; i < argc; ++i) {
        const sals::PolarPlan P = sals::polar_plan(std::strtod(argv[i], nullptr));
        std::printf("%d %d %.17g %.17g", P.n, (int)P.one_more, P.tau, P.top);
        for (int k = 0; k < P.n; ++k) std::printf(" %.17g", P.a[k]);
        std::printf("\n");
    }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("polar")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, "-o", str(d / "plan"), str(d / "plan.cpp")], check=True)

    def run(sums):
        out = subprocess.run([str(d / "plan"), *map(repr, sums)], check=True, capture_output=True, text=True, timeout=10).stdout
        return [[float(x) for x in line.split()] for line in out.splitlines()]
    return run


def test_sums_that_are_no_numbers_have_no_plan(plans):
    for P in plans([float("nan"), float("inf"), float("-inf"), -1.0]):
        assert P[0] == 0


def test_every_plan_reaches_the_orthogonal_factor(plans):
    """|E| from 0 to far above where it is scaled down, and what rounding makes of a bound: singular values from 1 to the bound."""
    bounds = [0.0, 1e-300, 1e-8, 0.01, 0.054, 0.055, 0.056, 0.1, 0.5, 1.0, 2.0, 5.999, 6.0, 6.001, 50.0, 4096.0, 1e70]
    for bound, P in zip(bounds, plans([b ** 4 for b in bounds])):
        n, one_more, tau, top, a = int(P[0]), bool(P[1]), P[2], P[3], P[4:]
        assert 1 <= n <= 6 and len(a) == n, (bound, P)
        assert 0.0 < tau <= 1.0 and tau * bound <= 6.0 * (1 + 1e-12)
        x = np.sqrt(1.0 + np.linspace(0.0, tau * bound, 1001) ** 2) / top
        for s in a:
            x = 1.5 * s * x - 0.5 * (s * x) ** 3
        if one_more:
            x = 1.5 * x - 0.5 * x ** 3
        assert np.max(np.abs(x * x - 1.0)) <= 7e-6, (bound, P)
