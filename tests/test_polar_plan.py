"""The host's plan of the steps to an orthogonal polar factor (polar_plan.hpp): it ends for whatever sums the device returns, and the
steps take every singular value to where the last one leaves X X^T - I as small as stated.  And the rule that ends the way in floats."""
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


LEAD = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "polar_plan.hpp"
// arguments: r, norms in descending order
int main(int argc, char** argv)
{
    std::vector<double> norm;
    for (int i = 2; i < argc; ++i) norm.push_back(std::strtod(argv[i], nullptr));
    std::printf("%d\n", sals::float_lead(norm.data(), std::atoi(argv[1])));
}
"""


@pytest.mark.parametrize("r,norms,lead", [(4, [2, 1, 1e-3, 1e-5], 4), (4, [2, 1, 1e-3, 7.9e-6], 3), (3, [2, 1, 1e-3, 1e-9], 3), (2, [1, 1e-9], 1),
                                          (1, [0, 0], 1), (2, [0, 0], 2), (3, [1e150, 1e146, 1e144], 2)])
def test_rows_that_floats_tell_apart(tmp_path, r, norms, lead):
    (tmp_path / "lead.cpp").write_text(LEAD)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, "-o", str(tmp_path / "lead"), str(tmp_path / "lead.cpp")], check=True)
    assert int(subprocess.run([str(tmp_path / "lead"), str(r), *map(repr, norms)], check=True, capture_output=True, text=True, timeout=10).stdout) == lead


BEGIN = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "polar_plan.hpp"
// arguments: |E|, number of angles, norms in descending order
int main(int argc, char** argv)
{
    std::vector<double> norm;
    for (int i = 3; i < argc; ++i) norm.push_back(std::strtod(argv[i], nullptr));
    std::printf("%d\n", (int)sals::float_begins(std::strtod(argv[1], nullptr), std::strtod(argv[2], nullptr), norm.data(), (int)norm.size()));
}
"""


def test_where_the_way_in_floats_begins(tmp_path):
    """Not from rows that are nearly orthogonal, not among nearly equal norms, not for a handful of angles."""
    (tmp_path / "begin.cpp").write_text(BEGIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, "-o", str(tmp_path / "begin"), str(tmp_path / "begin.cpp")], check=True)

    def begins(now, angles, norms):
        return subprocess.run([str(tmp_path / "begin"), repr(now), repr(angles), *map(repr, norms)], check=True, capture_output=True, text=True,
                              timeout=10).stdout.strip() == "1"
    norms = [1.0, 0.8, 0.3, 0.1]
    assert begins(2.0, 6, norms) and begins(2.0, 4, norms)
    assert not begins(2.0, 3, norms)                        # fewer angles than rows
    assert not begins(0.1, 6, norms)
    assert not begins(2.0, 6, [1.0, 0.99, 0.95, 0.91]) and begins(2.0, 6, [1.0, 0.99, 0.95, 0.9])
    assert not begins(2.0, 6, [1.0, 0.8, 0.3, float("nan")])


WAY = r"""
#include <cstdio>
#include <cstdlib>
#include "polar_plan.hpp"
// arguments: |E| of one transformation after the other, "p" once V has been polished; prints how many were made before it came to a stop
int main(int argc, char** argv)
{
    sals::FloatWay way;
    bool polished = false;
    int n = 0;
    for (int i = 1; i < argc; ++i) {
        if (argv[i][0] == 'p') { polished = true; continue; }
        ++n;
        if (way.stuck(std::strtod(argv[i], nullptr), polished)) { std::printf("%d\n", n); return 0; }
    }
    std::printf("0\n");
}
"""


@pytest.fixture(scope="module")
def stop(tmp_path_factory):
    d = tmp_path_factory.mktemp("way")
    (d / "way.cpp").write_text(WAY)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, "-o", str(d / "way"), str(d / "way.cpp")], check=True)
    return lambda norms: int(subprocess.run([str(d / "way"), *map(str, norms)], check=True, capture_output=True, text=True, timeout=10).stdout)


@pytest.mark.parametrize("norms", [
    [15.7, 10.8, 6.4, 3.8, 1.9, "p", 0.48, 0.006],                       # D = 256: a ratio of 0.6 below ten all the way
    [14.8, 9.0, 5.6, 3.4, "p", 1.2, 0.1],
    [121, 110, 101, 91, 81, 70, 58, 47, 34, 22, 13, 5.4, 1.2, "p", 0.12, 0.001],   # 1 / c^2, D = 2560: a slow beginning
    [91.7, 81.1, 83.4, 82.6, 80.3, 73.8, 64, 50, 30, 10, 2, "p", 0.1]])  # twelve decades: a plateau
def test_the_way_in_floats_goes_on_while_angles_fall(stop, norms):
    assert stop(norms) == 0


@pytest.mark.parametrize("norms,ends", [
    ([103, 67.8, 44.7, 40.7, 66.9, 57, 64, 60, 62], 8),                  # eigenvalues that repeat
    ([40, 20, 10, 20, 10, 20, 10, 20], 7),                               # up and down
    ([30, 10, 3, "p", 1.5, 1.6, 0.1], 5),                                # the rest behind the polish is for fp64
    ([5] * 9, 5)])
def test_the_way_in_floats_ends(stop, norms, ends):
    assert stop(norms) == ends
