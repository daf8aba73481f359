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
#ifndef NEAR
#define NEAR sals::kPolarNear
#endif
int main(int argc, char** argv)
{
    for (int i = 1; i < argc; ++i) {
        const sals::PolarPlan P = sals::polar_plan(std::strtod(argv[i], nullptr), NEAR);
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


DEFECT = r"""
#include <cstdio>
#include <cstdlib>
#include "polar_plan.hpp"
// arguments: bounds of |E|, one factor each ("p": a step in fp32 behind it); prints what their plans leave, and the bound of them all and whether it can
// be corrected, then the same behind one more step
int main(int argc, char** argv)
{
    sals::FloatDefect d;
    bool plain = true;
    for (int i = 1; i < argc; ++i) {
        if (argv[i][0] == 'p') { d.polish(); plain = false; continue; }
        const double b = std::strtod(argv[i], nullptr);
        const sals::PolarPlan P = sals::polar_plan(b * b * b * b, sals::kFloatPolar);
        std::printf("%.17g ", P.left);
        d.factor(P, plain);
    }
    std::printf("%.17g %d ", d.u, (int)d.correctable());
    d.polish();
    std::printf("%.17g %d\n", d.u, (int)d.correctable());
}
"""


@pytest.fixture(scope="module")
def defect(tmp_path_factory):
    d = tmp_path_factory.mktemp("defect")
    (d / "defect.cpp").write_text(DEFECT)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, "-o", str(d / "defect"), str(d / "defect.cpp")], check=True)
    return lambda *a: [float(x) for x in subprocess.run([str(d / "defect"), *map(str, a)], check=True, capture_output=True, text=True,
                                                        timeout=10).stdout.split()]


def test_plans_of_the_way_in_floats_leave_what_they_say(tmp_path, defect):
    """The plans that steer: singular values of every size end within the stated bound of one, at most 3/4 (1 - 0.97^2)^2 and its cube."""
    (tmp_path / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-DNEAR=sals::kFloatPolar", "-I", build.CSRC, "-o", str(tmp_path / "plan"), str(tmp_path / "plan.cpp")],
                   check=True)
    bounds = [float(b) for b in np.concatenate([np.geomspace(1e-6, 50.0, 200), np.linspace(0.1, 6.1, 200)])]
    plans = subprocess.run([str(tmp_path / "plan"), *(repr(b ** 4) for b in bounds)], check=True, capture_output=True, text=True, timeout=10).stdout
    worst = 0.0
    for bound, plan, left in zip(bounds, plans.splitlines(), defect(*bounds)):
        n, one_more, tau, top, *a = map(float, plan.split())
        assert 1 <= n <= 6
        x = np.sqrt(1.0 + np.linspace(0.0, tau * bound, 1001) ** 2) / top
        for s in a + [1.0] * int(one_more):
            x = 1.5 * s * x - 0.5 * (s * x) ** 3
        assert np.max(np.abs(x * x - 1.0)) <= left * (1 + 1e-9) + 1e-15, bound
        worst = max(worst, left)
    u = 1 - 0.97 ** 2
    assert 1e-3 < worst <= 0.75 * u * u + 0.25 * u ** 3


def test_what_adds_up_in_floats_is_taken_out_before_the_correction(defect):
    near_one = 2.263                                  # (a plan that leaves about as much as any)
    one = defect(near_one)
    assert one[0] > 1.5e-3 and one[-3] == 1.0         # a single factor can be corrected behind one step in fp32
    *_, u, fine, u1, fine1 = defect("p", near_one, near_one, near_one)
    assert u >= 3 * one[0] and fine == 0.0            # three that line up cannot
    assert u1 <= 0.8 * u * u + 3e-6 and fine1 == 1.0
    *_, u, fine, u1, fine1 = defect(*[near_one] * 40)  # a long way
    assert u >= 40 * one[0] and fine == 0.0 and u1 < 0.2 * u


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
