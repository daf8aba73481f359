// Calibration eigenvectors: the Newton-Schulz steps that take I + tau E, E skew, to its orthogonal polar factor (host code; the
// products are in k_calib_all.hpp).
//
// A step takes every singular value x of X to 3/2 a x - 1/2 (a x)^3, with a^2 = 3 / (1 + l + l^2) for values between l and 1 (J. Chen,
// E. Chow, "A stable scaling of Newton-Schulz for improving the sign function computation of a Hermitian matrix", 2014).  Those of I +
// tau E lie between 1 and sqrt(1 + tau^2 |E|^2).
#pragma once
#include <algorithm>
#include <cmath>

namespace sals {

// |E| at most: larger angles gain nothing (4, 6 and 10: 5.13, 5.11 and 5.11 ms at D = 1024; 5.43, 5.25, 5.28 with a spectrum c^-2)
constexpr double kAllCap = 6.0;
// Singular values from here on need one more step, which leaves 3/4 (1 - x^2)^2 = 7e-6 of X X^T - I
constexpr double kPolarNear = 0.9985;
// Rows in floats: up to this D, and singular values of their polar factors one step further from here on, which leaves 3 e-3 of X X^T - I (as
// good as 7e-6: 3.6 ms at D = 1024 with either, but three steps instead of four; 0.9 takes more transformations)
constexpr int kFloatMaxD = 2560;
constexpr double kFloatPolar = 0.97;
constexpr int kPolarSteps = 6;   // steps up to there, at most (kAllCap takes three)

struct PolarPlan {
    int n;                   // scaled steps; 0: there is no such transformation
    bool one_more;           // an unscaled step behind them
    double tau, top;         // X starts as (I + tau E) / top
    double a[kPolarSteps];   // the steps' scales
};
// a2: sum of squares of E E^T, of which the fourth root bounds |E|.  What is no number, or infinite, has no plan.  The scaled steps end
// with singular values from `near` on.
inline PolarPlan polar_plan(double a2, double near = kPolarNear)
{
    PolarPlan P{};
    if (!std::isfinite(a2) || a2 < 0.0) return P;
    const double bound = std::sqrt(std::sqrt(a2));
    P.tau = bound > kAllCap ? kAllCap / bound : 1.0;
    const double tb = P.tau * bound;
    P.top = std::sqrt(1.0 + tb * tb);
    double low = 1.0 / P.top;
    P.one_more = low < near;   // (angles so small to begin with are done by the first step)
    do {
        if (P.n == kPolarSteps) return PolarPlan{};
        const double a = low < near ? std::sqrt(3.0 / (1.0 + low + low * low)) : 1.0, x = a * low;
        P.a[P.n++] = a;
        low = 0.5 * x * (3.0 - x * x);
    } while (low < near);
    return P;
}

}  // namespace sals
