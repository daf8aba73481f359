// Calibration eigenvectors: the Newton-Schulz steps that take I + tau E, E skew, to its orthogonal polar factor, and when the way in
// floats ends (host code; the products are in k_calib_all.hpp).
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
    double left;             // X X^T - I behind all steps, at most (but for rounding)
};
// X X^T - I behind an unscaled step, at most, where it was at most u before (u + X X^T <= I: 1 - x^2 = u becomes 3/4 u^2 + 1/4 u^3)
inline double polar_defect(double u) { return u * u * (0.75 + 0.25 * u); }
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
    P.left = 1.0 - low * low;
    if (P.one_more) P.left = polar_defect(P.left);
    return P;
}

// The way in floats has come to a stop once transformations no longer bring |E| below 0.97 of the least so far: four in a row, as the rows
// of wide spectra pass a plateau of up to three (D = 2560, 10^(-12 c / D), r = D: 92, 81, 83, 83, 80, 74 ... 4), or one where V has been
// polished: fp64 halves small angles and more.  A limit of 0.9 of the one before, and of 0.6 below |E| = 10, left spectra early whose angles fall
// all the way, for fp64 to do the rest: calls in ms with sweeps first, with that limit and with this one, D = 2560 and r = D, 10^(-8 c / D)
// 50.7 / 62.9 / 30.4, 10^(-12 c / D) 51.8 / 81.7 / 49.7; D = 1024 and r = D, 10^(-12 c / D) 5.47 / 6.78 / 3.83; D = 256, 10^(-6 c / D) 1.81 / 1.41 /
// 1.10.  Three in a row: 10^(-13 c / D) at D = 2560 1.66 of the time with sweeps first, now 0.92.  Eigenvalues that repeat, where it does
// stop: D = 1024, sixteenfold 8.98 / 6.43 / 6.74, two of them 15.9 / 11.4 / 7.27.
struct FloatWay {
    double best = 1e300;
    int slow = 0;
    bool stuck(double now, bool polished)   // behind every transformation, which started from |E| = now
    {
        slow = now < 0.97 * best ? 0 : slow + 1;
        best = std::min(best, now);
        return slow >= (polished ? 1 : 4);
    }
};

// Bound of V V^T - I, V the product of the factors of the way in floats, in the spectral norm: what their plans leave adds up, and the
// rounding of plain bf16 or of pairs.  (Measured, D = 256 to 2560, 13 spectra, and this bound: 8e-5 to 1.1e-2 and 2.4e-3 to 1.7e-2 behind the factors in
// plain bf16, 1e-6 to 2.3e-3 and 4e-5 to 2.5e-3 at the end; the largest ones are 0.7 and 0.9 of their bounds.)
struct FloatDefect {
    double u = 0.0;
    void factor(const PolarPlan& P, bool plain) { u += P.left + u * P.left + (plain ? 5e-4 : 1e-4); }
    void polish() { u = polar_defect(u) + 3e-6; }
    // One more step in fp32 leaves what the correction in fp64 takes out to rounding (at most 1e-5, see k_calib_all.hpp)
    bool correctable() const { return polar_defect(u) <= 1e-5; }
};

// The way in floats is not begun where the rows of the factor are nearly orthogonal as they are, or of nearly equal norms (kFloatSpread of each
// other): eigenvalues that close are told apart in fp64 only, and the polar factors' rounding would mix them (eigenvalues within 1e-3: 6.3
// ms, and 4.8).  Nor where fewer pairs of rows than there are rows have an angle: a sweep passes over almost all pairs of blocks then, and turns
// those (D / 2 planes of two channels turned by 0.1: D = 256 0.37 ms with a sweep, 0.55 with floats, 2048 3.5 and 5.2, 2560 7.0 and 9.8; a
// covariance of tokens has them all).
// now: |E| behind the steps next to blocks; open: its angles, counted; norm: of the rows, descending
constexpr double kFloatFirst = 0.1, kFloatSpread = 0.9;
inline bool float_begins(double now, double open, const double* norm, int D)
{
    return now > kFloatFirst && norm[D - 1] <= kFloatSpread * norm[0] && open >= D;
}

// Rows whose angles the way in floats looks at: the r leading ones, but none of a norm below 4e-6 of the largest (norm: descending).  Their
// products with leading rows are rounding in fp32, and those among themselves would keep it from its end: a covariance of 4/5 D tokens, D =
// 512 and r = D, 4.16 ms with all rows, 2.61 so, 3.82 with sweeps first.  (1e-6: 2.43, but half of all eigenvalues zero, r = 5/8 D, 3.13 in
// place of 2.77.)
inline int float_lead(const double* norm, int r)
{
    while (r > 1 && norm[r - 1] < 4e-6 * norm[0]) --r;
    return r;
}

}  // namespace sals
