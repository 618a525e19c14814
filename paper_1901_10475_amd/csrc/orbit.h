// orbit.h -- Kepler propagation shared by the box and narrow-phase kernels.
//
// An object's position at time t (Sec. 7.1): the mean anomaly advances
// linearly, M = m0 + n t with n = sqrt(mu / a^3); Kepler's equation
// E - e sin E = M gives the eccentric anomaly (the exact solution of the
// true-anomaly ODE, Eq. nu-dot); in the orbit's plane the position is
// (a (cos E - e), b sin E), b = a sqrt(1 - e^2), and the three rotations
// R_z(raan) R_x(i) R_z(argp) take the plane's axes to ECI (vectors P, Q).
#pragma once
#include "cd_internal.h"

namespace cd {

// Per-object constants, with m0 advanced to the horizon's start.
__device__ inline ObjConst object_const(double a, double e, double inc, double raan,
                                        double argp, double m0, double mu, double start_s)
{
    double ci, si, cO, sO, cw, sw;
    sincos(inc, &si, &ci);
    sincos(raan, &sO, &cO);
    sincos(argp, &sw, &cw);
    ObjConst c;
    c.a = a;
    c.e = e;
    c.b = a * sqrt(1.0 - e * e);
    c.n = sqrt(mu / (a * a * a));
    c.m0 = m0 + c.n * start_s;
    c.vmax = sqrt(mu * (1.0 + e) / (a * (1.0 - e)));   // perigee speed, the largest
    // R_z(raan) R_x(inc) R_z(argp) applied to the perifocal x and y axes
    c.P[0] = cO * cw - sO * sw * ci;
    c.P[1] = sO * cw + cO * sw * ci;
    c.P[2] = sw * si;
    c.Q[0] = -cO * sw - sO * cw * ci;
    c.Q[1] = -sO * sw + cO * cw * ci;
    c.Q[2] = cw * si;
    return c;
}

// The cold start's single precision: the hardware's sine, cosine and reciprocal,
// since only a guess is formed from them (on the host, where the tests run the
// solver, the library's).
__host__ __device__ inline float start_sin(float x)
{
#ifdef __HIP_DEVICE_COMPILE__
    return __sinf(x);
#else
    return sinf(x);
#endif
}
__host__ __device__ inline float start_slope(float e, float x)   // dE/dM at x
{
#ifdef __HIP_DEVICE_COMPILE__
    return __builtin_amdgcn_rcpf(1.0f - e * __cosf(x));
#else
    return 1.0f / (1.0f - e * cosf(x));
#endif
}

// Cold start of Kepler's equation E - e sin E = M: delta = E - M solved by
// Newton in single precision on the reduced mean anomaly (|delta| <= e), good
// to about 1e-6, which is all that the double-precision step below needs.
__host__ __device__ inline double kepler_start(double M, double e)
{
    const double turn = 6.283185307179586476925286766559;
    const float m = (float)(M - turn * rint(M * 0.15915494309189533577));
    const float ef = (float)e;
    float x = ef * start_sin(m) * start_slope(ef, m);
    x = fminf(fmaxf(x, -ef), ef);
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        x -= (x - ef * start_sin(m + x)) * start_slope(ef, m + x);
        x = fminf(fmaxf(x, -ef), ef);
    }
    return M + (double)x;
}

// Warm start dM past a solved point (E, sin E, q = dE/dM): the second-order
// Taylor step.  Good for short steps only; of long steps of eccentric orbits
// the solve below drops it.
__host__ __device__ inline double kepler_next(double E, double sE, double q, double e, double dM)
{
    const double x = q * dM;
    return E + (x - 0.5 * (e * q) * sE * x * x);
}

// Kepler's equation E - e sin E = M from the guess in E (cold: from the cold
// start, formed in the one place where the restart below forms it); returns E, sin
// E, cos E and q = dE/dM = 1 / (1 - e cos E) (q near E, for the next guess).
//
// One sincos per solve.  With f = E - e sin E - M and d1 = f q the root lies
// at E - d, d = d1 (1 + a + 2 a^2 - b) + O(d1^4), a = e sin E q d1 / 2,
// b = e cos E q d1^2 / 6 (the reversed Taylor series of f); the step is
// accepted when a bound on the fourth-order term is below 1e-17, and sin and
// cos at the root come from the addition theorem with |d| <= 1e-3.  Guesses
// good to 1e-4 pass at once: the cold start up to e = 0.65 (more than eight in
// ten beyond), the warm one up to dM = 0.05 at e = 0.3 or 0.1 at e = 0.1.  f is formed from
// E - M, which is exact, so sin and cos are those of the root itself and not
// of its rounded value: rms error against 80-bit arithmetic 5.4e-17 for M up
// to 6.3 and 6.8e-17 for M up to 3000, where Newton to a fixed point (2 to 4
// sincos per solve) has 1.8e-16 and 8.5e-14.
//
// Newton from a guess far from the root may wander without end where 1 - e cos E
// is small (of a million solves at e = 0.65 and dM = 1.5, 1 700 did not end in
// 40 turns), so a guess that has not passed in kKeplerGuess turns gives way to
// the cold start, and every later turn stays within |E - M| <= e, which holds
// the root: at most 9 turns for e up to 0.999, 38 for 1 - e = 1e-12.  Both are
// marked as the rare case, which keeps them out of the way of the usual one (the
// per-object boxes of the 50 km steps 200 us without the marks, 129 registers and
// three waves; with them 180, 126 and four, as without the restart).
constexpr int kKeplerGuess = 3, kKeplerTurns = 100;
__host__ __device__ inline void kepler(double M, double e, double &E, double &sE, double &cE,
                                       double &q, bool cold = false)
{
    for (int turn = 1; turn <= kKeplerTurns; ++turn) {
        if (__builtin_expect(cold, 0))
            E = kepler_start(M, e);
        cold = turn == kKeplerGuess;
        double s, c;
        sincos(E, &s, &c);
        q = 1.0 / (1.0 - e * c);
        const double d1 = ((E - M) - e * s) * q;
        const double h = e * q * d1;
        const double a = 0.5 * s * h;
        const double b = c * h * d1 * (1.0 / 6.0);
        const double d = d1 * (1.0 + (a + (2.0 * a * a - b)));
        const double ad = fabs(d1), ah = fabs(h);
        if (ad <= 1e-3 && ad * ah * (ah * ah + ah * ad + ad * ad) <= 1e-17) {
            const double d2 = d * d;
            const double sd = d - d * d2 * (1.0 / 6.0);
            const double cd = d2 * (d2 * (1.0 / 24.0) - 0.5);   // cos d - 1
            sE = s + (s * cd - c * sd);
            cE = c + (c * cd + s * sd);
            E -= d;
            return;
        }
        E -= (ah < 0.25 && ad < 0.25) ? d : d1;
        if (__builtin_expect(turn > kKeplerGuess, 0))
            E = fmin(fmax(E, M - e), M + e);
    }
    sincos(E, &sE, &cE);
}

__device__ inline void position(const ObjConst &c, double sE, double cE, double p[3])
{
    double u = c.a * (cE - c.e);
    double v = c.b * sE;
    p[0] = u * c.P[0] + v * c.Q[0];
    p[1] = u * c.P[1] + v * c.Q[1];
    p[2] = u * c.P[2] + v * c.Q[2];
}

} // namespace cd
