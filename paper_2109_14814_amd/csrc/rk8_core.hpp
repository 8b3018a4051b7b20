// rk8_core.hpp -- pieces shared by the stroboscopic map (rk8.hip) and the
// refinement kernels (refine.hip): the Cooper-Verner order-8 tableau, the
// per-step stage tables of the time-dependent factor w(f) = 1 / (1 + e cos f),
// and the vector fields of the planar elliptic restricted three-body problem:
// pulsating rotating coordinates with the true anomaly as time, and the
// position-momentum form with time t of Sec. 3.3.
#pragma once

#include "ms_internal.hpp"

namespace ms {

constexpr int RK_S = 11;
constexpr double RK_TWO_PI = 6.283185307179586476925286766559;

struct Tableau {
    double a[RK_S][RK_S];
    double b[RK_S];
    double c[RK_S];
};

// Non-zero pattern of the Cooper-Verner tableau (zero terms are dropped at
// compile time; the values themselves come from cv_tableau and are checked
// against this pattern on the host).
constexpr bool RK_NZ[RK_S][RK_S] = {
    {0}, {1}, {1, 1}, {1, 1, 1}, {1, 0, 1, 1}, {1, 0, 1, 1, 1}, {1, 0, 1, 1, 1, 1},
    {1, 0, 0, 0, 1, 1, 1}, {1, 0, 0, 0, 1, 1, 1, 1}, {1, 0, 0, 0, 1, 1, 1, 1, 1}, {0, 0, 0, 0, 1, 1, 1, 1, 1, 1}};
constexpr bool RK_NZB[RK_S] = {1, 0, 0, 0, 0, 0, 0, 1, 1, 1, 1};

// Cooper & Verner (1972), SIAM J. Numer. Anal. 9, the order-8 method with 11
// stages.  Its coefficients lie in Q(sqrt 21); they are formed at compile
// time from RK_SQRT21, the double nearest to sqrt(21) (the host checks that
// sqrt(21.0) rounds to it), each operation rounded once as written.
constexpr double RK_SQRT21 = 4.5825756949558400065880471937280084889844565767679719026072421239;

constexpr Tableau cv_make_tableau()
{
    Tableau T{};
    const double q = RK_SQRT21;
    double (*a)[RK_S] = T.a;
    a[1][0] = 0.5;
    a[2][0] = 0.25; a[2][1] = 0.25;
    a[3][0] = 1.0 / 7.0; a[3][1] = -(7.0 + 3.0 * q) / 98.0; a[3][2] = (21.0 + 5.0 * q) / 49.0;
    a[4][0] = (11.0 + q) / 84.0; a[4][2] = (18.0 + 4.0 * q) / 63.0; a[4][3] = (21.0 - q) / 252.0;
    a[5][0] = (5.0 + q) / 48.0; a[5][2] = (9.0 + q) / 36.0; a[5][3] = (14.0 * q - 231.0) / 360.0; a[5][4] = (63.0 - 7.0 * q) / 80.0;
    a[6][0] = (10.0 - q) / 42.0; a[6][2] = (92.0 * q - 432.0) / 315.0; a[6][3] = (633.0 - 145.0 * q) / 90.0;
    a[6][4] = (115.0 * q - 504.0) / 70.0; a[6][5] = (63.0 - 13.0 * q) / 35.0;
    a[7][0] = 1.0 / 14.0; a[7][4] = (14.0 - 3.0 * q) / 126.0; a[7][5] = (13.0 - 3.0 * q) / 63.0; a[7][6] = 1.0 / 9.0;
    a[8][0] = 1.0 / 32.0; a[8][4] = (91.0 - 21.0 * q) / 576.0; a[8][5] = 11.0 / 72.0;
    a[8][6] = -(385.0 + 75.0 * q) / 1152.0; a[8][7] = (63.0 + 13.0 * q) / 128.0;
    a[9][0] = 1.0 / 14.0; a[9][4] = 1.0 / 9.0; a[9][5] = -(733.0 + 147.0 * q) / 2205.0;
    a[9][6] = (515.0 + 111.0 * q) / 504.0; a[9][7] = -(51.0 + 11.0 * q) / 56.0; a[9][8] = (132.0 + 28.0 * q) / 245.0;
    a[10][4] = (7.0 * q - 42.0) / 18.0; a[10][5] = (28.0 * q - 18.0) / 45.0; a[10][6] = -(273.0 + 53.0 * q) / 72.0;
    a[10][7] = (301.0 + 53.0 * q) / 72.0; a[10][8] = (28.0 - 28.0 * q) / 45.0; a[10][9] = (49.0 - 7.0 * q) / 18.0;
    const double b[RK_S] = {1.0 / 20.0, 0, 0, 0, 0, 0, 0, 49.0 / 180.0, 16.0 / 45.0, 49.0 / 180.0, 1.0 / 20.0};
    const double c[RK_S] = {0.0, 0.5, 0.5, (7.0 + q) / 14.0, (7.0 + q) / 14.0, 0.5, (7.0 - q) / 14.0,
                            (7.0 - q) / 14.0, 0.5, (7.0 + q) / 14.0, 1.0};
    for (int i = 0; i < RK_S; ++i) {
        T.b[i] = b[i];
        T.c[i] = c[i];
    }
    return T;
}

// The abscissae c_i as compile-time constants.
constexpr Tableau RK_T = cv_make_tableau();

// Host: the tableau; whether sqrt(21.0) rounds to RK_SQRT21 and the zeros
// match RK_NZ.
const Tableau &cv_tableau();
bool cv_pattern_ok();

// Stage values of the time-dependent coefficients, at the abscissa
// f = (n + c_i) h of stage i of step n of one period (h = 2 pi / steps):
//   w(f) = 1 / (1 + e cos f) (pulsating coordinates) and dw/de = -cos f w^2;
//   the separation of the primaries rho = 1 - e cos E(t) and the rate of
//   their true anomaly n(t) = sqrt(1 - e^2) / rho^2 at the time t = f, E the
//   eccentric anomaly (E - e sin E = t, periapse at t = 0).
// All are 2 pi periodic and even in the abscissa, so one period's values
// serve every period and both directions of integration.  The kernels
// compute them on the GPU: the maps a chunk of RK_CHUNK steps at a time
// into LDS, the refinement once per call into its workspace.  Nothing is
// allocated or copied from the host, so every call can be captured.
//
// The 11 abscissae are 4 and the next step's first: the maps keep RK_SLOTS
// values a step, and one more behind the last step.  A chunk's 253 are one
// for each thread of a block (with 11 for each of 32 steps, two rounds of
// Kepler's equation took 7% of the position-momentum map's time).
constexpr int RK_CHUNK = 63;
constexpr int RK_SLOTS = 4;
constexpr int RK_VALUES = RK_CHUNK * RK_SLOTS + 1;
constexpr double RK_SLOT_C[RK_SLOTS] = {RK_T.c[0], RK_T.c[1], RK_T.c[3], RK_T.c[6]};
constexpr int RK_SLOT[RK_S] = {0, 1, 1, 2, 2, 1, 3, 3, 1, 2, RK_SLOTS};   // of each stage; RK_SLOTS: the next step's 0
static_assert([] {
    for (int i = 0; i < RK_S; ++i)
        if (RK_T.c[i] != (RK_SLOT[i] == RK_SLOTS ? 1.0 : RK_SLOT_C[RK_SLOT[i] % RK_SLOTS])) return false;
    return RK_SLOT_C[0] == 0.0;
}(), "the stages' slots hold their abscissae");

MS_D double stage_abscissa(int64_t n, double c, int steps)
{
    const double h = RK_TWO_PI / (double)steps;
    return (double)n * h + c * h;
}

// Root of Kepler's equation E - e sin E = M for the primaries' orbit
// (Sec. 3.3, mean anomaly M = t).  E - M is 2 pi periodic in M and lies in
// [-e, e]; Newton's method from E = M + e sin M, kept inside that bracket (a
// step that leaves it is replaced by bisection), converges for every
// 0 <= e < 1.
MS_D double eccentric_anomaly(double M, double e)
{
    const double k = floor(M / RK_TWO_PI + 0.5);
    const double Mr = M - k * RK_TWO_PI;
    double lo = Mr - e, hi = Mr + e;
    double E = Mr + e * sin(Mr);
    if (!(E >= lo && E <= hi)) E = Mr;
    for (int it = 0; it < 100 && e > 0.0; ++it) {
        double sE, cE;
        sincos(E, &sE, &cE);
        const double g = E - e * sE - Mr;
        if (g == 0.0) break;
        if (g < 0.0) lo = E; else hi = E;
        double En = E - g / (1.0 - e * cE);
        if (!(En > lo && En < hi)) En = 0.5 * (lo + hi);
        const bool done = fabs(En - E) <= 2e-16 * (1.0 + fabs(E));
        E = En;
        if (done) break;
    }
    return E + k * RK_TWO_PI;
}

// (rho, n) at time t for eccentricity e.
MS_D double2 kepler_rho_n(double t, double e)
{
    const double rho = 1.0 - e * cos(eccentric_anomaly(t, e));
    return make_double2(rho, sqrt(1.0 - e * e) / (rho * rho));
}

// `threads` threads (this one is `first`) fill the stage values of steps
// n0 .. n0 + cnt - 1 (taken mod steps) into s_val[j * RK_SLOTS + slot], and the
// first of the step after them.
template <typename T, typename F>
MS_D void fill_stage_chunk(T *s_val, int first, int threads, int64_t n0, int cnt, int steps, F &&value)
{
    for (int i = first; i <= cnt * RK_SLOTS; i += threads) {
        const int j = i / RK_SLOTS, q = i % RK_SLOTS;
        const double c = q == 0 ? RK_SLOT_C[0] : q == 1 ? RK_SLOT_C[1] : q == 2 ? RK_SLOT_C[2] : RK_SLOT_C[3];
        s_val[i] = value(stage_abscissa((n0 + j) % steps, c, steps));
    }
}

struct Model {
    double mu, one_minus_mu;
};

// The tableau's 44 non-zero entries times the signed step h, row by row: the
// a_ij of stages 1..10, then the b_i.  With h in the coefficients a stage
// value is y plus one multiply-add per entry.
constexpr int RK_NC = 44;

struct RkCoef {
    double v[RK_NC];
};

RkCoef rk_coef(double h);

// m / r^3 from x = r^2 > 0: the hardware reciprocal square root y (about 23
// correct bits) gives y^3, corrected by the series of (1 - e)^(-3/2) in the
// residual e = 1 - x y^2 to second order; e is below 2^-21, so the first
// term left out is below 2^-61.  One cubic correction of the product takes
// 7 operations where two Newton steps of y followed by its cube took 10, and
// its rounding error is smaller (under 2 ulp, against up to 4).
MS_D double cube_series(double e)
{
    // 3/2 + 15/8 e.  Neither constant has an inline encoding; written as a
    // fused multiply-add the compiler moves 3/2 into the destination of
    // every use (a multiply-add in place, two 32-bit moves or one of 64 bits
    // before it: 22 a step).  The three-register form takes both as they are.
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(e), "s"(1.875), "v"(1.5));
    return r;
}

MS_D double mass_over_r3(double m, double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double y2 = y * y;
    const double e = fma(-x, y2, 1.0);
    const double c = m * (y2 * y);
    return fma(c * e, cube_series(e), c);
}

// The same, and q = 1 / r^2 = y^2 (1 + e + e^2).
MS_D double mass_over_r3(double m, double x, double &q)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double y2 = y * y;
    const double e = fma(-x, y2, 1.0);
    const double c = m * (y2 * y);
    q = fma(y2, fma(e, e, e), y2);
    return fma(c * e, cube_series(e), c);
}

// Right-hand sides, evaluated in place: on entry s holds a stage value, on
// return its derivative.  Every operation is written out (fused where it
// says fma), so that each kernel that evaluates them rounds alike.
//
// Pulsating frame at stage weight w: (x', y', w Omega_x + 2 y', w Omega_y -
// 2 x'), Omega = (x^2 + y^2)/2 + (1 - mu)/r1 + mu/r2, r1 = |(x + mu, y)|,
// r2 = |(x - 1 + mu, y)|.
MS_D void puls_field(const Model &md, double w, double (&s)[4])
{
    const double x = s[0], y = s[1], p = s[2], q = s[3];
    const double d1 = x + md.mu, d2 = x - md.one_minus_mu, y2 = y * y;
    const double g1 = mass_over_r3(md.one_minus_mu, fma(d1, d1, y2));
    const double g2 = mass_over_r3(md.mu, fma(d2, d2, y2));
    s[0] = p;
    s[1] = q;
    s[2] = fma(w, fma(-g1, d1, fma(-g2, d2, x)), q + q);
    s[3] = fma(w, fma(-(g1 + g2), y, y), -(p + p));
}

// The pulsating field with one tangent column in s[4..7]: v' = A v, plus
// dF/de (dwde = dw/de at the stage, 0 for a column of the state).
MS_D void puls_field_var(const Model &md, double w, double dwde, double (&s)[8])
{
    const double x = s[0], y = s[1], p = s[2], q = s[3];
    const double d1 = x + md.mu, d2 = x - md.one_minus_mu, y2 = y * y;
    double q1, q2;
    const double g1 = mass_over_r3(md.one_minus_mu, fma(d1, d1, y2), q1);
    const double g2 = mass_over_r3(md.mu, fma(d2, d2, y2), q2);
    const double h1 = 3.0 * g1 * q1, h2 = 3.0 * g2 * q2;                 // 3 m_i / r_i^5
    const double gs = g1 + g2, u = 1.0 - gs, t1 = h1 * d1, t2 = h2 * d2;
    const double ox = fma(-g1, d1, fma(-g2, d2, x)), oy = fma(-gs, y, y);
    const double oxx = fma(t1, d1, fma(t2, d2, u)), oyy = fma(h1 + h2, y2, u), oxy = (t1 + t2) * y;
    const double a = s[4], b = s[5], c = s[6], d = s[7];
    s[0] = p;
    s[1] = q;
    s[2] = fma(w, ox, q + q);
    s[3] = fma(w, oy, -(p + p));
    s[4] = c;
    s[5] = d;
    s[6] = fma(w, fma(oxx, a, oxy * b), fma(dwde, ox, d + d));
    s[7] = fma(w, fma(oxy, a, oyy * b), fma(dwde, oy, -(c + c)));
}

// Position-momentum model (Sec. 3.3) at a stage with separation rho and
// frame rate n: z' = J grad H for
//   H = (px^2 + py^2)/2 + n (px y - py x) - (1 - mu)/r1 - mu/r2,
//   r1 = |(x + mu rho, y)|, r2 = |(x - (1 - mu) rho, y)|,
// with NC tangent columns v' = J Hess(H) v behind the state (column c in
// s[4 + 4 c ..]).
template <int NC>
MS_D void pm_field(const Model &md, double rho, double n, double (&s)[4 + 4 * NC])
{
    const double x = s[0], y = s[1], p = s[2], q = s[3];
    const double d1 = fma(md.mu, rho, x), d2 = fma(-md.one_minus_mu, rho, x), y2 = y * y;
    const double r1 = fma(d1, d1, y2), r2 = fma(d2, d2, y2);
    double g1, g2, q1 = 0.0, q2 = 0.0;
    if constexpr (NC > 0) {
        g1 = mass_over_r3(md.one_minus_mu, r1, q1);
        g2 = mass_over_r3(md.mu, r2, q2);
    } else {
        g1 = mass_over_r3(md.one_minus_mu, r1);
        g2 = mass_over_r3(md.mu, r2);
    }
    const double gs = g1 + g2;
    s[0] = fma(n, y, p);
    s[1] = fma(-n, x, q);
    s[2] = fma(-g1, d1, fma(-g2, d2, n * q));
    s[3] = fma(-gs, y, -(n * p));
    if constexpr (NC > 0) {
        const double h1 = 3.0 * g1 * q1, h2 = 3.0 * g2 * q2;             // 3 m_i / r_i^5
        const double t1 = h1 * d1, t2 = h2 * d2;
        const double hxx = fma(-t1, d1, fma(-t2, d2, gs)), hyy = fma(-(h1 + h2), y2, gs), hxy = -((t1 + t2) * y);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            double *v = s + 4 + 4 * c;
            const double a = v[0], b = v[1], pa = v[2], pb = v[3];
            v[0] = fma(n, b, pa);
            v[1] = fma(-n, a, pb);
            v[2] = fma(-hxx, a, fma(-hxy, b, n * pb));
            v[3] = fma(-hxy, a, fma(-hyy, b, -(n * pa)));
        }
    }
}

// One step of y (D components) with the scaled coefficients c[0..43];
// field(i, s) evaluates the right-hand side of stage i in place.  The stage
// sums are taken in an order that keeps at most five D-vectors live (and y):
// stage 6 is opened before stages 2 and 3 are dropped, and stages 8 to 10
// and the increment are opened as soon as stage 6 is known, when the stages
// 0, 4, 5 and 6 are dropped.  The increment is summed on its own and added
// to y once, so that a step rounds at y's magnitude once; the stage values,
// whose rounding enters the step times h, are summed from y.
//
// Bound by FP64 issue: 180 multiply-adds of sums per state, 11 fields of 29
// operations and 22 reciprocal square roots (501 instructions a map step,
// 612 with the stage derivatives kept to the end, h applied per sum and two
// Newton steps per square root; 1,795 against 2,808 for the state with four
// tangent columns, where 440 live registers cost 770 moves a step to and
// from the accumulation registers).  F^3 of 526,593 states at 4000 steps a
// period: 96 ms, 133 before (114 by the step alone, then the rounds of blocks
// and the stage values' slots); DF of 262,144 states over a period: 60 ms, 84
// before.
template <int D, typename C, typename F>
MS_D void rk_step(double (&y)[D], const C &c, F &&field)
{
    // Nothing is moved across a stage's end (nor, within one, the sums ahead
    // of the field): the scheduler would trade registers for latency there.
    auto fence = [] { if constexpr (D > 8) __builtin_amdgcn_sched_barrier(0); };
    double k0[D], k1[D], k2[D], k3[D], k4[D], k5[D], k6[D], k7[D], k8[D], b[D];
#define MS_EACH for (int d = 0; d < D; ++d)
#pragma unroll
    MS_EACH k0[d] = y[d];
    field(0, k0);
    fence();
#pragma unroll
    MS_EACH k1[d] = fma(c[0], k0[d], y[d]);
    fence();
    field(1, k1);
    fence();
#pragma unroll
    MS_EACH k2[d] = fma(c[2], k1[d], fma(c[1], k0[d], y[d]));
#pragma unroll
    MS_EACH k1[d] = fma(c[4], k1[d], fma(c[3], k0[d], y[d]));      // stage 3, opened
    fence();
    field(2, k2);
    fence();
#pragma unroll
    MS_EACH k3[d] = fma(c[5], k2[d], k1[d]);
    fence();
    field(3, k3);
    fence();
#pragma unroll
    MS_EACH k4[d] = fma(c[8], k3[d], fma(c[7], k2[d], fma(c[6], k0[d], y[d])));
    fence();
    field(4, k4);
    fence();
#pragma unroll
    MS_EACH {
        k5[d] = fma(c[12], k4[d], fma(c[11], k3[d], fma(c[10], k2[d], fma(c[9], k0[d], y[d]))));
        k6[d] = fma(c[16], k4[d], fma(c[15], k3[d], fma(c[14], k2[d], fma(c[13], k0[d], y[d]))));
    }
    fence();
    field(5, k5);
    fence();
#pragma unroll
    MS_EACH k6[d] = fma(c[17], k5[d], k6[d]);
    fence();
    field(6, k6);
    fence();
#pragma unroll
    MS_EACH {
        const double z0 = k0[d], z4 = k4[d], z5 = k5[d], z6 = k6[d];
        k7[d] = fma(c[21], z6, fma(c[20], z5, fma(c[19], z4, fma(c[18], z0, y[d]))));
        k8[d] = fma(c[25], z6, fma(c[24], z5, fma(c[23], z4, fma(c[22], z0, y[d]))));
        k5[d] = fma(c[30], z6, fma(c[29], z5, fma(c[28], z4, fma(c[27], z0, y[d]))));     // stage 9
        k6[d] = fma(c[35], z6, fma(c[34], z5, fma(c[33], z4, y[d])));                     // stage 10
        b[d] = c[39] * z0;
    }
    fence();
    field(7, k7);
    fence();
#pragma unroll
    MS_EACH {
        k8[d] = fma(c[26], k7[d], k8[d]);
        k5[d] = fma(c[31], k7[d], k5[d]);
        k6[d] = fma(c[36], k7[d], k6[d]);
        b[d] = fma(c[40], k7[d], b[d]);
    }
    fence();
    field(8, k8);
    fence();
#pragma unroll
    MS_EACH {
        k5[d] = fma(c[32], k8[d], k5[d]);
        k6[d] = fma(c[37], k8[d], k6[d]);
        b[d] = fma(c[41], k8[d], b[d]);
    }
    fence();
    field(9, k5);
    fence();
#pragma unroll
    MS_EACH {
        k6[d] = fma(c[38], k5[d], k6[d]);
        b[d] = fma(c[42], k5[d], b[d]);
    }
    fence();
    field(10, k6);
    fence();
#pragma unroll
    MS_EACH y[d] += fma(c[43], k6[d], b[d]);
#undef MS_EACH
}

// The scaled coefficients of a kernel whose first parameter is an RkCoef, as
// a pointer that the compiler knows nothing about: taken once per step, so
// that the 88 scalar registers they fill are loaded again (from the scalar
// cache) where they are used.  Kept across the loop they would be spilled
// to vector lanes, two v_readlane each use.
using CoefPtr = const __attribute__((address_space(4))) double *;

MS_D CoefPtr step_coef()
{
    CoefPtr p = (CoefPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// How the maps with one thread per state share out a batch's blocks.
//
// A block is four waves, one a SIMD of a CU, and a wave alone on a SIMD
// issues at nine tenths of the rate of several: the time of one launch is
// that of the fullest CU, ceil(blocks / 256) rounds of a block's time, however
// little the last round holds (526,593 states are 2,058 blocks: 9 rounds for
// 8.04 of work; 71,680 states are 280: 2 for 1.09).  So the steps are cut
// into chunks and the (chunk, block) units, chunk by chunk, are dealt to
// launches of m x 256 blocks, m = blocks / 256 rounded down: a launch holds
// no block twice, and a block's chunks fall in successive launches.  Between
// launches a state waits in the output array.  The last launch alone is
// part empty: at most 1 / (chunks) of the time.
constexpr int FLOW_BLOCK = 256;
constexpr int64_t FLOW_CUS = 256;

struct FlowPlan {
    int64_t blocks;     // blocks of the whole batch
    int64_t chunk;      // steps of a unit
    int32_t launches;
    uint32_t grid;      // blocks of a launch
};

struct FlowUnit {
    int64_t block, s0, s1;      // steps [s0, s1) of the block's states
    bool ok;                    // false: past the last unit
};

MS_D FlowUnit flow_unit(const FlowPlan &p, int64_t u, int64_t nsteps)
{
    FlowUnit f;
    const int64_t c = u / p.blocks;
    f.block = u - c * p.blocks;
    f.s0 = c * p.chunk;
    f.ok = c == 0 || f.s0 < nsteps;     // (a call of no steps copies its states)
    f.s1 = f.s0 + p.chunk < nsteps ? f.s0 + p.chunk : nsteps;
    return f;
}

// resume: whether the states can be kept between launches.
inline FlowPlan flow_plan(int64_t blocks, int64_t nsteps, bool resume)
{
    FlowPlan p{blocks, nsteps > 0 ? nsteps : 1, 1, (uint32_t)blocks};
    const int64_t m = blocks / FLOW_CUS;
    const int64_t most = nsteps / (2 * RK_CHUNK);       // chunks of at least 126 steps
    if (!resume || m == 0 || blocks % FLOW_CUS == 0 || most < 4) return p;
    const int64_t n = most < 32 ? most : 32;
    const int64_t chunk = ceil_div(ceil_div(nsteps, n), RK_CHUNK) * RK_CHUNK;
    const int64_t launches = ceil_div(blocks * ceil_div(nsteps, chunk), m * FLOW_CUS);
    // the time in steps of a round: one wave a SIMD runs at 1.1 times a
    // round's time among several, and a launch costs about ten steps (10 us)
    const double one = (double)nsteps * (double)(m + 1);
    const double cut = (double)launches * ((double)chunk * (m == 1 ? 1.1 : (double)m) + 10.0);
    if (cut < one) {
        p.chunk = chunk;
        p.launches = (int32_t)launches;
        p.grid = (uint32_t)(m * FLOW_CUS);
    }
    return p;
}

}  // namespace ms
