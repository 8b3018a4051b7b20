// phase.hpp -- e^{i x} in the kernels that take one per frequency: by table and
// polynomial (Tang, "Table-driven implementation of the elementary functions"):
// n = rint(x / (pi / 32)), r = x - n pi / 32 with the constant in two parts, the
// first short enough that n times it is exact up to |n| = 2^20, and cos and sin
// of n pi / 32, kept in two parts as well, turned by r: the Taylor terms to r^8
// and r^7 are below 1e-17 for |r| <= pi / 64.  The correction is added to the
// table's value in the end, so the error is half a unit in the last place and
// little more.  About 25 FP64 instructions, a quarter of sincos, which remains
// for |x| above PH_MAX.
#pragma once

#include "ms_internal.hpp"

namespace ms {

constexpr double PH_COS[17][2] = {      // cos(k pi / 32): rounded, and the rest
    {0x1.0000000000000p+0, 0x0.0p+0},
    {0x1.fd88da3d12526p-1, -0x1.87df6378811c7p-55},
    {0x1.f6297cff75cb0p-1, 0x1.562172a361fd3p-56},
    {0x1.e9f4156c62ddap-1, 0x1.760b1e2e3f81ep-55},
    {0x1.d906bcf328d46p-1, 0x1.457e610231ac2p-56},
    {0x1.c38b2f180bdb1p-1, -0x1.6e0b1757c8d07p-56},
    {0x1.a9b66290ea1a3p-1, 0x1.9f630e8b6dac8p-60},
    {0x1.8bc806b151741p-1, -0x1.2c5e12ed1336dp-55},
    {0x1.6a09e667f3bcdp-1, -0x1.bdd3413b26456p-55},
    {0x1.44cf325091dd6p-1, 0x1.8076a2cfdc6b3p-57},
    {0x1.1c73b39ae68c8p-1, 0x1.b25dd267f6600p-55},
    {0x1.e2b5d3806f63bp-2, 0x1.e0d891d3c6841p-58},
    {0x1.87de2a6aea963p-2, -0x1.72cedd3d5a610p-57},
    {0x1.294062ed59f06p-2, -0x1.5d28da2c4612dp-56},
    {0x1.8f8b83c69a60bp-3, -0x1.26d19b9ff8d82p-57},
    {0x1.917a6bc29b42cp-4, -0x1.e2718d26ed688p-60},
    {0x0.0p+0, 0x0.0p+0}};
constexpr double PH_MAX = 1e5;
constexpr double PH_INV = 0x1.45f306dc9c883p+3;      // 32 / pi
constexpr double PH_P1 = 0x1.921fb54400000p-4, PH_P2 = 0x1.0b4611a626331p-38;

struct PhaseTable {
    double2 c[64], s[64];      // cos and sin of n pi / 32 in two parts
};

MS_D double2 ph_cos(int n)
{
    n &= 63;
    const int m = n > 32 ? 64 - n : n, k = m > 16 ? 32 - m : m;
    double2 v;
    v.x = PH_COS[k][0];
    v.y = PH_COS[k][1];
    if (m > 16) v = make_double2(-v.x, -v.y);
    return v;
}

MS_D void phase_table(PhaseTable &tab)
{
    for (int n = threadIdx.x; n < 64; n += blockDim.x) {
        tab.c[n] = ph_cos(n);
        tab.s[n] = ph_cos(n + 48);
    }
}

// |x| < PH_MAX.
MS_D void phase_near(const PhaseTable &tab, double x, double &cs, double &sn)
{
    const double n = rint(x * PH_INV);
    const double r = fma(-n, PH_P2, fma(-n, PH_P1, x)), z = r * r;
    const int k = (int)n & 63;
    const double2 c = tab.c[k], s = tab.s[k];
    const double sr = fma(r * z, fma(z, fma(z, -1.0 / 5040.0, 1.0 / 120.0), -1.0 / 6.0), r);
    const double cr = z * fma(z, fma(z, fma(z, 1.0 / 40320.0, -1.0 / 720.0), 1.0 / 24.0), -0.5);
    cs = c.x + fma(-s.x, sr, fma(c.x, cr, c.y));
    sn = s.x + fma(c.x, sr, fma(s.x, cr, s.y));
}

MS_D void phase(const PhaseTable &tab, double x, double &cs, double &sn)
{
    if (__builtin_expect(fabs(x) < PH_MAX, 1)) phase_near(tab, x, cs, sn);
    else sincos(x, &sn, &cs);
}

}  // namespace ms
