// rk8_pair.hpp -- the Runge-Kutta steps with two lanes per trajectory, for
// batches too small to fill the chip.
//
// A few hundred to some ten thousand trajectories give each SIMD at most one
// wave, and the time is then that of one wave working through its steps: its
// instructions at one FP64 operation per 4 cycles, and the waits of its
// dependent chain.  Two lanes share a trajectory: lane 0 of a pair holds x
// and its momentum (or velocity), lane 1 y and its own, so each carries half
// of the stage sums; lane 0 takes the force of the first primary and lane 1
// that of the second, and the halves are exchanged by quad-permuted moves
// (DPP, no LDS).  A map step is 345 instructions a lane against 501, and a
// step with one tangent column 688 against 957.  The scaled coefficients
// stay in vector registers: scalar loads would be waited for at every step.
#pragma once

#include "rk8_core.hpp"

namespace ms {

// The value of the other lane of the pair.
MS_D double pair_swap(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0xB1, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0xB1, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// What differs between the lanes of a pair: its primary's mass, where the
// primary sits along the lane's own axis (own) and along the other (oth), and
// the sign of the Coriolis terms.
struct PairLane {
    double m, own, oth, sg;
};

MS_D PairLane pair_lane(const Model &md, int lane)
{
    PairLane L;
    L.m = lane ? md.mu : md.one_minus_mu;
    L.own = lane ? 0.0 : md.mu;
    L.oth = lane ? -md.one_minus_mu : 0.0;
    L.sg = lane ? -1.0 : 1.0;
    return L;
}

// The scaled coefficients in vector registers.
struct PairCoef {
    double v[RK_NC];
    MS_D double operator[](int i) const { return v[i]; }
};

MS_D void pair_coef(PairCoef &c, const RkCoef &hc)
{
#pragma unroll
    for (int i = 0; i < RK_NC; ++i) {
        c.v[i] = hc.v[i];
        asm volatile("" : "+v"(c.v[i]));
    }
}

// Force per unit mass of both primaries along the lane's own axis, from the
// offsets a (own axis) and b (other axis) to the lane's primary.
MS_D double pair_force(const PairLane &L, double a, double b)
{
    const double g = mass_over_r3(L.m, fma(a, a, b * b));
    return fma(g, a, pair_swap(g * b));
}

// The same with the second derivatives of the potential along the own axis
// (hoo) and across (hot): sums over the primaries of g - h a^2 and -h a b,
// h = 3 m / r^5.
MS_D double pair_force(const PairLane &L, double a, double b, double &hoo, double &hot)
{
    double q;
    const double g = mass_over_r3(L.m, fma(a, a, b * b), q);
    const double h = 3.0 * g * q, ha = h * a, hb = h * b;
    const double ab = ha * b;
    hoo = fma(-ha, a, g) + pair_swap(fma(-hb, b, g));
    hot = -(ab + pair_swap(ab));
    return fma(g, a, pair_swap(g * b));
}

// Pulsating frame, in place: s = (own coordinate, own velocity), then
// (COL) the same of a tangent column; wd = (w, dw/de).
template <bool COL>
MS_D void puls_pair(const PairLane &L, double w, double dwde, double (&s)[COL ? 4 : 2])
{
    const double x = s[0], v = s[1], xo = pair_swap(x), vo = pair_swap(v), cor = 2.0 * L.sg;
    const double a = x + L.own, b = xo + L.oth;
    if constexpr (COL) {
        double hoo, hot;
        const double o = x - pair_force(L, a, b, hoo, hot);
        const double u = s[2], pu = s[3], uo = pair_swap(u), puo = pair_swap(pu);
        s[2] = pu;
        s[3] = fma(w, fma(1.0 - hoo, u, -hot * uo), fma(dwde, o, cor * puo));
        s[1] = fma(w, o, cor * vo);
    } else {
        s[1] = fma(w, x - pair_force(L, a, b), cor * vo);
    }
    s[0] = v;
}

// Position-momentum frame, in place, at separation rho and frame rate n.
template <bool COL>
MS_D void pm_pair(const PairLane &L, double rho, double n, double (&s)[COL ? 4 : 2])
{
    const double x = s[0], p = s[1], xo = pair_swap(x), po = pair_swap(p), sn = L.sg * n;
    const double a = fma(L.own, rho, x), b = fma(L.oth, rho, xo);
    if constexpr (COL) {
        double hoo, hot;
        const double f = pair_force(L, a, b, hoo, hot);
        const double u = s[2], pu = s[3], uo = pair_swap(u), puo = pair_swap(pu);
        s[2] = fma(sn, uo, pu);
        s[3] = fma(-hoo, u, fma(-hot, uo, sn * puo));
        s[1] = fma(sn, po, -f);
    } else {
        s[1] = fma(sn, po, -pair_force(L, a, b));
    }
    s[0] = fma(sn, xo, p);
}

// The maps on pairs of lanes.  Three compute waves and a fourth per block (one
// a SIMD of a CU), which works out the next chunk's stage values (V: w, or rho and n from
// Kepler's equation) while the others integrate the present one: solved by
// the compute waves themselves they would take a fifth of the time.
constexpr int PAIR_LANES = 3 * WAVE, PAIR_BLOCK = 4 * WAVE;

// COLS = 0: one pair per state.  COLS = 4: one pair per state and tangent
// column (the state goes with each column).
template <typename V, int COLS, typename STAGE, typename FIELD>
MS_D void pair_flow(const RkCoef &hc, const double *in, double *out, double *stm, int64_t n, const Model &md, int steps,
                    int64_t nsteps, STAGE &&stage_value, FIELD &&field)
{
    constexpr int D = COLS ? 4 : 2, PP = COLS ? COLS : 1;
    __shared__ V s_val[2][RK_VALUES];
    const bool producer = threadIdx.x >= PAIR_LANES;
    const int lane = threadIdx.x & 1;
    const int64_t pair = ((int64_t)blockIdx.x * (PAIR_LANES) + threadIdx.x) >> 1;
    const int64_t st = pair / PP;
    const int col = (int)(pair - st * PP);
    const bool live = !producer && st < n;
    auto chunk_len = [&](int64_t s0) { return nsteps - s0 < RK_CHUNK ? (int)(nsteps - s0) : RK_CHUNK; };
    double y[D];
#pragma unroll
    for (int d = 0; d < D; ++d) y[d] = 0.0;
    if (live) {
        y[0] = in[4 * st + lane];
        y[1] = in[4 * st + 2 + lane];
        if constexpr (COLS > 0) {
            y[2] = col == lane ? 1.0 : 0.0;
            y[3] = col == 2 + lane ? 1.0 : 0.0;
        }
    }
    fill_stage_chunk(s_val[0], threadIdx.x, PAIR_BLOCK, 0, chunk_len(0), steps, stage_value);
    __syncthreads();
    int64_t n_in = 0;
    int cur = 0;
    PairCoef c;
    PairLane L;
    if (!producer) {
        pair_coef(c, hc);
        L = pair_lane(md, lane);
    }
    for (int64_t s0 = 0; s0 < nsteps; s0 += RK_CHUNK, cur ^= 1) {
        const int cnt = chunk_len(s0);
        n_in = (n_in + cnt) % steps;
        if (producer) {
            if (s0 + cnt < nsteps) {
                fill_stage_chunk(s_val[cur ^ 1], threadIdx.x - PAIR_LANES, WAVE, n_in, chunk_len(s0 + cnt), steps,
                                 stage_value);
            }
        } else if (live) {
#pragma unroll 1
            for (int jj = 0; jj < cnt; ++jj) {
                const V *row = s_val[cur] + jj * RK_SLOTS;
                rk_step<D>(y, c, [&](int i, double (&s)[D]) { field(L, row[RK_SLOT[i]], s); });
            }
        }
        __syncthreads();
    }
    if (!live) return;
    if (out && col == 0) {
        out[4 * st + lane] = y[0];
        out[4 * st + 2 + lane] = y[1];
    }
    if constexpr (COLS > 0) {
        // Row-major 4 x 4 per state: stm[16 p + 4 i + j] = d out_i / d in_j.
        stm[16 * st + 4 * lane + col] = y[2];
        stm[16 * st + 4 * (2 + lane) + col] = y[3];
    }
}

// Up to these sizes every compute wave has a SIMD of its own (256 CUs of
// three, 32 pairs a wave).  A period of 4000 steps then takes 3.0 ms against
// 4.5 ms with one lane per state (whose waves have a SIMD each up to 65,536
// states), and with the matrix 5.4 ms against 7.7; with a second wave on a
// SIMD, 5.3 and 10.0 ms.
constexpr int64_t PAIR_STATES = 256 * 3 * 32;
constexpr int64_t PAIR_MATRICES = PAIR_STATES / 4;

inline unsigned pair_blocks(int64_t pairs) { return (unsigned)ceil_div(2 * pairs, PAIR_LANES); }

}  // namespace ms
