// fourier_taylor.hip -- points and partials of Fourier-Taylor
// parameterizations W(theta, s) = sum_k W_k(theta) s^k of a manifold, and of
// their globalization W(theta, s) = F^m(W(theta - m omega, lambda^-m s))
// (Sec. 7).
//
// The coefficients W_k are given by their spectra over theta (theta_spectrum
// of each coefficient row, scaled by 1/N, the pairs (x, y) and (px, py)
// packed as complex sequences).  Per query (theta, s) and frequency j the
// series in s is summed (the value V(j) and its s-derivative together), by
// Horner's rule for few queries and as a matrix product for many, and the
// terms e^{i j theta} V(j) and i j e^{i j theta} V(j) are added up over the
// lanes, the waves of a block and their steps: W, dW/dtheta and dW/ds.  This
// is the paper's "evaluate in s, FFT
// derivative in theta, interpolate trigonometrically", done in the
// frequency domain so that no per-query transform is needed: the
// trigonometric interpolant of the samples is the sum over their spectrum.
//
// Globalization: the local evaluation at (theta - m omega, lambda^-m s) (the
// s-derivative already scaled by lambda^-m), then F^m and DF^m of the point
// by the position-momentum map, then the two partials multiplied by DF^m.
//
// Refinement (ft_newton): the damped Newton iteration of Sec. 7 on
// f = W_u(theta_u, s_u) - W_s(theta_s, s_s) with Df from the four partials,
// one ft_partials per chart and one decision kernel per iteration.
#include <math.h>

#include <algorithm>
#include <string>

#include "newton.hpp"
#include "phase.hpp"

namespace ms {
namespace {

constexpr int FT_STEP = 32;          // frequencies of a wave's step
constexpr int FT_R = 8, FT_R_LOW = 3;   // coefficients of a lane in flight; orders below 3
template <int QT>
constexpr int FT_MAX_WAVES = QT > 2 ? 8 : 16;

struct FtArgs {
    const double *spec, *theta, *s;
    double *w, *dth, *ds;
    int64_t nq;
    double th_off, s_scale;
    int N, P;
};

MS_D double uni(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// v[0 .. 2 N) summed over the lanes' bits OFF ... LAST, halving: value j ends
// up in the lanes whose top bits of these are j.
template <int N, int OFF, int LAST>
MS_D double lane_sums(const double *v)
{
    const bool hi = (threadIdx.x & OFF) != 0;
    double h[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const double mine = hi ? v[j + N] : v[j], send = hi ? v[j] : v[j + N];
        h[j] = mine + __shfl_xor(send, OFF);
    }
    if constexpr (N > 1) {
        return lane_sums<N / 2, OFF / 2, LAST>(h);
    } else {
#pragma unroll
        for (int o = OFF / 2; o >= LAST; o /= 2) h[0] += __shfl_xor(h[0], o);
        return h[0];
    }
}

// QT queries per block by Horner's rule.  A lane takes one of the two complex
// pairs of every 32nd frequency and all QT queries, so that a coefficient is
// loaded once for QT of them; the next R coefficients are in flight.  The
// block's waves take steps of 32 frequencies in turn.  A table of 2048
// frequencies to order 25 is 1.7 MB, so what bounds it is the L2's
// 14 TB/s for many queries and the loads' latency for few: 4 queries per block
// take 31 us for 256 queries and 33 for 1000, one 20 for 64, 24 for 256 and 38
// for 300; a wave per query took 105 for up to 1024.  8 queries spill.  The
// orders below 3 load no more coefficients than they have (2048 frequencies,
// 3000 queries to order 0: 30.0 us, 34.3 with 8).
template <int QT>
struct FtShared {
    double sum[FT_MAX_WAVES<QT>][3][4 * QT];
    PhaseTable ph;
};

template <int QT, int R>
MS_D void ft_eval(FtShared<QT> &s_sum, int64_t q0, const FtArgs &g)
{
    phase_table(s_sum.ph);
    __syncthreads();
    const double *spec = g.spec, *theta = g.theta, *s = g.s;
    const int N = g.N, P = g.P;
    const int64_t nq = g.nq;
    const double th_off = g.th_off, s_scale = g.s_scale;
    const int lane = threadIdx.x % 64, wv = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), n_waves = blockDim.x / 64, p = lane & 1;
    double t[QT], sl[QT];
#pragma unroll
    for (int q = 0; q < QT; ++q) {
        const int64_t k = q0 + q < nq ? q0 + q : nq - 1;
        t[q] = uni(theta[k] - th_off);
        sl[q] = uni(s[k] * s_scale);
    }
    const int steps = (N + FT_STEP - 1) / FT_STEP;
    const int lowest = -((N - 1) / 2);
    double aw[2 * QT] = {}, ath[2 * QT] = {}, as[2 * QT] = {};
    double2 x[R];                   // coefficients in flight
    const double *top = spec + 4 * (int64_t)N * P;
    const int64_t row = 4 * (int64_t)N;
    const double *ahead = top;      // row of the next coefficients to load, k_ahead rows below the top
    int k_ahead = 0;
    auto offset = [&](int m) {
        const int idx = FT_STEP * m + (lane >> 1), js = lowest + idx;
        return (uint32_t)(4 * (idx >= N ? 0 : js < 0 ? js + N : js) + 2 * p);
    };
    auto get = [&](uint32_t at) {
        const double2 c = *reinterpret_cast<const double2 *>(ahead + at);
        if (k_ahead < P) ahead -= row;      // (past the last row: once more, unused)
        ++k_ahead;
        return c;
    };
    auto fetch = [&](int m) {
        const uint32_t at = offset(m);
        ahead = top;
        k_ahead = 0;
#pragma unroll
        for (int u = 0; u < R; ++u) x[u] = get(at);
    };
    auto step = [&](int m, auto last) {
        const uint32_t at = offset(m);
        const int idx = FT_STEP * m + (lane >> 1), js = lowest + idx;
        // the series in s at this frequency, value and derivative together
        double vr[QT] = {}, vi[QT] = {}, dr[QT] = {}, di[QT] = {};
        auto horner = [&](int u) {
#pragma unroll
            for (int q = 0; q < QT; ++q) {
                dr[q] = fma(dr[q], sl[q], vr[q]);
                di[q] = fma(di[q], sl[q], vi[q]);
                vr[q] = fma(vr[q], sl[q], x[u].x);
                vi[q] = fma(vi[q], sl[q], x[u].y);
            }
        };
        int k = 0;
        for (; k + R <= P + 1; k += R)
#pragma unroll
            for (int u = 0; u < R; ++u) {
                horner(u);
                x[u] = get(at);
            }
#pragma unroll
        for (int u = 0; u < R - 1; ++u)
            if (k + u <= P) horner(u);
        if (m + n_waves < steps) fetch(m + n_waves);
        if (last && idx >= N)
#pragma unroll
            for (int q = 0; q < QT; ++q) vr[q] = vi[q] = dr[q] = di[q] = 0.0;
        // The mode N / 2 is the cosine: a real factor on both parts.  It adds
        // nothing to the theta derivative: the derivative is taken at the
        // samples (coefficient j times i j, whose real part is 0 at
        // j = N/2) and then interpolated.
        const bool nyq = last && 2 * js == N;
        const double jd = (double)js;
        // the phases: the lanes of the two pairs take half of them each
        double cs[QT], sn[QT];
        if constexpr (QT == 1) {
            phase(s_sum.ph, (double)js * t[0], cs[0], sn[0]);
        } else {
#pragma unroll
            for (int q = 0; q < QT; q += 2) {
                double c, e;
                phase(s_sum.ph, (double)js * (p ? t[q + 1] : t[q]), c, e);
                const double oc = __shfl_xor(c, 1), oe = __shfl_xor(e, 1);
                cs[q] = p ? oc : c;
                sn[q] = p ? oe : e;
                cs[q + 1] = p ? c : oc;
                sn[q + 1] = p ? e : oe;
            }
        }
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            const double f = cs[q], e = nyq ? 0.0 : sn[q];
            // (each part by itself at the cosine mode: 0 times an infinite one is no number)
            const double xr = nyq ? 0.0 : vr[q], xi = nyq ? 0.0 : vi[q];
            const double re = fma(vr[q], f, -(xi * e)), im = fma(xr, e, vi[q] * f);
            aw[2 * q] += re;
            aw[2 * q + 1] += im;
            ath[2 * q] = fma(-jd, nyq ? 0.0 : im, ath[2 * q]);       // i js (re + i im)
            ath[2 * q + 1] = fma(jd, nyq ? 0.0 : re, ath[2 * q + 1]);
            as[2 * q] = fma(dr[q], f, fma(nyq ? 0.0 : -di[q], e, as[2 * q]));
            as[2 * q + 1] = fma(nyq ? 0.0 : dr[q], e, fma(di[q], f, as[2 * q + 1]));
        }
    };
    if (wv < steps) fetch(wv);
    for (int m = wv; m < steps; m += n_waves) {
        if (m < steps - 1) step(m, std::false_type{});
        else step(m, std::true_type{});
    }
    const double sums[3] = {lane_sums<QT, 32, 2>(aw), lane_sums<QT, 32, 2>(ath), lane_sums<QT, 32, 2>(as)};
    constexpr int SHARE = 64 / (2 * QT);
    if (lane % SHARE < 2) {
        const int j = lane / SHARE;      // 2 query + part
#pragma unroll
        for (int i = 0; i < 3; ++i) s_sum.sum[wv][i][4 * (j >> 1) + 2 * p + (j & 1)] = sums[i];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 12 * QT; i += blockDim.x) {
        const int kind = i / (4 * QT), e = i % (4 * QT);
        const int64_t q = q0 + e / 4;
        if (q >= nq) continue;
        double v = s_sum.sum[0][kind][e];
        for (int k = 1; k < n_waves; ++k) v += s_sum.sum[k][kind][e];
        if (kind == 2) v *= s_scale;     // d/ds of W(theta, lambda^-m s)
        if (!isfinite(theta[q] - th_off) || !isfinite(s[q] * s_scale)) v = NAN;
        (kind == 0 ? g.w : kind == 1 ? g.dth : g.ds)[4 * q + e % 4] = v;
    }
}

template <int QT, int R>
__global__ void __launch_bounds__(64 * FT_MAX_WAVES<QT>) k_ft_eval(FtArgs g)
{
    __shared__ FtShared<QT> s_sum;
    ft_eval<QT, R>(s_sum, (int64_t)blockIdx.x * QT, g);
}

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int FT_TILE = 16;
constexpr int FT_TILE_WAVES = 8;

// 16 queries per block on the matrix cores: V(j) and its derivative are the
// products of the queries' powers s^k and k s^(k-1) (16 rows, kept in
// registers, to order 4 KA - 1) with the coefficients at 16 frequencies.  A
// wave takes one complex pair and every fourth step of 16 frequencies; a lane
// then holds four queries at one frequency and adds their terms.  The powers
// are rounded once and summed from the highest down, so that the result is as
// close as Horner's (the error against longer arithmetic is the same, and
// half of it is the sum over j).
//
// FP64 matrix instructions run at the rate of the vector ones here, but their
// operands are the coefficients themselves, loaded once for 16 queries, and
// the phases run beside them.  4096 queries of 2048 frequencies to order 25:
// 84 to 94 us from 225 with a wave per query, 133 with four queries a block (the
// L2's rate) and 53 at the card's matrix rate.
template <int KA>
__global__ void __launch_bounds__(64 * FT_TILE_WAVES) k_ft_tile(FtArgs g)
{
    __shared__ double s_sum[FT_TILE_WAVES / 2][3][4 * FT_TILE];
    __shared__ FtShared<1> s_one;
    __shared__ uint32_t s_bad;
    const int N = g.N, P = g.P, lane = threadIdx.x % 64, quad = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), p = wv & 1, part = wv >> 1;
    constexpr int PARTS = FT_TILE_WAVES / 2;
    const int64_t q0 = (int64_t)blockIdx.x * FT_TILE;
    auto query = [&](int q) { return q0 + q < g.nq ? q0 + q : g.nq - 1; };
    if (threadIdx.x == 0) s_bad = 0;
    phase_table(s_one.ph);
    __syncthreads();
    // powers s^k (rows: queries) and k s^(k - 1), k = 4 a + 3 - quad; rounded once
    double pv[KA], pd[KA];
    {
        const double sl = g.s[query(lane & 15)] * g.s_scale;
        double hi = 1.0, lo = 0.0, prev = 0.0;
#pragma unroll
        for (int k = 0; k < 4 * KA; ++k) {
            if (3 - (k & 3) == quad) {
                pv[k >> 2] = k <= P ? hi : 0.0;
                pd[k >> 2] = k <= P ? (double)k * prev : 0.0;
            }
            prev = hi;
            const double x = hi * sl, e = fma(lo, sl, fma(hi, sl, -x));
            hi = x + e;
            lo = e - (hi - x);
        }
    }
    const int steps = (N + 15) / 16, lowest = -((N - 1) / 2);
    double t[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) t[r] = g.theta[query(quad + 4 * r)] - g.th_off;
    double aw[8] = {}, ath[8] = {}, as[8] = {};
    double2 x[KA];
    auto fetch = [&](int m) {
        const int idx = 16 * m + (lane & 15), js = lowest + idx;
        const uint32_t at = (uint32_t)(4 * (idx >= N ? 0 : js < 0 ? js + N : js) + 2 * p);
#pragma unroll
        for (int a = 0; a < KA; ++a) {
            const int k = 4 * a + 3 - quad;
            x[a] = *reinterpret_cast<const double2 *>(g.spec + 4 * (int64_t)N * (k <= P ? k : P) + at);
        }
    };
    if (part < steps) fetch(part);
    for (int m = part; m < steps; m += PARTS) {
        v4d vr = {}, vi = {}, dr = {}, di = {};
#pragma unroll
        for (int a = KA - 1; a >= 0; --a) {
            vr = __builtin_amdgcn_mfma_f64_16x16x4f64(pv[a], x[a].x, vr, 0, 0, 0);
            vi = __builtin_amdgcn_mfma_f64_16x16x4f64(pv[a], x[a].y, vi, 0, 0, 0);
            dr = __builtin_amdgcn_mfma_f64_16x16x4f64(pd[a], x[a].x, dr, 0, 0, 0);
            di = __builtin_amdgcn_mfma_f64_16x16x4f64(pd[a], x[a].y, di, 0, 0, 0);
        }
        if (m + PARTS < steps) fetch(m + PARTS);
        const int idx = 16 * m + (lane & 15), js = lowest + idx;
        if (idx >= N) vr = vi = dr = di = v4d{};
        const bool nyq = 2 * js == N;
        const double jd = nyq ? 0.0 : (double)js;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double f, e;
            phase(s_one.ph, (double)js * t[r], f, e);
            if (nyq) e = 0.0;
            const double re = fma(vr[r], f, -(vi[r] * e)), im = fma(vr[r], e, vi[r] * f);
            aw[2 * r] += re;
            aw[2 * r + 1] += im;
            ath[2 * r] = fma(-jd, im, ath[2 * r]);
            ath[2 * r + 1] = fma(jd, re, ath[2 * r + 1]);
            as[2 * r] = fma(dr[r], f, fma(-di[r], e, as[2 * r]));
            as[2 * r + 1] = fma(dr[r], e, fma(di[r], f, as[2 * r + 1]));
        }
    }
    const double sums[3] = {lane_sums<4, 8, 1>(aw), lane_sums<4, 8, 1>(ath), lane_sums<4, 8, 1>(as)};
    if ((lane & 1) == 0) {
        const int j = (lane & 15) >> 1, q = quad + 4 * (j >> 1);
#pragma unroll
        for (int i = 0; i < 3; ++i) s_sum[part][i][4 * q + 2 * p + (j & 1)] = sums[i];
    }
    __syncthreads();
    if (threadIdx.x < 12 * FT_TILE) {
        const int kind = threadIdx.x / (4 * FT_TILE), e = threadIdx.x % (4 * FT_TILE);
        const int64_t q = q0 + e / 4;
        if (q < g.nq) {
            double v = 0.0;
#pragma unroll
            for (int k = 0; k < PARTS; ++k) v += s_sum[k][kind][e];
            if (kind == 2) v *= g.s_scale;     // d/ds of W(theta, lambda^-m s)
            const bool fin = isfinite(g.theta[q] - g.th_off) && isfinite(g.s[q] * g.s_scale);
            if (fin && !isfinite(v)) atomicOr(&s_bad, 1u << (e / 4));
            (kind == 0 ? g.w : kind == 1 ? g.dth : g.ds)[4 * q + e % 4] = fin ? v : NAN;
        }
    }
    __syncthreads();
    // Horner's rule gives a number in cases where 0 times a power or a
    // coefficient that is none does not
    for (uint32_t bad = s_bad; bad; bad &= bad - 1) {
        ft_eval<1, FT_R>(s_one, q0 + __builtin_ctz(bad), g);
        __syncthreads();
    }
}

// The waves of a block: two per SIMD over the card (which the registers of
// four queries allow), as 8 or 4, since a block of 5 to 7 keeps a CU to itself
// and 1100 to 2000 queries then take two rounds (2048 frequencies, 1800 queries
// to order 8: 34.0 us, 51.6 with 5 waves).  Where blocks
// queue, fewer waves with at least four steps each spend less on the sums over
// lanes and waves (128 frequencies, 8192 queries to order 0 and 25: 9.3 and
// 19.2 us, 17.6 and 25.7 with four waves; but 5000 queries of 256 to order 25
// 26.5 for 25.1: beyond order 8 from 8192 queries on).
template <int QT>
int eval_waves(int64_t blocks, int64_t steps, int order)
{
    if (blocks <= 256)
        return (int)std::min<int64_t>(std::min<int64_t>(ceil_div((int64_t)2048, blocks), FT_MAX_WAVES<QT>), steps);
    const int64_t most = blocks > (order <= 8 ? 1024 : 2047) ? steps / 4 : steps;
    return most >= 4 ? 4 : most >= 2 ? 2 : 1;
}

template <int QT>
void launch_ft_eval(const FtArgs &g, hipStream_t st)
{
    const int64_t blocks = ceil_div(g.nq, (int64_t)QT), steps = ceil_div((int64_t)g.N, (int64_t)FT_STEP);
    const int waves = eval_waves<QT>(blocks, steps, g.P);
    const auto kernel = g.P < FT_R_LOW ? k_ft_eval<QT, FT_R_LOW> : k_ft_eval<QT, FT_R>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3((unsigned)(64 * waves)), 0, st, g);
}

template <int KA>
void launch_ft_tile(const FtArgs &g, hipStream_t st)
{
    hipLaunchKernelGGL(k_ft_tile<KA>, dim3((unsigned)ceil_div(g.nq, (int64_t)FT_TILE)), dim3(64 * FT_TILE_WAVES), 0, st,
                       g);
}

// Whether the matrix cores take a call.  Their blocks of 16 queries, one to a
// CU, take as long for 1 query as for 4096, and whole steps of orders; blocks
// of four queries go by 1024, two to a CU at once.  In us, x being N / 2048: a
// round of 4096 queries takes 2.7 + 34 x, 2.9 + 41.5 x, 3.9 + 55 x or 4.7 +
// 77.6 x up to order 3, 7, 15 or 27, and 1024 queries by fours 1.03 a full
// block's waves and (9.34 + 0.72 order) x, 7.46 for 9.34 below order 3, and
// 2.4 once.  (Fitted to 33 to 5000 frequencies, 1000 to 40000 queries, every
// kind of order; the choice is 0.2% from the faster of the two on the average.
// 2048 frequencies, 4096 queries to order 0, 3, 8 and 25: 38.6, 38.6, 61.0 and 84
// here, 37.5, 52.8, 63.3 and 116 by fours; 6144: 74.6, 74.7, 119 and 165 here, 54,
// 76, 92 and 171 by fours; 2048: 20.9, 29.1, 34.4 and 61 by fours.)  Spectra
// beyond an XCD's L2 (4 MB) cost the fours, which read them four times as
// often, some 15% more.
inline bool tiles_pay(int64_t nq, int N, int order)
{
    if (order > 27) return false;
    const double x = N / 2048.0, fours = (double)ceil_div(nq, (int64_t)1024), tiles = (double)ceil_div(nq, (int64_t)4096);
    const int waves = std::min(4, eval_waves<4>(ceil_div(nq, (int64_t)4), ceil_div((int64_t)N, (int64_t)FT_STEP), order));
    const double start = order <= 3 ? 2.7 : order <= 7 ? 2.9 : order <= 15 ? 3.9 : 4.7;
    const double slope = order <= 3 ? 34.0 : order <= 7 ? 41.5 : order <= 15 ? 55.0 : 77.6;
    const double by_fours = 2.4 + fours * (1.03 * waves / 4 + x * ((order < 3 ? 7.46 : 9.34) + 0.72 * order));
    const bool beyond = (int64_t)N * (order + 1) * 32 > 4 << 20;
    return tiles * (start + x * slope) < (beyond ? 1.15 : 1.0) * by_fours;
}

// dth <- M dth, ds <- M ds per query (M row-major 4 x 4).
__global__ void __launch_bounds__(256) k_apply_stm(const double *__restrict__ stm, double *dth, double *ds, int64_t nq)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nq) return;
    const double *M = stm + 16 * q;
    double a[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        a[i] = dth[4 * q + i];
        b[i] = ds[4 * q + i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        dth[4 * q + i] = M[4 * i] * a[0] + M[4 * i + 1] * a[1] + M[4 * i + 2] * a[2] + M[4 * i + 3] * a[3];
        ds[4 * q + i] = M[4 * i] * b[0] + M[4 * i + 1] * b[1] + M[4 * i + 2] * b[2] + M[4 * i + 3] * b[3];
    }
}

// Parameters and partials of one side of the Newton problems.
struct FtSide {
    double *th, *s, *w, *dth, *ds, *stm;
};

MS_D void ftn_split(int64_t k, const NewtonState &ns, const FtSide &u, const FtSide &v)
{
    u.th[k] = ns.q[4 * k + 0];
    u.s[k] = ns.q[4 * k + 1];
    v.th[k] = ns.q[4 * k + 2];
    v.s[k] = ns.q[4 * k + 3];
}

__global__ void __launch_bounds__(256) k_ftn_init(const double *x0, NewtonState ns, int64_t K, FtSide u, FtSide v,
                                                  unsigned long long *running)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k == 0) running[0] = running[1] = 0;
    if (k >= K) return;
    newton_init(k, x0, ns);
    ftn_split(k, ns, u, v);
}

// One decision per running problem; counts the problems still running in
// running[par] and clears the other counter for the next iteration.
__global__ void __launch_bounds__(256) k_ftn_update(NewtonState ns, NewtonCfg cfg, int64_t K, FtSide u, FtSide v,
                                                    unsigned long long *running, int par)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k == 0) running[par ^ 1] = 0;
    if (k >= K || ns.status[k] >= 0) return;
    double f[4], M[4][4];
    for (int c = 0; c < 4; ++c) {
        f[c] = u.w[4 * k + c] - v.w[4 * k + c];
        M[c][0] = u.dth[4 * k + c];
        M[c][1] = u.ds[4 * k + c];
        M[c][2] = -v.dth[4 * k + c];
        M[c][3] = -v.ds[4 * k + c];
    }
    newton_decide(k, f, M, ns, cfg);
    if (ns.status[k] < 0) {
        ftn_split(k, ns, u, v);
        atomicAdd(&running[par], 1ull);
    }
}

__global__ void __launch_bounds__(256) k_ftn_finish(NewtonState ns, int64_t K, double *x_out, double *f_out,
                                                    double *r_out, int32_t *st_out, int32_t *tr_out)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    newton_finish(k, ns, x_out, f_out, r_out, st_out, tr_out);
}

// Linear continuation predictor (Sec. 8), one row per thread.
__global__ void __launch_bounds__(256) k_cont_predict(const double *x0, const double *x1, const double *om0,
                                                      const double *om1, const double *dom, int64_t K, double *out)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    double q = 0.0;
    if (x1) {
        if (dom[2 * k] != 0.0) q = dom[2 * k] / (om0[2 * k] - om1[2 * k]);
        else if (dom[2 * k + 1] != 0.0) q = dom[2 * k + 1] / (om0[2 * k + 1] - om1[2 * k + 1]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const double a = x0[4 * k + c];
        out[4 * k + c] = x1 ? a + q * (a - x1[4 * k + c]) : a;
    }
}

// Workspace layout of ft_newton for K problems (256-byte aligned pieces).
struct FtnLayout {
    size_t total;
    size_t o[24];
};

FtnLayout ftn_layout(int64_t K)
{
    FtnLayout L;
    const size_t d4b = (size_t)K * 32, d1b = (size_t)K * 8, i1b = (size_t)K * 4, d16b = (size_t)K * 128;
    const size_t sizes[] = {d4b, d4b, d4b, d4b, d1b, d1b, i1b, i1b, i1b,     // p q delta fp rp alpha status trials based
                            d1b, d1b, d4b, d4b, d4b, d16b,                   // side u: th s w dth ds stm
                            d1b, d1b, d4b, d4b, d4b, d16b,                   // side s
                            16};                                             // running counters
    size_t at = 0;
    for (size_t i = 0; i < sizeof(sizes) / sizeof(sizes[0]); ++i) {
        L.o[i] = at;
        at += (sizes[i] + 255) & ~(size_t)255;
    }
    L.total = at;
    return L;
}

}  // namespace
}  // namespace ms

using namespace ms;

extern "C" int continuation_predict(const double *x0_dev, const double *omega0_dev, const double *domega_dev,
                                    const double *x1_dev, const double *omega1_dev, int64_t K, double *out_dev,
                                    void *stream)
{
    if (K < 0 || (K > 0 && (!x0_dev || !out_dev || (x1_dev && (!omega0_dev || !omega1_dev || !domega_dev)))))
        return fail(MS_E_ARG, "continuation_predict: bad argument");
    if (K == 0) return MS_OK;
    if (ceil_div(K, 256) > 0x7fffffff) return fail(MS_E_ARG, "continuation_predict: too many rows");
    hipLaunchKernelGGL(k_cont_predict, dim3((unsigned)ceil_div(K, 256)), dim3(256), 0, (hipStream_t)stream, x0_dev,
                       x1_dev, omega0_dev, omega1_dev, domega_dev, K, out_dev);
    MS_HIP(hipGetLastError());
    return MS_OK;
}

extern "C" int ft_newton_workspace_size(int64_t K, size_t *bytes)
{
    if (K < 0 || !bytes) return fail(MS_E_ARG, "ft_newton_workspace_size: bad argument");
    *bytes = ftn_layout(K).total;
    return MS_OK;
}

extern "C" int ft_newton(const double *params_in_dev, double *params_out_dev, int64_t K, const ft_chart_t *U,
                         const ft_chart_t *S, const map_params_t *map, const newton_params_t *np, double *f_dev,
                         double *r_dev, int32_t *status_dev, int32_t *trials_dev, void *ws, size_t ws_bytes,
                         void *stream)
{
    if (K < 0 || !U || !S || !map || !np || (K > 0 && (!params_in_dev || !params_out_dev)))
        return fail(MS_E_ARG, "ft_newton: bad argument");
    if (np->max_trials < 0 || np->max_trials > 100000) return fail(MS_E_ARG, "ft_newton: max_trials out of range");
    if (!(np->alpha0 > 0.0 && np->alpha0 <= 1.0) || !(np->alpha_min > 0.0) || !(np->tol >= 0.0))
        return fail(MS_E_ARG, "ft_newton: need 0 < alpha0 <= 1, alpha_min > 0, tol >= 0");
    if (!U->spec_dev || !S->spec_dev) return fail(MS_E_ARG, "ft_newton: chart spectra missing");
    if (K == 0) return MS_OK;
    if (K > ((int64_t)1 << 28)) return fail(MS_E_ARG, "ft_newton: K too large");
    const FtnLayout L = ftn_layout(K);
    if (!ws || ws_bytes < L.total) return fail(MS_E_WORKSPACE, "ft_newton: workspace too small");
    char *w = (char *)ws;
    NewtonState ns;
    ns.p = (double *)(w + L.o[0]);
    ns.q = (double *)(w + L.o[1]);
    ns.delta = (double *)(w + L.o[2]);
    ns.fp = (double *)(w + L.o[3]);
    ns.rp = (double *)(w + L.o[4]);
    ns.alpha = (double *)(w + L.o[5]);
    ns.status = (int32_t *)(w + L.o[6]);
    ns.trials = (int32_t *)(w + L.o[7]);
    ns.based = (int32_t *)(w + L.o[8]);
    FtSide su{(double *)(w + L.o[9]), (double *)(w + L.o[10]), (double *)(w + L.o[11]), (double *)(w + L.o[12]),
              (double *)(w + L.o[13]), (double *)(w + L.o[14])};
    FtSide ss{(double *)(w + L.o[15]), (double *)(w + L.o[16]), (double *)(w + L.o[17]), (double *)(w + L.o[18]),
              (double *)(w + L.o[19]), (double *)(w + L.o[20])};
    unsigned long long *running = (unsigned long long *)(w + L.o[21]);
    NewtonCfg cfg;
    cfg.tol2 = np->tol * np->tol;
    cfg.alpha0 = np->alpha0;
    cfg.alpha_min = np->alpha_min;
    cfg.max_trials = np->max_trials;
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid((unsigned)ceil_div(K, 256));
    map_params_t mu_map = *map, ms_map = *map;
    mu_map.n_periods = U->n_periods;
    ms_map.n_periods = S->n_periods;
    hipLaunchKernelGGL(k_ftn_init, grid, dim3(256), 0, st, params_in_dev, ns, K, su, ss, running);
    MS_HIP(hipGetLastError());
    for (int it = 0; it <= np->max_trials; ++it) {
        int rc = ft_partials(U->spec_dev, U->n_theta, U->order, su.th, su.s, K, U->omega, U->lambda, &mu_map, su.w,
                             su.dth, su.ds, su.stm, stream);
        if (rc) return rc;
        rc = ft_partials(S->spec_dev, S->n_theta, S->order, ss.th, ss.s, K, S->omega, S->lambda, &ms_map, ss.w,
                         ss.dth, ss.ds, ss.stm, stream);
        if (rc) return rc;
        const int par = it & 1;
        hipLaunchKernelGGL(k_ftn_update, grid, dim3(256), 0, st, ns, cfg, K, su, ss, running, par);
        MS_HIP(hipGetLastError());
        unsigned long long left = 0;
        MS_HIP(hipMemcpyAsync(&left, running + par, sizeof left, hipMemcpyDeviceToHost, st));
        MS_HIP(hipStreamSynchronize(st));
        if (left == 0) break;
    }
    hipLaunchKernelGGL(k_ftn_finish, grid, dim3(256), 0, st, ns, K, params_out_dev, f_dev, r_dev, status_dev,
                       trials_dev);
    MS_HIP(hipGetLastError());
    return MS_OK;
}

extern "C" int ft_partials(const double *spec_dev, int32_t n_theta, int32_t order, const double *theta_dev,
                           const double *s_dev, int64_t n_query, double omega, double lambda,
                           const map_params_t *map, double *w_dev, double *dth_dev, double *ds_dev,
                           double *stm_dev, void *stream)
{
    if (n_query < 0 || n_theta < 1 || order < 0 ||
        (n_query > 0 && (!spec_dev || !theta_dev || !s_dev || !w_dev || !dth_dev || !ds_dev)))
        return fail(MS_E_ARG, "ft_partials: bad argument");
    const int m = map ? map->n_periods : 0;
    if (m != 0 && !stm_dev) return fail(MS_E_ARG, "ft_partials: stm_dev is required when n_periods != 0");
    if (m != 0 && !(lambda > 0.0 && isfinite(lambda) && isfinite(omega)))
        return fail(MS_E_ARG, "ft_partials: need a finite omega and lambda > 0");
    if (n_query == 0) return MS_OK;
    if (ceil_div(n_query, 4) > 0x7fffffff) return fail(MS_E_ARG, "ft_partials: too many queries for one launch");
    hipStream_t st = (hipStream_t)stream;
    const double th_off = (double)m * omega;
    const double s_scale = m == 0 ? 1.0 : pow(lambda, -(double)m);
    const FtArgs g{spec_dev, theta_dev, s_dev, w_dev, dth_dev, ds_dev, n_query, th_off, s_scale, (int)n_theta, (int)order};
    const auto eval = n_query <= 256 ? launch_ft_eval<1>
                      : !tiles_pay(n_query, n_theta, order) ? launch_ft_eval<4>
                      : order <= 3 ? launch_ft_tile<1> : order <= 7 ? launch_ft_tile<2>
                      : order <= 15 ? launch_ft_tile<4> : launch_ft_tile<7>;
    eval(g, st);
    MS_HIP(hipGetLastError());
    if (m == 0) return MS_OK;
    int rc = pertbp_map_stm(w_dev, w_dev, stm_dev, n_query, map, 0, stream);
    if (rc) return rc;
    hipLaunchKernelGGL(k_apply_stm, dim3((unsigned)ceil_div(n_query, 256)), dim3(256), 0, st, stm_dev, dth_dev,
                       ds_dev, n_query);
    MS_HIP(hipGetLastError());
    return MS_OK;
}
