// refine.hip -- the refinement problem of Sec. 7 on the GPU.
//
// For two parameterised patches x_u(th1, s1) = bu + th1 du1 + s1 du2 and
// x_s(th2, s2) = bs + th2 ds1 + s2 ds2, the mismatch is
//   f(th1, s1, th2, s2) = F^{n_u}(x_u(th1, s1)) - F^{n_s}(x_s(th2, s2)),
// with F the stroboscopic map integrated by the fixed-step order-8 method.
//   * residual: f and r = |f|^2;
//   * tangent: the Jacobian J = df/d(th1, s1, th2, s2, e) by integrating the
//     variational equations with the same method (the state transition
//     matrices DF^m of Sec. 7, applied to the patch directions), exactly the
//     derivative of the discrete map; e enters through w(f) = 1/(1 + e cos f);
//   * adjoint: the gradient of r by the discrete adjoint (transpose) of every
//     Runge-Kutta step, run backwards from the seed dr/dF = +-2f a segment of
//     steps at a time, with the forward states kept only every `ckpt_every`
//     steps;
//   * damped Newton (Sec. 7): x <- x - alpha Df^{-1} f, alpha halved until r
//     decreases.
//
// Two lanes per trajectory (hit, side) for the state pass and per
// (trajectory, tangent column) for the tangent pass (one each in batches that
// fill the chip), one thread per (segment, trajectory, column) for the
// adjoint's segment Jacobians; blocks of one wave, so that the few hundred to
// few thousand trajectories spread over the compute units.
#include <math.h>
#include <string.h>

#include "newton.hpp"
#include "rk8_pair.hpp"

namespace ms {

// The tableau in constant memory, initialised at compile time (every device
// holds it from the moment the code object is loaded).
__constant__ Tableau c_cv = cv_make_tableau();

namespace {

constexpr int S = RK_S;
constexpr int RF_CHUNK = 32;         // steps of stage values in LDS
constexpr int RF_BLOCK = 64;

struct SideMap {
    const double *w;       // stage values w(f), steps x S (in the workspace)
    const double *dwde;    // stage values dw/de, steps x S (in the workspace)
    int64_t nsteps;
    int32_t steps;         // steps per period
    int32_t pad;
};

struct RefArgs {
    RkCoef hc[2];           // scaled coefficients of each side (first: step_coef reads them from the kernel arguments)
    const double *params;   // K x 4 (th1, s1, th2, s2)
    const double *U, *Sp;   // patches, 12 doubles each (base, d1, d2)
    int64_t K;
    int64_t pstride;        // doubles between consecutive hits' patches (0 or 12)
    Model md;
    SideMap side[2];        // 0: unstable side (x_u), 1: stable side (x_s)
    int64_t ck;             // checkpoint interval (steps)
    double *ckpt;           // n_ck x 2K x 4 (adjoint; NULL otherwise)
    double *yend;           // 2K x 4
    double *dend;           // 3 x 2K x 4 (tangent)
    double *gpart;          // 2K x 3 (adjoint)
    const int32_t *status;  // K Newton status words; only hits with status < 0 run (NULL: all run)
};

MS_D void store_d4(double *p, const double *y)
{
    double2 *o = reinterpret_cast<double2 *>(p);
    o[0] = make_double2(y[0], y[1]);
    o[1] = make_double2(y[2], y[3]);
}

// Start of a hit's trajectory on one side: the patch point x(th, s) =
// base + th d1 + s d2 (each operation rounded as written).
MS_D void traj_start(const RefArgs &a, int side, int64_t k, double y[4], const double *&patch)
{
    const double *pr = a.params + 4 * k + 2 * side;
    patch = (side ? a.Sp : a.U) + a.pstride * k;
    double th = pr[0], s = pr[1];
#pragma unroll
    for (int c = 0; c < 4; ++c) y[c] = (patch[c] + th * patch[4 + c]) + s * patch[8 + c];
}

MS_D bool hit_active(const RefArgs &a, int64_t k) { return a.status == nullptr || a.status[k] < 0; }

// The coefficients of a side for one-lane steps (k_adj_segments and large
// batches): scalar, as the side is the grid's y index and so the same for
// every thread.
MS_D CoefPtr side_coef(int side) { return step_coef() + side * RK_NC; }

// Hits up to which trajectories run on pairs of lanes: those whose waves have
// a SIMD each (1,024 waves of 32 pairs, and two trajectories a hit; with the
// tangents' three columns, six).  The state pass then takes 9.1 ms for 12,000
// steps, 16 with one lane each, and the tangent pass 1.52 us a step against
// 1.9; with a second wave on a SIMD pairs take longer than one lane a column
// (8,192 hits: 1,062 us for 400 steps against 820).  The rules
// depend on K alone, so that the forward pass and the adjoint's recomputation
// run the same code.
constexpr int64_t PAIR_HITS = 1024 * 32 / 2;
constexpr int64_t PAIR_TANGENT_HITS = 1024 * 32 / 6;

// Steps [s0, s1) of a trajectory, on a block of one wave: of the state alone
// (COL = false) or of the state and one tangent column (the variational
// equations v' = A(f, y) v, plus dF/de when `ecol`, integrated with the same
// stages, which is the exact derivative of the discrete step).  PAIR: two
// lanes per trajectory, y = (own coordinate, own velocity, then the
// column's); else y = (x, y, x', y', then the column).  The stage values of
// RF_CHUNK steps lie in LDS and the next chunk's are on their way from the
// tables meanwhile.  before(s, y) sees the state before step s.
template <bool PAIR, bool COL>
constexpr int flow_dim() { return (PAIR ? 2 : 4) * (COL ? 2 : 1); }

template <bool PAIR, bool COL, typename BEFORE>
MS_D void ref_flow(const RefArgs &a, int side, bool live, int64_t s0, int64_t s1, bool ecol,
                   double (&y)[flow_dim<PAIR, COL>()], BEFORE &&before)
{
    constexpr int D = flow_dim<PAIR, COL>(), N = RF_CHUNK * S, PER = (N + RF_BLOCK - 1) / RF_BLOCK;
    __shared__ double s_w[N], s_d[COL ? N : 1];
    // A wave whose hits are all done (the block is one wave) leaves at once:
    // the refinement queues all its passes in advance, and one that goes
    // through the chunks of 12,000 steps without a step takes 274 us, not 4.
    if (ballot(live) == 0) return;
    const SideMap &sm = a.side[side];
    const int64_t tot = (int64_t)sm.steps * S;
    const double ec = ecol ? 1.0 : 0.0;
    double nw[PER], nd[COL ? PER : 1];
    auto fetch = [&](int64_t s) {
        const int64_t base = (s % sm.steps) * S;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = threadIdx.x + q * RF_BLOCK;
            int64_t k = base + i;
            while (k >= tot) k -= tot;
            if (i < N) {
                nw[q] = sm.w[k];
                if constexpr (COL) nd[q] = sm.dwde[k];
            }
        }
    };
    PairCoef pc;
    PairLane L;
    if constexpr (PAIR) {
        pair_coef(pc, a.hc[side]);
        L = pair_lane(a.md, threadIdx.x & 1);
    }
    if (s0 < s1) fetch(s0);
    for (int64_t sc = s0; sc < s1; sc += RF_CHUNK) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = threadIdx.x + q * RF_BLOCK;
            if (i < N) {
                s_w[i] = nw[q];
                if constexpr (COL) s_d[i] = nd[q];
            }
        }
        __syncthreads();
        if (sc + RF_CHUNK < s1) fetch(sc + RF_CHUNK);
        const int cnt = s1 - sc < RF_CHUNK ? (int)(s1 - sc) : RF_CHUNK;
        if (!live) continue;
#pragma unroll 1
        for (int jj = 0; jj < cnt; ++jj) {
            before(sc + jj, y);
            const double *w = s_w + jj * S, *d = s_d + jj * S;
            if constexpr (PAIR) {
                rk_step<D>(y, pc, [&](int i, double (&s)[D]) {
                    puls_pair<COL>(L, w[i], COL ? ec * d[i] : 0.0, s);
                });
            } else {
                rk_step<D>(y, side_coef(side), [&](int i, double (&s)[D]) {
                    if constexpr (COL) puls_field_var(a.md, w[i], ec * d[i], s);
                    else puls_field(a.md, w[i], s);
                });
            }
        }
    }
}

// A trajectory's four components to or from the lane's part of y (v: the
// first of them, at y[OFF]).
template <bool PAIR, int OFF, int D>
MS_D void put_state(double *p, const double (&y)[D])
{
    if constexpr (PAIR) {
        const int l = threadIdx.x & 1;
        p[l] = y[OFF];
        p[2 + l] = y[OFF + 1];
    } else {
        store_d4(p, y + OFF);
    }
}

template <bool PAIR, int OFF, int D>
MS_D void get_state(const double *p, double (&y)[D])
{
    if constexpr (PAIR) {
        const int l = threadIdx.x & 1;
        y[OFF] = p[l];
        y[OFF + 1] = p[2 + l];
    } else {
        const d4 v = load_d4(p);
        y[OFF] = v.x; y[OFF + 1] = v.y; y[OFF + 2] = v.z; y[OFF + 3] = v.w;
    }
}

// State pass: endpoint of every trajectory; with a.ckpt, the state before
// every ck-th step.  The grid's y index is the side.
template <bool PAIR>
__global__ void __launch_bounds__(RF_BLOCK) k_ref_state(RefArgs a)
{
    constexpr int D = flow_dim<PAIR, false>();
    const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / (PAIR ? 2 : 1);
    const int64_t T2 = 2 * a.K, t = blockIdx.y * a.K + i;
    const bool live = i < a.K && hit_active(a, i);
    double y[D] = {};
    if (live) {
        double y0[4];
        const double *patch;
        traj_start(a, blockIdx.y, i, y0, patch);
        get_state<PAIR, 0>(y0, y);
    }
    int64_t next = 0;      // the next checkpoint's step
    ref_flow<PAIR, false>(a, blockIdx.y, live, 0, a.side[blockIdx.y].nsteps, false, y, [&](int64_t s, double (&v)[D]) {
        if (a.ckpt && s == next) {
            put_state<PAIR, 0>(a.ckpt + ((s / a.ck) * T2 + t) * 4, v);
            next += a.ck;
        }
    });
    if (live) put_state<PAIR, 0>(a.yend + 4 * t, y);
}

// Tangent pass: a trajectory and one of its columns d/dth, d/ds, d/de.
template <bool PAIR>
__global__ void __launch_bounds__(RF_BLOCK) k_ref_tangent(RefArgs a)
{
    constexpr int D = flow_dim<PAIR, true>(), C = D / 2;
    const int64_t gid = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / (PAIR ? 2 : 1);
    const int col = (int)(gid / a.K);
    const int64_t k = gid - col * a.K, T2 = 2 * a.K, t = blockIdx.y * a.K + k;
    const bool live = gid < 3 * a.K && hit_active(a, k), ecol = col == 2;
    double y[D] = {};
    if (live) {
        double y0[4];
        const double *patch;
        traj_start(a, blockIdx.y, k, y0, patch);
        get_state<PAIR, 0>(y0, y);
        if (!ecol) get_state<PAIR, C>(patch + 4 * (col + 1), y);
    }
    ref_flow<PAIR, true>(a, blockIdx.y, live, 0, a.side[blockIdx.y].nsteps, ecol, y, [](int64_t, double (&)[D]) {});
    if (!live) return;
    put_state<PAIR, C>(a.dend + ((int64_t)col * T2 + t) * 4, y);
    if (col == 0) put_state<PAIR, 0>(a.yend + 4 * t, y);
}

// f, r (and J, grad = 2 J^T f in tangent mode) per hit.
__global__ void __launch_bounds__(RF_BLOCK) k_ref_combine(RefArgs a, int tangent, double *f_out, double *r_out,
                                                          double *J_out, double *g_out)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.K) return;
    const int64_t T2 = 2 * a.K;
    const double *yu = a.yend + 4 * k, *ys = a.yend + 4 * (a.K + k);
    double f[4], r = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        f[c] = yu[c] - ys[c];
        r += f[c] * f[c];
    }
    if (f_out) store_d4(f_out + 4 * k, f);
    if (r_out) r_out[k] = r;
    if (!tangent) return;
    double J[4][5];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        J[c][0] = a.dend[(0 * T2 + k) * 4 + c];
        J[c][1] = a.dend[(1 * T2 + k) * 4 + c];
        J[c][2] = -a.dend[(0 * T2 + a.K + k) * 4 + c];
        J[c][3] = -a.dend[(1 * T2 + a.K + k) * 4 + c];
        J[c][4] = a.dend[(2 * T2 + k) * 4 + c] - a.dend[(2 * T2 + a.K + k) * 4 + c];
    }
    if (J_out)
        for (int c = 0; c < 4; ++c)
            for (int j = 0; j < 5; ++j) J_out[20 * k + 5 * c + j] = J[c][j];
    if (g_out)
        for (int j = 0; j < 5; ++j) {
            double acc = 0.0;
            for (int c = 0; c < 4; ++c) acc += J[c][j] * f[c];
            g_out[5 * k + j] = 2.0 * acc;
        }
}

// The adjoint goes backwards over segments of ADJ_SEG steps (counted from
// the first step, whatever the checkpoint interval, so that the result does
// not depend on that), a window of segments at a time.  For one window:
//   k_adj_states    per (checkpoint interval, trajectory): the states at the
//                   starts of the window's segments, recomputed from the
//                   checkpoints (not needed when these lie at the starts);
//   k_adj_segments  per (segment, trajectory, column): the Jacobian of the
//                   segment's steps, P = d y_end / d y_start (columns 0-3, a
//                   unit vector carried by the tangent steps) and
//                   d y_end / d e (column 4), all segments in parallel;
//   k_adj_reverse   per trajectory: lam <- P^T lam and ge += (d y_end/de) . lam
//                   from the last segment of the window down to the first.
// This is the transpose of the discrete map, segment by segment.  With a
// Jacobian per step instead (kept in memory, 160 bytes a step, and applied
// one after another) the backward part of 128 hits took 6.3 ms, 5.0 of them
// the 12,000 dependent loads and products of each trajectory; with segments
// 0.72 ms (0.67 for the Jacobians, which are bound by FP64 issue).
constexpr int64_t ADJ_SEG = 100;

template <bool PAIR>
__global__ void __launch_bounds__(RF_BLOCK) k_adj_states(RefArgs a, int64_t s_lo, int64_t s_hi, int64_t nblk,
                                                         double *states)
{
    constexpr int D = flow_dim<PAIR, false>();
    const int64_t T2 = 2 * a.K, seg = blockIdx.x / nblk;
    const int64_t i = ((blockIdx.x - seg * nblk) * blockDim.x + threadIdx.x) / (PAIR ? 2 : 1);
    const int64_t t = blockIdx.y * a.K + i, ck0 = s_lo / a.ck + seg;
    const int64_t s0 = ck0 * a.ck;
    int64_t s1 = s0 + a.ck < s_hi ? s0 + a.ck : s_hi;
    if (s1 > a.side[blockIdx.y].nsteps) s1 = a.side[blockIdx.y].nsteps;
    if (s0 >= s1) return;
    const bool live = i < a.K;
    double y[D] = {};
    if (live) get_state<PAIR, 0>(a.ckpt + (ck0 * T2 + t) * 4, y);
    // the first segment start at or after s0, and the last before s1: no
    // step past it is needed
    int64_t next = (s0 > s_lo ? (s0 + ADJ_SEG - 1) / ADJ_SEG * ADJ_SEG : s_lo);
    const int64_t last = (s1 - 1) / ADJ_SEG * ADJ_SEG;
    if (next > last) return;
    ref_flow<PAIR, false>(a, blockIdx.y, live, s0, last + 1, false, y, [&](int64_t s, double (&v)[D]) {
        if (s == next) {
            put_state<PAIR, 0>(states + ((s - s_lo) / ADJ_SEG * T2 + t) * 4, v);
            next += ADJ_SEG;
        }
    });
}

__global__ void __launch_bounds__(RF_BLOCK) __attribute__((amdgpu_waves_per_eu(3, 8)))
k_adj_segments(RefArgs a, int64_t s_lo, int64_t s_hi, int64_t nblk, const double *states, double *jac)
{
    const int64_t T2 = 2 * a.K, sg = blockIdx.x / nblk;
    const int64_t gid = (blockIdx.x - sg * nblk) * blockDim.x + threadIdx.x;
    const int64_t i = gid / 5, t = blockIdx.y * a.K + i;
    const int col = (int)(gid - i * 5);
    const int64_t s0 = s_lo + sg * ADJ_SEG;
    int64_t s1 = s0 + ADJ_SEG < s_hi ? s0 + ADJ_SEG : s_hi;
    if (s1 > a.side[blockIdx.y].nsteps) s1 = a.side[blockIdx.y].nsteps;
    if (s0 >= s1) return;
    const bool live = i < a.K;
    double y[8] = {};
    if (live) get_state<false, 0>(states + (sg * T2 + t) * 4, y);
#pragma unroll
    for (int c = 0; c < 4; ++c) y[4 + c] = c == col ? 1.0 : 0.0;
    ref_flow<false, true>(a, blockIdx.y, live, s0, s1, col == 4, y, [](int64_t, double (&)[8]) {});
    if (live) put_state<false, 4>(jac + ((sg * T2 + t) * 5 + col) * 4, y);
}

// lam (4) and ge per trajectory live in adj[5 t ...]; init seeds lam = +-2 f.
__global__ void __launch_bounds__(RF_BLOCK) k_adj_reverse(RefArgs a, int64_t s_lo, int64_t s_hi, const double *jac,
                                                          double *adj, const double *f, int init)
{
    const int64_t T2 = 2 * a.K;
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T2) return;
    const int side = t >= a.K ? 1 : 0;
    const int64_t k = t - (side ? a.K : 0);
    double lam[4], ge;
    if (init) {
        const double sg = side ? -2.0 : 2.0;
        for (int c = 0; c < 4; ++c) lam[c] = sg * f[4 * k + c];
        ge = 0.0;
    } else {
        for (int c = 0; c < 4; ++c) lam[c] = adj[5 * t + c];
        ge = adj[5 * t + 4];
    }
    const int64_t hi = s_hi < a.side[side].nsteps ? s_hi : a.side[side].nsteps;
#pragma unroll 4
    for (int64_t sg = (hi - s_lo + ADJ_SEG - 1) / ADJ_SEG - 1; sg >= 0; --sg) {
        const double *J = jac + (sg * T2 + t) * 20;   // 5 columns of 4
        double m[5][4];
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            const d4 q = load_d4(J + 4 * c);
            m[c][0] = q.x; m[c][1] = q.y; m[c][2] = q.z; m[c][3] = q.w;
        }
        ge += ((m[4][0] * lam[0] + m[4][1] * lam[1]) + m[4][2] * lam[2]) + m[4][3] * lam[3];
        double nl[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) nl[c] = ((m[c][0] * lam[0] + m[c][1] * lam[1]) + m[c][2] * lam[2]) + m[c][3] * lam[3];
#pragma unroll
        for (int c = 0; c < 4; ++c) lam[c] = nl[c];
    }
    for (int c = 0; c < 4; ++c) adj[5 * t + c] = lam[c];
    adj[5 * t + 4] = ge;
}

// Per trajectory: the gradient with respect to its patch parameters
// (lam . d1, lam . d2) and its share of d r / d e.
__global__ void __launch_bounds__(RF_BLOCK) k_adj_finish(RefArgs a, const double *adj)
{
    const int64_t T2 = 2 * a.K;
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T2) return;
    const int side = t >= a.K ? 1 : 0;
    const int64_t k = t - (side ? a.K : 0);
    const double *patch = (side ? a.Sp : a.U) + a.pstride * k;
    double g0 = 0.0, g1 = 0.0;
    for (int c = 0; c < 4; ++c) {
        g0 += adj[5 * t + c] * patch[4 + c];
        g1 += adj[5 * t + c] * patch[8 + c];
    }
    a.gpart[3 * t + 0] = g0;
    a.gpart[3 * t + 1] = g1;
    a.gpart[3 * t + 2] = adj[5 * t + 4];
}

__global__ void __launch_bounds__(RF_BLOCK) k_ref_grad(RefArgs a, double *g_out)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.K) return;
    const double *gu = a.gpart + 3 * k, *gs = a.gpart + 3 * (a.K + k);
    g_out[5 * k + 0] = gu[0];
    g_out[5 * k + 1] = gu[1];
    g_out[5 * k + 2] = gs[0];
    g_out[5 * k + 3] = gs[1];
    g_out[5 * k + 4] = gu[2] + gs[2];
}

// The stage values of both sides for one period (entry (n, i) at step n of
// a period, stage i), into the workspace: w, and dw/de when wanted.
struct TableArgs {
    double *w[2], *dwde[2];
    int32_t steps[2];
    double e;
};

__global__ void __launch_bounds__(256) k_ref_tables(TableArgs t)
{
    const int64_t n0 = (int64_t)t.steps[0] * S, n1 = (int64_t)t.steps[1] * S;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n0 + n1) return;
    const int sd = i >= n0;
    const int64_t k = sd ? i - n0 : i;
    const int64_t step = k / S;
    const int q = (int)(k - step * S);
    const double cf = cos(stage_abscissa(step, c_cv.c[q], t.steps[sd]));
    const double om = 1.0 / (1.0 + t.e * cf);
    t.w[sd][k] = om;
    if (t.dwde[sd]) t.dwde[sd][k] = -cf * om * om;
}

// ------------------------------------------------------------ damped Newton

__global__ void __launch_bounds__(RF_BLOCK) k_newton_init(const double *x0, NewtonState ns, int64_t K)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    newton_init(k, x0, ns);
}

// One decision per running hit after the tangent pass at its trial point q.
__global__ void __launch_bounds__(RF_BLOCK) k_newton_update(RefArgs a, NewtonState ns, NewtonCfg cfg)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.K || ns.status[k] >= 0) return;
    const int64_t T2 = 2 * a.K;
    const double *yu = a.yend + 4 * k, *ys = a.yend + 4 * (a.K + k);
    double f[4], M[4][4];
    for (int c = 0; c < 4; ++c) {
        f[c] = yu[c] - ys[c];
        M[c][0] = a.dend[(0 * T2 + k) * 4 + c];
        M[c][1] = a.dend[(1 * T2 + k) * 4 + c];
        M[c][2] = -a.dend[(0 * T2 + a.K + k) * 4 + c];
        M[c][3] = -a.dend[(1 * T2 + a.K + k) * 4 + c];
    }
    newton_decide(k, f, M, ns, cfg);
}

__global__ void __launch_bounds__(RF_BLOCK) k_newton_finish(NewtonState ns, int64_t K, double *x_out, double *f_out,
                                                            double *r_out, int32_t *st_out, int32_t *tr_out)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    newton_finish(k, ns, x_out, f_out, r_out, st_out, tr_out);
}

// ---------------------------------------------------------------- host side

struct RefLayout {
    size_t o_w[2], o_dwde[2], o_yend, o_dend, o_gpart, o_ckpt, o_states, o_jac, o_adj, o_nw, total;
    int64_t n_ck, win_steps, n_steps_max;
};

inline size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

int64_t side_steps(const map_params_t *m)
{
    int64_t np = m->n_periods < 0 ? -(int64_t)m->n_periods : m->n_periods;
    return (int64_t)m->steps_per_period * np;
}

int check_maps(const map_params_t *fwd, const map_params_t *bwd)
{
    if (!fwd || !bwd) return fail(MS_E_ARG, "refine: NULL map parameters");
    for (const map_params_t *m : {fwd, bwd}) {
        if (m->steps_per_period <= 0) return fail(MS_E_ARG, "refine: steps_per_period must be > 0");
        if (!(m->e >= 0.0 && m->e < 1.0) || !(m->mu >= 0.0 && m->mu <= 1.0))
            return fail(MS_E_ARG, "refine: need 0 <= e < 1 and 0 <= mu <= 1");
    }
    if (fwd->mu != bwd->mu || fwd->e != bwd->e)
        return fail(MS_E_ARG, "refine: both sides must use the same mu and e");
    return MS_OK;
}

// Segments per adjoint window: as many as fit ADJ_WINDOW_BYTES of start
// states and segment Jacobians (at least one).
constexpr int64_t ADJ_WINDOW_BYTES = (int64_t)256 << 20;
constexpr int64_t ADJ_BYTES_PER_SEG = 32 + 5 * 32;   // per trajectory: state + 5 Jacobian columns

RefLayout ref_layout(int64_t K, const map_params_t *fwd, const map_params_t *bwd, int32_t ck, int32_t mode)
{
    RefLayout L;
    memset(&L, 0, sizeof L);
    const size_t T2 = (size_t)(2 * K);
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = al256(o + (bytes ? bytes : 1)); return at; };
    const map_params_t *m[2] = {fwd, bwd};
    for (int sd = 0; sd < 2; ++sd) {
        const size_t tb = (size_t)m[sd]->steps_per_period * S * 8;
        L.o_w[sd] = take(tb);
        L.o_dwde[sd] = take(mode != MS_REFINE_RESIDUAL ? tb : 0);
    }
    L.o_yend = take(T2 * 32);
    L.o_dend = take((mode == MS_REFINE_TANGENT || mode == MS_REFINE_NEWTON) ? 3 * T2 * 32 : 0);
    L.o_gpart = take(mode == MS_REFINE_ADJOINT ? T2 * 24 : 0);
    if (mode == MS_REFINE_ADJOINT) {
        const int64_t a = side_steps(fwd), b = side_steps(bwd);
        L.n_steps_max = a > b ? a : b;
        L.n_ck = ceil_div(L.n_steps_max, ck);
        const int64_t n_seg = ceil_div(L.n_steps_max, ADJ_SEG);
        int64_t segs = ADJ_WINDOW_BYTES / ((int64_t)(T2 > 0 ? T2 : 1) * ADJ_BYTES_PER_SEG);
        if (segs > n_seg) segs = n_seg;
        if (segs > (1 << 20) / ADJ_SEG) segs = (1 << 20) / ADJ_SEG;     // (launch sizes in 32 bits)
        if (segs < 1) segs = 1;
        L.win_steps = segs * ADJ_SEG;
        L.o_ckpt = take((size_t)L.n_ck * T2 * 32);
        L.o_states = take((size_t)segs * T2 * 32);
        L.o_jac = take((size_t)segs * T2 * 160);
        L.o_adj = take(T2 * 40);
    } else {
        L.o_ckpt = take(0);
        L.o_states = take(0);
        L.o_jac = take(0);
        L.o_adj = take(0);
    }
    L.o_nw = take(mode == MS_REFINE_NEWTON ? (size_t)K * (18 * 8 + 3 * 4) + 9 * 256 : 0);
    L.total = o;
    return L;
}

// Kernel arguments of one call, with the stage values of both sides in the
// workspace; queues the kernel that computes them.
int make_args(RefArgs &a, const double *params, int64_t K, const patch_t *U, const patch_t *Sp, int32_t stride,
              const map_params_t *fwd, const map_params_t *bwd, int32_t ck, int need_dwde, char *ws,
              const RefLayout &L, hipStream_t st)
{
    if (!cv_pattern_ok()) return fail(MS_E_ARG, "refine: internal tableau pattern mismatch");
    memset(&a, 0, sizeof a);
    a.params = params;
    a.U = (const double *)U;
    a.Sp = (const double *)Sp;
    a.K = K;
    a.pstride = stride ? 12 : 0;
    a.md = Model{fwd->mu, 1.0 - fwd->mu};
    a.ck = ck;
    const map_params_t *m[2] = {fwd, bwd};
    TableArgs t;
    t.e = fwd->e;
    for (int sd = 0; sd < 2; ++sd) {
        SideMap &sm = a.side[sd];
        t.w[sd] = (double *)(ws + L.o_w[sd]);
        t.dwde[sd] = need_dwde ? (double *)(ws + L.o_dwde[sd]) : nullptr;
        t.steps[sd] = m[sd]->steps_per_period;
        sm.w = t.w[sd];
        sm.dwde = need_dwde ? t.dwde[sd] : t.w[sd];
        sm.nsteps = side_steps(m[sd]);
        sm.steps = m[sd]->steps_per_period;
        a.hc[sd] = rk_coef((m[sd]->n_periods < 0 ? -RK_TWO_PI : RK_TWO_PI) / (double)m[sd]->steps_per_period);
    }
    const int64_t n = ((int64_t)t.steps[0] + t.steps[1]) * S;
    MS_LAUNCH("k_ref_tables", k_ref_tables, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, t);
    MS_HIP(hipGetLastError());
    return MS_OK;
}

unsigned blocks_for(int64_t n) { return (unsigned)ceil_div(n > 0 ? n : 1, RF_BLOCK); }

void launch_tangent(const RefArgs &a, hipStream_t st)
{
    if (a.K <= PAIR_TANGENT_HITS)
        MS_LAUNCH("k_ref_tangent", k_ref_tangent<true>, dim3(blocks_for(6 * a.K), 2), dim3(RF_BLOCK), 0, st, a);
    else
        MS_LAUNCH("k_ref_tangent", k_ref_tangent<false>, dim3(blocks_for(3 * a.K), 2), dim3(RF_BLOCK), 0, st, a);
}

}  // namespace
}  // namespace ms

using namespace ms;

extern "C" int refine_workspace_size(int64_t K, const map_params_t *fwd, const map_params_t *bwd, int32_t ckpt_every,
                                     int32_t mode, size_t *bytes)
{
    if (!bytes || K < 0) return fail(MS_E_ARG, "refine_workspace_size: bad argument");
    int rc = check_maps(fwd, bwd);
    if (rc) return rc;
    if (mode < MS_REFINE_RESIDUAL || mode > MS_REFINE_NEWTON) return fail(MS_E_ARG, "refine_workspace_size: bad mode");
    if (mode == MS_REFINE_ADJOINT && ckpt_every <= 0) return fail(MS_E_ARG, "refine: ckpt_every must be > 0");
    *bytes = ref_layout(K, fwd, bwd, ckpt_every > 0 ? ckpt_every : 1, mode).total;
    return MS_OK;
}

extern "C" int refine_grad(const double *params_dev, int64_t K, const patch_t *U_dev, const patch_t *S_dev,
                           int32_t patch_stride, const map_params_t *fwd, const map_params_t *bwd, int32_t ckpt_every,
                           int32_t mode, double *f_dev, double *r_dev, double *grad_dev, double *J_dev, void *ws,
                           size_t ws_bytes, void *stream)
{
    if (K < 0 || (K > 0 && (!params_dev || !U_dev || !S_dev))) return fail(MS_E_ARG, "refine_grad: bad argument");
    if (patch_stride != 0 && patch_stride != 1) return fail(MS_E_ARG, "refine_grad: patch_stride must be 0 or 1");
    if (mode < MS_REFINE_RESIDUAL || mode > MS_REFINE_TANGENT) return fail(MS_E_ARG, "refine_grad: bad mode");
    if (mode == MS_REFINE_ADJOINT && ckpt_every <= 0) return fail(MS_E_ARG, "refine_grad: the adjoint needs ckpt_every > 0");
    if (K > ((int64_t)1 << 28)) return fail(MS_E_ARG, "refine_grad: K too large");
    int rc = check_maps(fwd, bwd);
    if (rc) return rc;
    if (K == 0) return MS_OK;
    if (mode == MS_REFINE_ADJOINT && (!f_dev || !grad_dev))
        return fail(MS_E_ARG, "refine_grad: the adjoint needs f_dev and grad_dev");
    const int32_t ck = mode == MS_REFINE_ADJOINT ? ckpt_every : 1;
    RefLayout L = ref_layout(K, fwd, bwd, ck, mode);
    if (!ws || ws_bytes < L.total) return fail(MS_E_WORKSPACE, "refine_grad: workspace too small");
    char *w = (char *)ws;
    hipStream_t st = (hipStream_t)stream;
    RefArgs a;
    if ((rc = make_args(a, params_dev, K, U_dev, S_dev, patch_stride, fwd, bwd, ck, mode != MS_REFINE_RESIDUAL, w, L,
                        st)))
        return rc;
    a.yend = (double *)(w + L.o_yend);
    a.dend = (double *)(w + L.o_dend);
    a.gpart = (double *)(w + L.o_gpart);
    const int64_t T2 = 2 * K;
    const bool pair = K <= PAIR_HITS;
    if (mode == MS_REFINE_TANGENT) {
        launch_tangent(a, st);
        MS_LAUNCH("k_ref_combine", k_ref_combine, dim3(blocks_for(K)), dim3(RF_BLOCK), 0, st, a, 1, f_dev, r_dev, J_dev,
                  grad_dev);
    } else {
        if (mode == MS_REFINE_ADJOINT) a.ckpt = (double *)(w + L.o_ckpt);
        if (pair)
            MS_LAUNCH("k_ref_state", k_ref_state<true>, dim3(blocks_for(2 * K), 2), dim3(RF_BLOCK), 0, st, a);
        else
            MS_LAUNCH("k_ref_state", k_ref_state<false>, dim3(blocks_for(K), 2), dim3(RF_BLOCK), 0, st, a);
        MS_LAUNCH("k_ref_combine", k_ref_combine, dim3(blocks_for(K)), dim3(RF_BLOCK), 0, st, a, 0, f_dev, r_dev,
                  (double *)nullptr, (double *)nullptr);
        if (mode == MS_REFINE_ADJOINT) {
            double *states = (double *)(w + L.o_states), *jac = (double *)(w + L.o_jac), *adj = (double *)(w + L.o_adj);
            const int64_t W = L.win_steps;
            int64_t nwin = ceil_div(L.n_steps_max, W);
            if (nwin < 1) nwin = 1;
            for (int64_t wi = nwin - 1; wi >= 0; --wi) {
                const int64_t s_lo = wi * W;
                const int64_t s_hi = s_lo + W < L.n_steps_max ? s_lo + W : L.n_steps_max;
                // the window's start states: the checkpoints themselves when they
                // lie at the segments' starts
                const double *from = ck == ADJ_SEG ? a.ckpt + (s_lo / ADJ_SEG) * T2 * 4 : states;
                if (s_hi > s_lo) {
                    if (ck != ADJ_SEG) {
                        const int64_t nck = ceil_div(s_hi, (int64_t)ck) - s_lo / ck;
                        const unsigned nb = blocks_for(pair ? 2 * K : K);
                        const dim3 grid((unsigned)(nck * nb), 2);
                        if (pair)
                            MS_LAUNCH("k_adj_states", k_adj_states<true>, grid, dim3(RF_BLOCK), 0, st, a, s_lo, s_hi,
                                      (int64_t)nb, states);
                        else
                            MS_LAUNCH("k_adj_states", k_adj_states<false>, grid, dim3(RF_BLOCK), 0, st, a, s_lo, s_hi,
                                      (int64_t)nb, states);
                    }
                    const unsigned nb = blocks_for(5 * K);
                    MS_LAUNCH("k_adj_segments", k_adj_segments,
                              dim3((unsigned)(ceil_div(s_hi - s_lo, ADJ_SEG) * nb), 2), dim3(RF_BLOCK), 0, st, a, s_lo,
                              s_hi, (int64_t)nb, from, jac);
                }
                MS_LAUNCH("k_adj_reverse", k_adj_reverse, dim3(blocks_for(T2)), dim3(RF_BLOCK), 0, st, a, s_lo, s_hi,
                          (const double *)jac, adj, (const double *)f_dev, (int)(wi == nwin - 1));
            }
            MS_LAUNCH("k_adj_finish", k_adj_finish, dim3(blocks_for(T2)), dim3(RF_BLOCK), 0, st, a, (const double *)adj);
            MS_LAUNCH("k_ref_grad", k_ref_grad, dim3(blocks_for(K)), dim3(RF_BLOCK), 0, st, a, grad_dev);
        }
    }
    MS_HIP(hipGetLastError());
    return MS_OK;
}

extern "C" int refine_newton(const double *params_in_dev, double *params_out_dev, int64_t K, const patch_t *U_dev,
                             const patch_t *S_dev, int32_t patch_stride, const map_params_t *fwd,
                             const map_params_t *bwd, const newton_params_t *np, double *f_dev, double *r_dev,
                             int32_t *status_dev, int32_t *trials_dev, void *ws, size_t ws_bytes, void *stream)
{
    if (K < 0 || !np || (K > 0 && (!params_in_dev || !params_out_dev || !U_dev || !S_dev)))
        return fail(MS_E_ARG, "refine_newton: bad argument");
    if (patch_stride != 0 && patch_stride != 1) return fail(MS_E_ARG, "refine_newton: patch_stride must be 0 or 1");
    if (np->max_trials < 0 || np->max_trials > 100000) return fail(MS_E_ARG, "refine_newton: max_trials out of range");
    if (!(np->alpha0 > 0.0 && np->alpha0 <= 1.0) || !(np->alpha_min > 0.0) || !(np->tol >= 0.0))
        return fail(MS_E_ARG, "refine_newton: need 0 < alpha0 <= 1, alpha_min > 0, tol >= 0");
    if (K > ((int64_t)1 << 28)) return fail(MS_E_ARG, "refine_newton: K too large");
    int rc = check_maps(fwd, bwd);
    if (rc) return rc;
    if (K == 0) return MS_OK;
    RefLayout L = ref_layout(K, fwd, bwd, 1, MS_REFINE_NEWTON);
    if (!ws || ws_bytes < L.total) return fail(MS_E_WORKSPACE, "refine_newton: workspace too small");
    char *w = (char *)ws;
    NewtonState ns;
    {
        size_t o = L.o_nw;
        auto take = [&](size_t bytes) { size_t at = o; o = al256(o + bytes); return w + at; };
        ns.p = (double *)take((size_t)K * 32);
        ns.q = (double *)take((size_t)K * 32);
        ns.delta = (double *)take((size_t)K * 32);
        ns.fp = (double *)take((size_t)K * 32);
        ns.rp = (double *)take((size_t)K * 8);
        ns.alpha = (double *)take((size_t)K * 8);
        ns.status = (int32_t *)take((size_t)K * 4);
        ns.trials = (int32_t *)take((size_t)K * 4);
        ns.based = (int32_t *)take((size_t)K * 4);
        if ((size_t)(o) > L.total) return fail(MS_E_WORKSPACE, "refine_newton: internal layout");
    }
    hipStream_t st = (hipStream_t)stream;
    RefArgs a;
    if ((rc = make_args(a, ns.q, K, U_dev, S_dev, patch_stride, fwd, bwd, 1, 1, w, L, st))) return rc;
    a.yend = (double *)(w + L.o_yend);
    a.dend = (double *)(w + L.o_dend);
    a.status = ns.status;
    NewtonCfg cfg;
    cfg.tol2 = np->tol * np->tol;
    cfg.alpha0 = np->alpha0;
    cfg.alpha_min = np->alpha_min;
    cfg.max_trials = np->max_trials;
    MS_LAUNCH("k_newton_init", k_newton_init, dim3(blocks_for(K)), dim3(RF_BLOCK), 0, st, params_in_dev, ns, K);
    for (int it = 0; it <= np->max_trials; ++it) {
        launch_tangent(a, st);
        MS_LAUNCH("k_newton_update", k_newton_update, dim3(blocks_for(K)), dim3(RF_BLOCK), 0, st, a, ns, cfg);
    }
    MS_LAUNCH("k_newton_finish", k_newton_finish, dim3(blocks_for(K)), dim3(RF_BLOCK), 0, st, ns, K, params_out_dev,
              f_dev, r_dev, status_dev, trials_dev);
    MS_HIP(hipGetLastError());
    return MS_OK;
}
