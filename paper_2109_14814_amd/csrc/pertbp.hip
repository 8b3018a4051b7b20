// pertbp.hip -- stroboscopic map F of the planar elliptic restricted
// three-body problem in the position-momentum coordinates of Sec. 3.3 (time t,
// frame turning with the primaries but not rescaled, periapse at t = 0), and
// its state transition matrix DF^m (the derivative the parameterization
// formulas of Sec. 7 need).
//
// Same fixed-step order-8 Runge-Kutta method as the pulsating map.  The
// time-dependent coefficients, the separation rho(t) of the primaries and the
// rate n(t) of their true anomaly, come from Kepler's equation; each block
// solves it for the stage times of RK_CHUNK steps at a time into LDS (both
// are 2 pi periodic and even in t, so one period's values serve every period
// and both directions).  Nothing is allocated; every call can be captured.
//
// The map runs one thread per state.  The matrix runs 4 / NC threads per
// state, each carrying the state and NC of the 4 tangent columns (the
// variational equations integrated with the same stages, so the result is
// the exact derivative of the discrete map): NC = 4 computes the field once
// per state (the default for large batches: fastest on gfx950 although it
// runs at one wave per SIMD: 60.3 ms for a period of 262,144 states, 62 at
// two waves with 140 bytes spilled), NC = 1 keeps the fewest registers live
// and gives small batches four times the threads.
#include <math.h>

#include <string>

#include "rk8_pair.hpp"

namespace ms {
namespace {

constexpr int PM_BLOCK = FLOW_BLOCK;

// NC = 0: state only.  NC > 0: state and tangent columns g NC .. g NC + NC - 1
// of DF, g = thread index within its state.
template <int NC>
__global__ void __launch_bounds__(PM_BLOCK) __attribute__((amdgpu_waves_per_eu(NC == 0 ? 5 : NC == 1 ? 3 : NC == 2 ? 2 : 1, 8)))
k_pm_flow(RkCoef, const double *in, double *out, double *stm, int64_t n, Model md, double ecc, int steps,
          int64_t nsteps, FlowPlan plan, int64_t unit0)
{
    constexpr int G = NC > 0 ? 4 / NC : 1;   // threads per state
    constexpr int D = 4 + 4 * NC;            // the state, then the thread's columns
    __shared__ double2 s_rn[RK_VALUES];
    const FlowUnit u = flow_unit(plan, unit0 + blockIdx.x, nsteps);
    if (!u.ok) return;
    const int64_t gid = u.block * blockDim.x + threadIdx.x;
    const bool live = gid < n * G;      // every thread of the block fills the stage values
    const int64_t p = live ? gid / G : 0;
    const int g = (int)(gid - (gid / G) * G);
    double z[D];
    if (live) {
        const d4 s = load_d4((u.s0 == 0 ? in : out) + 4 * p);
        z[0] = s.x; z[1] = s.y; z[2] = s.z; z[3] = s.w;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            z[4 + 4 * c + i] = u.s0 > 0 && live ? stm[16 * p + 4 * i + g * NC + c] : (i == g * NC + c) ? 1.0 : 0.0;
    int64_t n_in = u.s0 % steps;
    for (int64_t st0 = u.s0; st0 < u.s1; st0 += RK_CHUNK) {
        const int cnt = u.s1 - st0 < RK_CHUNK ? (int)(u.s1 - st0) : RK_CHUNK;
        __syncthreads();      // the previous chunk's values are no longer read
        fill_stage_chunk(s_rn, threadIdx.x, blockDim.x, n_in, cnt, steps, [&](double t) { return kepler_rho_n(t, ecc); });
        __syncthreads();
        n_in = (n_in + cnt) % steps;
        if (!live) continue;
        for (int jj = 0; jj < cnt; ++jj) {
            const double2 *row = s_rn + jj * RK_SLOTS;
            rk_step<D>(z, step_coef(), [&](int i, double (&s)[D]) { pm_field<NC>(md, row[RK_SLOT[i]].x, row[RK_SLOT[i]].y, s); });
        }
    }
    if (!live) return;
    if (out && g == 0) {
        double2 *o = reinterpret_cast<double2 *>(out + 4 * p);
        o[0] = make_double2(z[0], z[1]);
        o[1] = make_double2(z[2], z[3]);
    }
    if constexpr (NC > 0) {
        // Row-major 4 x 4 per state: stm[16 p + 4 i + j] = d out_i / d in_j.
#pragma unroll
        for (int q = 0; q < NC; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) stm[16 * p + 4 * i + g * NC + q] = z[4 + 4 * q + i];
    }
}

// COLS = 0 or 4: the map, or the map and DF, on pairs of lanes.
template <int COLS>
__global__ void __launch_bounds__(PAIR_BLOCK) k_pm_pair(RkCoef hc, const double *in, double *out, double *stm,
                                                        int64_t n, Model md, double ecc, int steps, int64_t nsteps)
{
    pair_flow<double2, COLS>(
        hc, in, out, stm, n, md, steps, nsteps, [&](double t) { return kepler_rho_n(t, ecc); },
        [](const PairLane &L, const double2 &rn, double (&s)[COLS ? 4 : 2]) { pm_pair<COLS != 0>(L, rn.x, rn.y, s); });
}

int pm_check(const char *who, const double *in_dev, const void *out_dev, int64_t n, const map_params_t *p)
{
    const std::string w(who);
    if (!p || n < 0 || (n > 0 && (!in_dev || !out_dev))) return fail(MS_E_ARG, w + ": bad argument");
    if (p->steps_per_period <= 0) return fail(MS_E_ARG, w + ": steps_per_period must be > 0");
    if (!(p->e >= 0.0 && p->e < 1.0) || !(p->mu >= 0.0 && p->mu <= 1.0))
        return fail(MS_E_ARG, w + ": need 0 <= e < 1 and 0 <= mu <= 1");
    if (!cv_pattern_ok()) return fail(MS_E_ARG, w + ": internal tableau pattern mismatch");
    return MS_OK;
}

template <int COLS>
int pm_pair_launch(const double *in, double *out, double *stm, int64_t n, const map_params_t *p, hipStream_t st)
{
    const int np = p->n_periods < 0 ? -p->n_periods : p->n_periods;
    const int64_t nsteps = (int64_t)p->steps_per_period * np;
    const double h = (p->n_periods < 0 ? -RK_TWO_PI : RK_TWO_PI) / (double)p->steps_per_period;
    hipLaunchKernelGGL(k_pm_pair<COLS>, dim3(pair_blocks(n * (COLS ? COLS : 1))), dim3(PAIR_BLOCK), 0, st, rk_coef(h),
                       in, out, stm, n, Model{p->mu, 1.0 - p->mu}, p->e, p->steps_per_period, nsteps);
    MS_HIP(hipGetLastError());
    return MS_OK;
}

template <int NC>
int pm_launch(const double *in, double *out, double *stm, int64_t n, const map_params_t *p, hipStream_t st)
{
    const int np = p->n_periods < 0 ? -p->n_periods : p->n_periods;
    const int64_t nsteps = (int64_t)p->steps_per_period * np;
    const double h = (p->n_periods < 0 ? -RK_TWO_PI : RK_TWO_PI) / (double)p->steps_per_period;
    constexpr int G = NC > 0 ? 4 / NC : 1;
    const int64_t threads = n * G;
    // The launch counts work-items in 32 bits.
    if (n > (((int64_t)1 << 32) - PM_BLOCK) / G) return fail(MS_E_ARG, "pertbp: too many states for one launch");
    Model md{p->mu, 1.0 - p->mu};
    // between launches the state waits in out (the columns in stm)
    const FlowPlan plan = flow_plan(ceil_div(threads, PM_BLOCK), nsteps, out != nullptr);
    for (int l = 0; l < plan.launches; ++l) {
        hipLaunchKernelGGL(k_pm_flow<NC>, dim3(plan.grid), dim3(PM_BLOCK), 0, st, rk_coef(h), in, out, stm, n, md, p->e,
                           p->steps_per_period, nsteps, plan, (int64_t)l * plan.grid);
        MS_HIP(hipGetLastError());
    }
    return MS_OK;
}

}  // namespace
}  // namespace ms

using namespace ms;

extern "C" int pertbp_map(const double *in_dev, double *out_dev, int64_t n_states, const map_params_t *p,
                          void *stream)
{
    int rc = pm_check("pertbp_map", in_dev, out_dev, n_states, p);
    if (rc || n_states == 0) return rc;
    if (n_states <= PAIR_STATES) return pm_pair_launch<0>(in_dev, out_dev, nullptr, n_states, p, (hipStream_t)stream);
    return pm_launch<0>(in_dev, out_dev, nullptr, n_states, p, (hipStream_t)stream);
}

extern "C" int pertbp_map_stm(const double *in_dev, double *out_dev, double *stm_dev, int64_t n_states,
                              const map_params_t *p, int32_t cols_per_thread, void *stream)
{
    int rc = pm_check("pertbp_map_stm", in_dev, stm_dev, n_states, p);
    if (rc) return rc;
    // default: the fewest instructions a state whose threads leave no SIMD
    // with more than one wave (a second wave doubles the time: a lone wave
    // issues at nine tenths of the rate): a period of 4000 steps takes 6.2 ms
    // on pairs of lanes up to 6,144 states, 8.5 ms at 1 column per thread up
    // to 16,384, 11.1 ms at 2 up to 32,768 and 15.0 ms at 4 up to 65,536;
    // beyond, 4 columns take the least work (60 ms for 262,144 states; 78 at
    // 2, 122 at 1)
    const bool pair = cols_per_thread == 0 && n_states <= PAIR_MATRICES;
    if (cols_per_thread == 0) cols_per_thread = n_states <= 16384 ? 1 : n_states <= 32768 ? 2 : 4;
    if (cols_per_thread != 1 && cols_per_thread != 2 && cols_per_thread != 4)
        return fail(MS_E_ARG, "pertbp_map_stm: cols_per_thread must be 0, 1, 2 or 4");
    if (n_states == 0) return MS_OK;
    if (out_dev && (const void *)out_dev < (const void *)(stm_dev + 16 * n_states) &&
        (const void *)stm_dev < (const void *)(out_dev + 4 * n_states))
        return fail(MS_E_ARG, "pertbp_map_stm: out and stm overlap");
    if ((const void *)in_dev < (const void *)(stm_dev + 16 * n_states) &&
        (const void *)stm_dev < (const void *)(in_dev + 4 * n_states))
        return fail(MS_E_ARG, "pertbp_map_stm: in and stm overlap");
    hipStream_t st = (hipStream_t)stream;
    if (pair) return pm_pair_launch<4>(in_dev, out_dev, stm_dev, n_states, p, st);
    switch (cols_per_thread) {
    case 1: return pm_launch<1>(in_dev, out_dev, stm_dev, n_states, p, st);
    case 2: return pm_launch<2>(in_dev, out_dev, stm_dev, n_states, p, st);
    default: return pm_launch<4>(in_dev, out_dev, stm_dev, n_states, p, st);
    }
}
