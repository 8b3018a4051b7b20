// spectral.hip -- periodic theta operations on the rows of a mesh's vertex
// grid: translation a(theta_i) -> a(theta_i + rho) (the re-alignment of the
// globalised points of Sec. 6.1), theta derivatives (Sec. 7) and
// trigonometric interpolation at arbitrary theta (Sec. 7).
//
// A row is n_theta vertices of one s-value, theta_i = 2 pi i / n_theta, in the
// AoS layout of the mesh (4 doubles per vertex, theta fastest).  Frequencies
// are the signed ones; for even n_theta the coefficient at n_theta / 2 acts
// as the real mode cos(n_theta theta / 2), so real rows stay real.
//
// theta_shift: eight samples per thread, so a workgroup takes one row of 2048
// or several shorter ones.  The two real pairs of a vertex are packed as
// complex sequences z0 = x + i y and z1 = px + i py (the spectral multiplier is
// Hermitian, so it acts on both parts independently) and go through a Stockham
// FFT of radix 8 (a last pass of radix 4 or 2 for the remaining factor) in
// registers; between passes the sequences change places through LDS, one after
// the other in the same 36 KB, so that three workgroups fit a CU and one's
// loads and stores run beside another's butterflies.  The LDS index is padded
// by one slot per 8 so that the strided writes of the first passes spread over
// the banks.  The first forward pass reads the row straight from global memory
// and the last inverse pass writes it back (scaled by 1 / N); the inverse runs
// the radices in reverse order, so the last forward pass, the multiplier
// (j k)^order e^{j k rho} and the first inverse pass work on the same registers
// with no exchange between them.  The twiddle factors come from a table made
// once per (device, N) on the host and read through the caches, each pass's
// own in the order in which its lanes read them; the multiplier's phases from
// phase.hpp.
//
// 4096 rows of 2048, 268 MB read and as many written, 107 us at the rate of a
// large copy (5.0 TB/s): 135 to 141 us from 184 with both sequences in 72 KB,
// a sine and cosine per coefficient and one table of N factors gathered at
// strides (which alone cost 25); with four workgroups on a CU the 128
// registers spill: 167.  The spectrum alone takes 106, from 126.  4096 rows of
// 64, 32 rows to a workgroup: 11 us a call from 43.
//
// theta_interp: the barycentric form of the trigonometric interpolant (no
// transform): with theta = theta_i0 + delta,
//   a(theta) = sin(N delta / 2) / N * sum_i (-1)^d a_i g(delta / 2 + pi d / N),
// d = i0 - i reduced to [-N/2, N/2), g = cot for even N and 1 / sin for odd N.
// The weights come from the row length's cotangents by the addition theorem;
// up to four queries of a row share its samples.
#include <math.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "phase.hpp"

namespace ms {
namespace {

constexpr int SP_THREADS = 256;
constexpr int SP_MAX_LOG2 = 11;   // n_theta <= 2048
constexpr double SP_PI = 3.141592653589793238462643383279502884;
constexpr int SP_RADIX = 8;               // largest radix of a pass

// LDS slot of element i: padded so that the strided writes of the first
// passes (stride R elements) spread over the banks.
MS_D int pslot(int i) { return i + (i >> 3); }
template <int N>
constexpr int padded_size() { return N + (N >> 3); }

// Threads of a row, rows of a workgroup and samples of a thread.
template <int N>
constexpr int row_threads() { return N >= 8 ? N / 8 : 1; }
template <int N>
constexpr int block_rows() { return SP_THREADS / row_threads<N>(); }
template <int N>
constexpr int per_thread() { return N >= 8 ? 8 : N; }

MS_D double2 cmul(double2 a, double2 b)
{
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}

MS_D double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
MS_D double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// Multiplication by -i (forward) or +i (inverse).
template <bool INV>
MS_D double2 mul_mi(double2 b)
{
    return INV ? make_double2(-b.y, b.x) : make_double2(b.y, -b.x);
}

// 4-point DFT of (a, b, c, d) in place.
template <bool INV>
MS_D void dft4(double2 &a, double2 &b, double2 &c, double2 &d)
{
    double2 a0 = cadd(a, c), a1 = csub(a, c);
    double2 b0 = cadd(b, d), b1 = mul_mi<INV>(csub(b, d));
    a = cadd(a0, b0);
    c = csub(a0, b0);
    b = cadd(a1, b1);
    d = csub(a1, b1);
}

// R-point DFT in place (R = 2, 4 or 8); INV selects the sign of the exponent.
template <int R, bool INV>
MS_D void small_dft(double2 *v)
{
    if constexpr (R == 2) {
        double2 a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if constexpr (R == 4) {
        dft4<INV>(v[0], v[1], v[2], v[3]);
    } else {
        // even and odd halves, then X[k] = E[k] + w^k O[k], X[k+4] = E[k] - w^k O[k],
        // w = e^{-+i pi / 4}
        double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
        double2 o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
        dft4<INV>(e0, e1, e2, e3);
        dft4<INV>(o0, o1, o2, o3);
        const double h = 0.70710678118654752440084436210484903928;
        // w o1, w^2 o2 = -+i o2, w^3 o3
        double2 t1 = INV ? make_double2((o1.x - o1.y) * h, (o1.x + o1.y) * h)
                         : make_double2((o1.x + o1.y) * h, (o1.y - o1.x) * h);
        double2 t2 = mul_mi<INV>(o2);
        double2 t3 = INV ? make_double2(-(o3.x + o3.y) * h, (o3.x - o3.y) * h)
                         : make_double2((o3.y - o3.x) * h, -(o3.x + o3.y) * h);
        v[0] = cadd(e0, o0);
        v[4] = csub(e0, o0);
        v[1] = cadd(e1, t1);
        v[5] = csub(e1, t1);
        v[2] = cadd(e2, t2);
        v[6] = csub(e2, t2);
        v[3] = cadd(e3, t3);
        v[7] = csub(e3, t3);
    }
}

// Radix of pass p of the forward transform: SP_RADIX while it fits, then 4
// or 2 for the remaining factor.  The inverse transform runs the same radices
// in reverse order, so that its first pass takes exactly the values the last
// forward pass leaves in each thread's registers.
template <int LOGN>
struct Plan {
    static constexpr int LR = 3;
    static constexpr int FULL = LOGN / LR;
    static constexpr int REST = LOGN % LR;
    static constexpr int NP = FULL + (REST ? 1 : 0);
    static constexpr int radix(int p) { return p < FULL ? SP_RADIX : (REST == 2 ? 4 : 2); }
    // sub-transform length Ns before forward pass p
    static constexpr int ns_fwd(int p) { return p == 0 ? 1 : ns_fwd(p - 1) * radix(p - 1); }
    static constexpr int radix_inv(int p) { return radix(NP - 1 - p); }
    static constexpr int ns_inv(int p) { return p == 0 ? 1 : ns_inv(p - 1) * radix_inv(p - 1); }
    // where a pass's twiddle factors begin in the table: (radix - 1) Ns of
    // each pass but the first, the forward ones before the inverse ones
    static constexpr int tw_fwd(int p) { return p <= 1 ? 0 : tw_fwd(p - 1) + (radix(p - 1) - 1) * ns_fwd(p - 1); }
    static constexpr int tw_inv(int p) { return p <= 1 ? tw_fwd(NP) : tw_inv(p - 1) + (radix_inv(p - 1) - 1) * ns_inv(p - 1); }
};

// The registers of a thread: both sequences.  Pass of radix R: butterfly q of
// the thread, j = t + q row_threads, holds element r of it in v[s][q R + r].
template <int N>
using Regs = double2[2][per_thread<N>()];

// Stockham pass of radix R, sub-transform length Ns, over both sequences in
// registers.  Butterfly j holds element j + r N/R (r = 0..R-1), twiddles it by
// e^{-+2 pi i r (j mod Ns) / (Ns R)} (entry (r - 1) Ns + (j mod Ns) of the pass's
// table, conjugated for the inverse) and transforms.
template <bool FEW, int N, int R, int Ns, bool INV>
MS_D void butterflies(Regs<N> &v, int t, const double2 *__restrict__ tw)
{
    constexpr int T = row_threads<N>();
#pragma unroll
    for (int q = 0; q < per_thread<N>() / R; ++q) {
        double2 w[R];
        bool turn = false;
        if constexpr (Ns > 1) {
            const int k = (t + q * T) % Ns;
            // (a factor of 1 is left out, and with it what 0 times an infinite
            // part, or one that is no number, would put into the other)
            turn = INV || k != 0;
#pragma unroll
            for (int r = 1; r < R; ++r) {
                w[r] = tw[(r - 1) * Ns + k];
                if (INV) w[r].y = -w[r].y;
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (turn) {
#pragma unroll
                for (int r = 1; r < R; ++r) v[s][q * R + r] = cmul(v[s][q * R + r], w[r]);
            }
            small_dft<R, INV>(v[s] + q * R);
            // one sequence's butterfly at a time in the registers
            if constexpr (!FEW) __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Element that a pass of radix R and length Ns leaves in register i, where
// butterfly j's are (j / Ns) Ns R + (j mod Ns) + r Ns.
template <int N, int R, int Ns>
MS_D int element(int t, int i)
{
    const int j = t + i / R * row_threads<N>();
    return (j / Ns) * Ns * R + j % Ns + i % R * Ns;
}

// From the places of a pass (R, Ns) to the inputs of the next, of radix R2.
// FEW: both sequences at once, z holds room for two; the threads beyond the
// row's have no part in it.
template <bool FEW, int N, int R, int Ns, int R2>
MS_D void exchange(Regs<N> &v, int t, double2 *z)
{
    constexpr int E = per_thread<N>(), T = row_threads<N>(), STEP = FEW ? padded_size<N>() : 0;
    const bool on = !FEW || (int)threadIdx.x < T;
    auto put = [&](int s) {
        if (!on) return;
#pragma unroll
        for (int i = 0; i < E; ++i) z[s * STEP + pslot(element<N, R, Ns>(t, i))] = v[s][i];
    };
    auto get = [&](int s) {
        if (!on) return;
#pragma unroll
        for (int i = 0; i < E; ++i) v[s][i] = z[s * STEP + pslot(t + i / R2 * T + i % R2 * (N / R2))];
    };
    put(0);
    if constexpr (FEW) put(1);
    __syncthreads();
    get(0);
    if constexpr (!FEW) {
        __syncthreads();
        put(1);
        __syncthreads();
    }
    get(1);
}

template <int N>
MS_D double frequency(int k) { return 2 * k > N ? (double)(k - N) : (double)k; }

template <int N>
MS_D double2 row_phase(int k, double rho)
{
    double sn, cs;
    sincos(frequency<N>(k) * rho, &sn, &cs);
    return make_double2(cs, sn);
}

// The multiplier at the coefficients that the last forward pass (radix R,
// Ns = N / R: coefficient j + r N/R) leaves in the registers.  z: the row's
// LDS, where the thread's own inputs of that pass are free.  FEW: the phases
// are in z, one of each coefficient.
template <bool FEW, int N, int R>
MS_D void multiply(Regs<N> &v, int t, const PhaseTable *ph, double rho, int order, double2 *z)
{
    constexpr int E = per_thread<N>(), T = row_threads<N>();
    auto coef = [&](int i) { return t + i / R * T + i % R * (N / R); };
    const bool near = !FEW && fabs(rho) * (0.5 * N) < PH_MAX;
    if (!FEW && !near) {
#pragma nounroll
        for (int i = 0; i < E; ++i) z[pslot(coef(i))] = row_phase<N>(coef(i), rho);
    }
#pragma unroll
    for (int i = 0; i < E; ++i) {
        const int k = coef(i);
        const double ks = frequency<N>(k);
        double2 m;
        if (near) phase_near(*ph, ks * rho, m.x, m.y);
        else m = z[FEW ? k : pslot(k)];
        if (order == 1) m = make_double2(-ks * m.y, ks * m.x);
        else if (order == 2) m = make_double2(-ks * ks * m.x, -ks * ks * m.y);
        // the cosine mode: Re[(j N/2)^order e^{j (N/2) rho}]
        if (2 * k == N) m.y = 0.0;
        v[0][i] = cmul(v[0][i], m);
        v[1][i] = cmul(v[1][i], m);
        // (eight phases at a time do not fit the registers)
        if constexpr (!FEW) __builtin_amdgcn_sched_barrier(0);
    }
}

// Forward passes P.. up to the last.
template <bool FEW, int LOGN, int P>
MS_D void forward_passes(Regs<1 << LOGN> &v, int t, const double2 *tw, double2 *z)
{
    using PL = Plan<LOGN>;
    constexpr int N = 1 << LOGN, R = PL::radix(P), NS = PL::ns_fwd(P), TW = PL::tw_fwd(P);
    butterflies<FEW, N, R, NS, false>(v, t, tw + TW);
    if constexpr (P < PL::NP - 1) {
        if constexpr (P > 0) __syncthreads();
        exchange<FEW, N, R, NS, PL::radix(P + 1)>(v, t, z);
        forward_passes<FEW, LOGN, P + 1>(v, t, tw, z);
    }
}

// Inverse passes P.. up to the last (the inputs in place).
template <bool FEW, int LOGN, int P>
MS_D void inverse_passes(Regs<1 << LOGN> &v, int t, const double2 *tw, double2 *z)
{
    using PL = Plan<LOGN>;
    constexpr int N = 1 << LOGN, R = PL::radix_inv(P), NS = PL::ns_inv(P), TW = PL::tw_inv(P);
    butterflies<FEW, N, R, NS, true>(v, t, tw + TW);
    if constexpr (P < PL::NP - 1) {
        __syncthreads();
        exchange<FEW, N, R, NS, PL::radix_inv(P + 1)>(v, t, z);
        inverse_passes<FEW, LOGN, P + 1>(v, t, tw, z);
    }
}

// A row's samples as the inputs of the first pass (radix R).
template <int N, int R>
MS_D void load_row(Regs<N> &v, int t, const double *src, bool live)
{
#pragma unroll
    for (int i = 0; i < per_thread<N>(); ++i) {
        const int e = t + i / R * row_threads<N>() + i % R * (N / R);
        const d4 w = live ? load_d4(src + 4 * e) : d4{0.0, 0.0, 0.0, 0.0};
        v[0][i] = make_double2(w.x, w.y);
        v[1][i] = make_double2(w.z, w.w);
    }
}

// The outputs of the last pass (radix R, Ns), scaled by 1 / N.
template <int N, int R, int Ns>
MS_D void store_row(const Regs<N> &v, int t, double *dst)
{
    const double inv = 1.0 / (double)N;
#pragma unroll
    for (int i = 0; i < per_thread<N>(); ++i) {
        double2 *o = reinterpret_cast<double2 *>(dst + 4 * element<N, R, Ns>(t, i));
        o[0] = make_double2(v[0][i].x * inv, v[0][i].y * inv);
        o[1] = make_double2(v[1][i].x * inv, v[1][i].y * inv);
    }
}

// A workgroup's rows and threads, and the LDS of a row.  FEW, for the few rows
// that do not fill the chip, where a row's chain of waits is the time: one row
// a workgroup, both sequences side by side in LDS, which halves the waits
// between the passes, and up to 256 threads, of which those beyond the row's
// only take their share of the phases' sines and cosines.
template <int N, bool FEW>
constexpr int group_rows() { return FEW ? 1 : block_rows<N>(); }
template <int N, bool FEW>
constexpr int group_threads() { return !FEW || N >= 512 ? SP_THREADS : N >= 128 ? N / 2 : 64; }
template <int N, bool FEW>
constexpr int row_slots() { return (FEW ? 2 : 1) * padded_size<N>(); }

// row_map (optional): output row of each input row; a negative entry drops
// the row.
template <int LOGN, bool FEW>
__global__ void __launch_bounds__(SP_THREADS) __attribute__((amdgpu_waves_per_eu(FEW ? 1 : 3)))
k_theta_shift(const double *in, double *out, const double2 *__restrict__ tw, const double *rho_dev, double rho, int order,
              const int64_t *row_map, int64_t n_rows)
{
    using PL = Plan<LOGN>;
    constexpr int N = 1 << LOGN, T = row_threads<N>(), RM = PL::radix(PL::NP - 1);
    __shared__ double2 s_z[group_rows<N, FEW>()][row_slots<N, FEW>()];
    const int t = threadIdx.x % T, own = FEW ? 0 : threadIdx.x / T;
    const int64_t row = (int64_t)blockIdx.x * group_rows<N, FEW>() + own;
    double2 *z = s_z[own];
    const int64_t orow = row >= n_rows ? -1 : row_map ? row_map[row] : row;
    const bool live = orow >= 0 && (!FEW || (int)threadIdx.x < T);
    Regs<N> v;
    const double r = orow >= 0 ? (rho_dev ? rho_dev[row] : rho) : 0.0;
    if constexpr (FEW) {
        __shared__ double2 s_ph[N];
        load_row<N, PL::radix(0)>(v, t, in + row * (int64_t)N * 4, live);
        for (int k = threadIdx.x; k < N; k += group_threads<N, FEW>()) s_ph[k] = row_phase<N>(k, r);
        forward_passes<FEW, LOGN, 0>(v, t, tw, z);
        if constexpr (PL::NP == 1) __syncthreads();
        multiply<FEW, N, RM>(v, t, nullptr, r, order, s_ph);
    } else {
        __shared__ PhaseTable s_ph;
        phase_table(s_ph);
        load_row<N, PL::radix(0)>(v, t, in + row * (int64_t)N * 4, live);
        forward_passes<FEW, LOGN, 0>(v, t, tw, z);
        if constexpr (PL::NP == 1) __syncthreads();      // the phases' table
        multiply<FEW, N, RM>(v, t, &s_ph, r, order, z);
    }
    inverse_passes<FEW, LOGN, 0>(v, t, tw, z);
    if (live) store_row<N, PL::radix_inv(PL::NP - 1), PL::ns_inv(PL::NP - 1)>(v, t, out + orow * (int64_t)N * 4);
}

// Forward transform only: out(r, j) = (Z0(j), Z1(j)) / N in natural order,
// four doubles per frequency (Re Z0, Im Z0, Re Z1, Im Z1), the layout of the
// input rows.
template <int LOGN, bool FEW>
__global__ void __launch_bounds__(SP_THREADS) __attribute__((amdgpu_waves_per_eu(FEW ? 1 : 4)))
k_theta_spectrum(const double *in, double *out, const double2 *__restrict__ tw, int64_t n_rows)
{
    using PL = Plan<LOGN>;
    constexpr int N = 1 << LOGN, T = row_threads<N>();
    __shared__ double2 s_z[group_rows<N, FEW>()][row_slots<N, FEW>()];
    const int t = threadIdx.x % T;
    const int64_t row = (int64_t)blockIdx.x * group_rows<N, FEW>() + threadIdx.x / T;
    Regs<N> v;
    load_row<N, PL::radix(0)>(v, t, in + row * (int64_t)N * 4, row < n_rows);
    forward_passes<FEW, LOGN, 0>(v, t, tw, s_z[threadIdx.x / T]);
    if (row < n_rows) store_row<N, PL::radix(PL::NP - 1), PL::ns_fwd(PL::NP - 1)>(v, t, out + row * (int64_t)N * 4);
}

// ------------------------------------------------------------- interpolation

constexpr int IP_BLOCK = 1024;
constexpr int IP_MAX_N = 2048;            // the cotangents of a row length up to this lie in LDS
constexpr int IP_MAX_Q = 256;             // queries of a block (grouped: its share)
constexpr int IP_LIST = 3 * IP_MAX_Q;
constexpr int IP_SLICE = 1 << 16;         // queries grouped together
constexpr int IP_MAX_BINS = 8192;
constexpr uint32_t IP_START = 0x1ffff;    // a bin's word: start (17 bits; all ones: too large), rank from bit 17

// One query by the barycentric form with a sine and cosine per sample, by
// one wave: any offset delta from sample i0, any N.
MS_D void interp_one(const double *a, int N, int64_t i0, double delta, double *o)
{
    const int lane = threadIdx.x % 64;
    const bool even = (N & 1) == 0;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = lane; i < N; i += 64) {
        int64_t d = i0 - i;                 // in (-N, N); the kernel is N-periodic in d
        if (2 * d >= N) d -= N;
        else if (2 * d < -N) d += N;
        double sn, cs;
        sincos(0.5 * delta + SP_PI * (double)d / (double)N, &sn, &cs);
        double w = even ? cs / sn : 1.0 / sn;
        if (d & 1) w = -w;
        d4 v = load_d4(a + 4 * (int64_t)i);
        acc[0] += w * v.x;
        acc[1] += w * v.y;
        acc[2] += w * v.z;
        acc[3] += w * v.w;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) acc[c] += __shfl_xor(acc[c], off);
    if (lane < 4) {
        const double f = sin(0.5 * (double)N * delta) / (double)N;
        double s = lane == 0 ? acc[0] : lane == 1 ? acc[1] : lane == 2 ? acc[2] : acc[3];
        o[lane] = f * s;
    }
}

// The same, a wave per query: where the tables of k_theta_interp do not fit
// or do not pay.
__global__ void __launch_bounds__(256) k_theta_interp_plain(const double *in, int N, int64_t n_rows,
                                                           const int64_t *rows, const double *theta, int64_t nq,
                                                           double *out)
{
    const int64_t q = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    const int lane = threadIdx.x % 64;
    if (q >= nq) return;   // whole waves
    const int64_t row = rows[q];
    const double th = theta[q];
    double *o = out + 4 * q;
    const double step = 2.0 * SP_PI / (double)N;
    const double i0f = rint(th / step);
    if (row < 0 || row >= n_rows || !isfinite(th) || !isfinite(i0f)) {
        if (lane < 4) o[lane] = NAN;
        return;
    }
    const double *a = in + row * (int64_t)N * 4;
    const double delta = th - i0f * step;
    int64_t i0 = (int64_t)fmod(i0f, (double)N);   // exact, in (-N, N)
    if (i0 < 0) i0 += N;
    if (fabs(delta) < 1e-200) {
        if (lane < 4) o[lane] = a[4 * i0 + lane];
        return;
    }
    interp_one(a, N, i0, delta, o);
}

MS_D double uni(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// The queries of a block in LDS: up to LEN.  (Ungrouped, 9 KB for 256 instead of
// 28 for three shares: beside the table of an odd 1023 or an even 2048 a fourth
// block fits a CU, and a third beside an odd 2047; 4096 queries of one row 16.1,
// 15.4 and 26.2 us for 19.9, 18.1 and 26.8.)
template <int LEN>
struct IpList {
    double t[LEN];       // tan(delta / 2)
    double f[LEN];       // factor of the sum: (-1)^i0 sin(N delta / 2) / N (odd N: / cos(delta / 2))
    int64_t row[LEN];    // -1: nothing to do
    int32_t i0[LEN];     // -1: |theta| so large that delta is not below a step
    uint32_t q[LEN];     // query, from the slice's first; ~0: none
    uint32_t tile[LEN];  // first entry, entries << 16 (0: one with i0 = -1)
    uint32_t n_tiles, unsorted;
};

// n / d for d of ordinary size: the hardware reciprocal (about 23 correct
// bits) and one cubic correction of the quotient.  Every weight has its own:
// with one reciprocal for four (138 us for 65536 queries in 4096 rows of 2048
// samples, 143 so) a query's last bits depend on the queries beside it, and so on the
// order in which the grouping takes them.
MS_D double quotient(double n, double d)
{
    const double y = __builtin_amdgcn_rcp(d);
    const double e = fma(-d, y, 1.0), t = n * y;
    return fma(t, fma(e, e, e), t);
}

// QT queries of one row, U samples per lane and step (QT U = 4): with
// t = tan(delta / 2) and d = i0 - i,
//   cot(delta / 2 + pi d / N) = (cot(pi d / N) - t) / (1 + t cot(pi d / N))
//   1 / sin(delta / 2 + pi d / N) = 1 / (sin(pi d / N) (1 + t cot(pi d / N)) cos(delta / 2)),
// where |t cot| < 3/4 but for d = 0, whose weight is 1 / t.  Entry x of the
// table is cot(-pi x / N), 0 < x < N, with 1 / sin(pi x / N) for odd N: a
// lane's samples below i0 have x = i - i0 + N, those above x = i - i0, where
// 1 / sin(pi d / N) is minus the entry's.  So the lane's sums change sign
// there (odd N), and the sum's sign in the end.  The two steps in which lanes
// pass i0, and the last one of a length that is no multiple of the step, go
// sample by sample.  (-1)^d is (-1)^i0 for the query times (-1)^i, a sign per
// lane: the steps are of 64 samples.
template <bool ODD, int QT, class List>
MS_D void interp_tile(const List &s, int e0, int len, const double *tab, const double *__restrict__ in, int N,
                      double *out)
{
    constexpr int U = 4 / QT;
    const int lane = threadIdx.x % 64;
    double t[QT];
    int i0[QT], x[QT];
    uint64_t fix = 0;
#pragma unroll
    for (int q = 0; q < QT; ++q) {
        const int e = e0 + (q < len ? q : len - 1);
        t[q] = uni(s.t[e]);
        i0[q] = __builtin_amdgcn_readfirstlane(s.i0[e]);
        fix |= 1ull << (i0[q] / (64 * U)) | 1ull << ((i0[q] + 63) / (64 * U));
        x[q] = lane - i0[q] + N;
    }
    const uint64_t row = (uint64_t)s.row[e0];
    const double *a = in + 4 * (int64_t)((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)row) |
                                         (uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(row >> 32)) << 32) * N;
    double acc[4 * QT] = {};
    double num[4], den[4];
    auto entry = [&](int j, int q, int k) {
        if constexpr (ODD) {
            const double2 c = reinterpret_cast<const double2 *>(tab)[k];
            den[j] = fma(t[q], c.x, 1.0);
            num[j] = c.y;
        } else {
            const double c = tab[k];
            den[j] = fma(t[q], c, 1.0);
            num[j] = c - t[q];
        }
    };
    auto load = [&](d4 *v, int k) {
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = load_d4(a + 256 * (k + u) + 4 * lane);
    };
    auto add = [&](const d4 *v) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = j / U, u = j % U;
            acc[4 * q] = fma(num[j], v[u].x, acc[4 * q]);
            acc[4 * q + 1] = fma(num[j], v[u].y, acc[4 * q + 1]);
            acc[4 * q + 2] = fma(num[j], v[u].z, acc[4 * q + 2]);
            acc[4 * q + 3] = fma(num[j], v[u].w, acc[4 * q + 3]);
        }
    };
    const int steps = (N + 64 * U - 1) / (64 * U), full = N / (64 * U);
    if (full < steps) fix |= 1ull << full;
    int k = 0;      // step: samples 64 U k + 64 u + lane
    while (k < steps) {
        const uint64_t ahead = fix >> k;
        const int stop = ahead ? min(k + (int)__builtin_ctzll(ahead), steps) : steps;
        if (k < stop) {
            d4 v[U];
            load(v, U * k);
            for (; k < stop; ++k) {
                d4 w[U];
                load(w, U * (k + 1 < stop ? k + 1 : k));       // the next step's, in flight over this one
#pragma unroll
                for (int j = 0; j < 4; ++j) entry(j, j / U, x[j / U] + 64 * (j % U));
#pragma unroll
                for (int j = 0; j < 4; ++j) num[j] = quotient(num[j], den[j]);
                add(v);
#pragma unroll
                for (int q = 0; q < QT; ++q) x[q] += 64 * U;
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = w[u];
            }
        }
        if (k >= steps) break;
        const int i_first = lane + 64 * U * k, i_last = i_first + 64 * (U - 1);
        d4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            v[u] = i_first + 64 * u < N ? load_d4(a + 4 * (i_first + 64 * u)) : d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = i_first + 64 * (j % U), d = i - i0[j / U];
            entry(j, j / U, i >= N ? 0 : d < 0 ? d + N : d);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = j / U, i = i_first + 64 * (j % U);
            num[j] = i == i0[q] ? (ODD ? -1.0 : 1.0) / t[q] : quotient(num[j], den[j]);
            if (ODD && i < i0[q] && i_last >= i0[q]) num[j] = -num[j];
        }
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            // the lane passes i0 in this step
            if (ODD && i_first - 64 < i0[q] && i_last >= i0[q])
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[4 * q + c] = -acc[4 * q + c];
            x[q] = i_last + 64 - i0[q] + (i_last < i0[q] ? N : 0);
        }
        add(v);
        ++k;
    }
    // a row may end before a lane passes i0
    if constexpr (ODD)
#pragma unroll
        for (int q = 0; q < QT; ++q)
            if (lane + 64 * (U * steps - 1) < i0[q])
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[4 * q + c] = -acc[4 * q + c];
    // the lanes' sums: value j of 4 QT ends up on the lanes whose top bits are j
#pragma unroll
    for (int n = 2 * QT, off = 32; n >= 1; n >>= 1, off >>= 1) {
        const bool hi = (lane & off) != 0;
#pragma unroll
        for (int j = 0; j < n; ++j) {
            const double mine = hi ? acc[j + n] : acc[j], send = hi ? acc[j] : acc[j + n];
            acc[j] = mine + __shfl_xor(send, off);
        }
    }
    constexpr int SHARE = 64 / (4 * QT);
#pragma unroll
    for (int off = SHARE / 2; off > 1; off >>= 1) acc[0] += __shfl_xor(acc[0], off);
    const double other = __shfl_xor(acc[0], 1);
    if (lane % SHARE != 0) return;
    const int j = lane / SHARE, q = j / 4;
    if (q < len) out[4 * (int64_t)s.q[e0 + q] + j % 4] = s.f[e0 + q] * (acc[0] - other);
}

struct InterpArgs {
    const double *in;
    const int64_t *rows;
    const double *theta;
    double *out;
    int64_t n_rows, nq;
    int N;
    int share;               // queries of a block
    int slice, per_slice;    // grouped: queries of a slice, blocks of a slice
    int bins, shift;         // grouped: bins of 2^shift rows
};

// A block takes `share` queries, keeps the row length's cotangents in LDS
// and gives its waves tiles of up to four queries of the same row, whose
// samples are then loaded once for all four.  GROUPED (many queries per row,
// in any order): a slice of up to 65536 queries is dealt to its blocks by
// rows.  Every block counts the slice's queries per bin of rows in LDS (one
// scan of the row indices), takes the bins that start in its share of the
// sorted order and, in a second scan, their queries.  A bin of more than a
// share is left out of that order: its queries go to the blocks by their
// place in the slice, so that a block has at most three shares whatever the
// rows are.
//
// 65536 queries in 4096 rows of 2048 samples: 143 us, from 555 with a wave
// per query and a sine, cosine and division per sample (about 100 FP64
// instructions, now 12 and a reciprocal), which read the rows 16 times.
// Without the grouping 614: the rows' bytes bound it.  Now 25 us go to the
// grouping, 8 to the table and the offsets, the rest to the sums, at about
// half the FP64 rate.  Four
// queries in flight with their next samples take the 128 registers of four
// waves per SIMD; a wave's two scalar steps cost as much as four others.
template <bool ODD, bool GROUPED>
__global__ void __launch_bounds__(IP_BLOCK) k_theta_interp(InterpArgs g)
{
    extern __shared__ double s_dyn[];     // the bins, then the cotangents
    __shared__ IpList<GROUPED ? IP_LIST : IP_MAX_Q> s;
    const int tid = threadIdx.x, nt = GROUPED ? IP_BLOCK : (int)blockDim.x, lane = tid % 64, wv = tid / 64;
    const int N = g.N;
    int64_t q0;
    int n_list;
    if constexpr (GROUPED) {
        __shared__ uint32_t s_wave[IP_BLOCK / 64], s_lo, s_hi;
        if (tid == 0) {
            s_lo = ~0u;
            s_hi = 0;
        }
        uint32_t *bin = reinterpret_cast<uint32_t *>(s_dyn);
        const int b = (int)(blockIdx.x % (unsigned)g.per_slice);
        q0 = (int64_t)(blockIdx.x / (unsigned)g.per_slice) * g.slice;
        const int n = (int)(g.nq - q0 < g.slice ? g.nq - q0 : g.slice);
        const int64_t *rows = g.rows + q0;
        auto bin_of = [&](int64_t r) { return r < 0 || r >= g.n_rows ? 0u : (uint32_t)(r >> g.shift); };
        for (int i = tid; i < g.bins; i += IP_BLOCK) bin[i] = 0;
        for (int i = tid; i < 3 * g.share; i += IP_BLOCK) s.q[i] = ~0u;
        __syncthreads();
        // the thread's row bins stay in registers, two in each
        constexpr int PER = IP_SLICE / IP_BLOCK;
        uint32_t mine[PER / 2];
#pragma unroll
        for (int c = 0; c < PER; c += 16) {
            if (c * IP_BLOCK >= n) break;
            int64_t r[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int i = tid + (c + u) * IP_BLOCK;
                r[u] = i < n ? rows[i] : 0;
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const uint32_t h = bin_of(r[u]);
                const bool in = tid + (c + u) * IP_BLOCK < n;
                // one row's queries one after another: one add for the wave
                if (ballot(in && h == (uint32_t)__builtin_amdgcn_readfirstlane(h)) == ~0ull) {
                    if (lane == 0) atomicAdd(&bin[h], 64u);
                } else if (in) {
                    atomicAdd(&bin[h], 1u);
                }
                mine[(c + u) / 2] = (u & 1) ? mine[(c + u) / 2] | h << 16 : h;
            }
        }
        __syncthreads();
        // starts of the bins in the sorted order
        const int per = (g.bins + IP_BLOCK - 1) / IP_BLOCK;
        const int b0 = tid * per, b1 = b0 + per < g.bins ? b0 + per : g.bins;
        uint32_t sum = 0;
        for (int i = b0; i < b1; ++i) sum += bin[i] <= (uint32_t)g.share ? bin[i] : 0;
        uint32_t inc = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(inc, o);
            if (lane >= o) inc += y;
        }
        if (lane == 63) s_wave[wv] = inc;
        __syncthreads();
        uint32_t at = inc - sum;
        for (int w = 0; w < wv; ++w) at += s_wave[w];
        // the block's bins: those that start in its share of the order
        const uint32_t first = (uint32_t)(b * g.share);
        uint32_t lo = ~0u, hi = 0;
        for (int i = b0; i < b1; ++i) {
            const uint32_t c = bin[i];
            const bool fits = c <= (uint32_t)g.share;
            if (fits && c && at - first < (uint32_t)g.share) {
                lo = min(lo, (uint32_t)i);
                hi = (uint32_t)i + 1;
            }
            bin[i] = fits ? at : IP_START;
            at += fits ? c : 0;
        }
        if (hi) {
            atomicMin(&s_lo, lo);
            atomicMax(&s_hi, hi);
        }
        __syncthreads();
        lo = s_lo;
        hi = s_hi;
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            const int i = tid + c * IP_BLOCK;
            if (c * IP_BLOCK >= n) break;
            if (i >= n) continue;
            const uint32_t h = mine[c / 2] >> (c & 1 ? 16 : 0) & 0xffff;
            const bool window = (uint32_t)i - first < (uint32_t)g.share;
            if (!window && h - lo >= hi - lo) continue;
            const uint32_t start = bin[h] & IP_START;
            if (start == IP_START) {
                if (window) s.q[2 * g.share + (uint32_t)i - first] = (uint32_t)i;
            } else if (start - first < (uint32_t)g.share) {
                const uint32_t rank = atomicAdd(&bin[h], IP_START + 1) >> 17;
                s.q[start - first + rank] = (uint32_t)i;
            }
        }
        n_list = 3 * g.share;
        __syncthreads();
    } else {
        q0 = (int64_t)blockIdx.x * g.share;
        n_list = (int)(g.nq - q0 < g.share ? g.nq - q0 : g.share);
    }
    if (tid == 0) s.n_tiles = s.unsorted = 0;
    // A share may hold several queries of a row, but not side by side: those
    // by their place in the slice, and a direct block's if the rows are few.
    if (GROUPED || g.n_rows <= g.share) {
        const int e0 = GROUPED ? 2 * g.share : 0, ne = n_list - e0;
        for (int e = tid; e < ne; e += nt) {
            if constexpr (!GROUPED) s.q[e] = (uint32_t)e;
            s.row[e0 + e] = s.q[e0 + e] == ~0u ? INT64_MAX : g.rows[q0 + s.q[e0 + e]];
            s.tile[e] = 0;
        }
        __syncthreads();
        const int e = tid % g.share, part = tid / g.share, parts = nt / g.share;
        if (tid < ne && tid > 0 && s.row[e0 + tid] < s.row[e0 + tid - 1]) s.unsorted = 1;
        __syncthreads();
        if (s.unsorted) {
            if (e < ne && part < parts) {
                const int64_t row = s.row[e0 + e];
                uint32_t r = 0;
                for (int j = part; j < ne; j += parts) {
                    const int64_t o = s.row[e0 + j];
                    r += o < row || (o == row && j < e);
                }
                atomicAdd(&s.tile[e], r);
            }
            uint32_t q = 0;
            if (tid < ne) q = s.q[e0 + tid];
            __syncthreads();
            if (tid < ne) s.q[e0 + s.tile[tid]] = q;
        }
        __syncthreads();
    } else {
        for (int e = tid; e < n_list; e += nt) s.q[e] = (uint32_t)e;
        __syncthreads();
    }
    for (int x = tid; x <= N / 2; x += nt) {
        // entries x and N - x: cot(-pi x / N) and minus that (and 1 / sin(pi x / N) twice)
        double sn = 1.0, cs = 0.0;
        if (x) sincospi((double)x / (double)N, &sn, &cs);
        const int y = x ? N - x : 0;
        if constexpr (ODD) {
            reinterpret_cast<double2 *>(s_dyn)[x] = make_double2(-cs / sn, 1.0 / sn);
            reinterpret_cast<double2 *>(s_dyn)[y] = make_double2(cs / sn, 1.0 / sn);
        } else {
            s_dyn[x] = -cs / sn;
            s_dyn[y] = cs / sn;
        }
    }
    // the queries: offsets from their nearest samples
    const double step = 2.0 * SP_PI / (double)N;
    for (int e = tid; e < n_list; e += nt) {
        int64_t row = -1;
        if (s.q[e] != ~0u) {
            const int64_t q = q0 + s.q[e];
            row = g.rows[q];
            const double th = g.theta[q];
            const double i0f = rint(th / step);
            double *o = g.out + 4 * q;
            if (row < 0 || row >= g.n_rows || !isfinite(th) || !isfinite(i0f)) {
                // no such row, or |theta| beyond any meaningful angle
                row = -1;
                o[0] = o[1] = o[2] = o[3] = NAN;
            } else {
                const double delta = th - i0f * step;
                int32_t i0 = fabs(i0f) < 1e9 ? (int32_t)i0f % N : (int32_t)fmod(i0f, (double)N);
                if (i0 < 0) i0 += N;
                if (fabs(delta) < 1e-200) {
                    const double *a = g.in + (row * (int64_t)N + i0) * 4;
#pragma unroll
                    for (int c = 0; c < 4; ++c) o[c] = a[c];
                    row = -1;
                } else {
                    double sn, cs;
                    sincos(0.5 * delta, &sn, &cs);
                    s.t[e] = sn / cs;
                    double f = sin(0.5 * (double)N * delta) / (double)N;
                    if (ODD) f /= cs;
                    s.f[e] = ((i0 & 1) != 0) != ODD ? -f : f;      // (odd N: see interp_tile)
                    s.i0[e] = fabs(delta) < 0.75 * step ? i0 : -1;
                }
            }
        }
        s.row[e] = row;
    }
    __syncthreads();
    // tiles: up to four neighbours of the same row, fewer where a tile for
    // each of the block's waves takes that
    const int waves = nt / 64, more = GROUPED || n_list >= 4 * waves ? 3 : n_list >= 2 * waves ? 1 : 0;
    for (int e = tid; e - lane < n_list; e += nt) {
        const int64_t row = e < n_list ? s.row[e] : -1;
        const bool lone = row >= 0 && s.i0[e] < 0;
        const bool head = lane == 0 || row < 0 || lone || s.row[e - 1] != row || s.i0[e - 1] < 0;
        const uint64_t heads = ballot(head);
        const uint64_t below = heads & (~0ull >> (63 - lane));
        const int at = lane - (63 - __builtin_clzll(below));
        const bool start = row >= 0 && (at & more) == 0;
        const uint64_t after = lane == 63 ? 0 : heads >> (lane + 1);
        const int run = after ? 1 + __builtin_ctzll(after) : 64 - lane;
        const uint64_t starts = ballot(start);
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&s.n_tiles, (uint32_t)__builtin_popcountll(starts));
        base = __builtin_amdgcn_readfirstlane(base);
        if (start)
            s.tile[base + __builtin_popcountll(starts & ~(~0ull << lane))] =
                (uint32_t)e | (lone ? 0u : (uint32_t)(run <= more ? run : more + 1) << 16);
    }
    __syncthreads();
    double *out = g.out + 4 * q0;
    const int n_tiles = (int)s.n_tiles;
    for (int k = wv; k < n_tiles; k += waves) {
        const uint32_t w = __builtin_amdgcn_readfirstlane(s.tile[k]);
        const int e = (int)(w & 0xffff), len = (int)(w >> 16);
        if (len > 2) interp_tile<ODD, 4>(s, e, len, s_dyn, g.in, N, out);
        else if (len == 2) interp_tile<ODD, 2>(s, e, len, s_dyn, g.in, N, out);
        else if (len == 1) interp_tile<ODD, 1>(s, e, len, s_dyn, g.in, N, out);
        else {
            const double th = g.theta[q0 + s.q[e]], i0f = rint(th / step);
            int64_t i0 = (int64_t)fmod(i0f, (double)N);
            if (i0 < 0) i0 += N;
            interp_one(g.in + s.row[e] * (int64_t)N * 4, N, i0, th - i0f * step, out + 4 * (int64_t)s.q[e]);
        }
    }
}

// The twiddle factors of all passes (Plan) per (device, N), kept for the life
// of the process (11 lengths, at most 56 KB each).  2 m / N is exact for a
// power of two N, so each entry is the rounded cosine and sine of one rounded
// argument.
template <int LOGN>
std::vector<double2> make_twiddles()
{
    using PL = Plan<LOGN>;
    constexpr int N = 1 << LOGN;
    std::vector<double2> w;
    auto add = [&](int R, int Ns) {
        for (int r = 1; r < R; ++r)
            for (int k = 0; k < Ns; ++k) {
                const double a = SP_PI * (2.0 * (double)(r * k * (N / (Ns * R))) / (double)N);
                w.push_back(make_double2(cos(a), -sin(a)));
            }
    };
    for (int p = 1; p < PL::NP; ++p) add(PL::radix(p), PL::ns_fwd(p));
    for (int p = 1; p < PL::NP; ++p) add(PL::radix_inv(p), PL::ns_inv(p));
    if (w.empty()) w.push_back(make_double2(1.0, 0.0));
    return w;
}

std::mutex g_tw_mu;
std::map<std::pair<int, int>, double2 *> g_tw;

template <int LOGN>
int twiddles(const double2 **out)
{
    int dev = 0;
    MS_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_tw_mu);
    auto key = std::make_pair(dev, LOGN);
    auto it = g_tw.find(key);
    if (it != g_tw.end()) { *out = it->second; return MS_OK; }
    const std::vector<double2> w = make_twiddles<LOGN>();
    double2 *d = nullptr;
    MS_HIP(hipMalloc(&d, w.size() * sizeof(double2)));
    hipError_t er = hipMemcpy(d, w.data(), w.size() * sizeof(double2), hipMemcpyHostToDevice);
    if (er != hipSuccess) { (void)hipFree(d); return hip_fail(er, "copy twiddle table"); }
    g_tw[key] = d;
    *out = d;
    return MS_OK;
}

struct ShiftArgs {
    const double *in;
    double *out;
    const double *rho_dev;
    double rho;
    int order;
    const int64_t *row_map;
    int64_t n_rows;
};

template <int LOGN, bool FEW>
int launch_shift(const ShiftArgs &a, hipStream_t st)
{
    constexpr int N = 1 << LOGN;
    const double2 *tw = nullptr;
    if (int rc = twiddles<LOGN>(&tw)) return rc;
    const dim3 grid((unsigned)ceil_div(a.n_rows, (int64_t)group_rows<N, FEW>()));
    hipLaunchKernelGGL((k_theta_shift<LOGN, FEW>), grid, dim3(group_threads<N, FEW>()), 0, st, a.in, a.out, tw, a.rho_dev,
                       a.rho, a.order, a.row_map, a.n_rows);
    MS_HIP(hipGetLastError());
    return MS_OK;
}

template <int LOGN, bool FEW>
int launch_spectrum(const ShiftArgs &a, hipStream_t st)
{
    constexpr int N = 1 << LOGN;
    const double2 *tw = nullptr;
    if (int rc = twiddles<LOGN>(&tw)) return rc;
    const dim3 grid((unsigned)ceil_div(a.n_rows, (int64_t)group_rows<N, FEW>()));
    hipLaunchKernelGGL((k_theta_spectrum<LOGN, FEW>), grid, dim3(FEW ? row_threads<N>() : SP_THREADS), 0, st, a.in, a.out, tw,
                       a.n_rows);
    MS_HIP(hipGetLastError());
    return MS_OK;
}

typedef int (*RowsLaunch)(const ShiftArgs &, hipStream_t);
constexpr RowsLaunch SHIFT_OF[SP_MAX_LOG2 + 1] = {
    nullptr, launch_shift<1, false>, launch_shift<2, false>, launch_shift<3, false>, launch_shift<4, false>,
    launch_shift<5, false>, launch_shift<6, false>, launch_shift<7, false>, launch_shift<8, false>,
    launch_shift<9, false>, launch_shift<10, false>, launch_shift<11, false>};
constexpr RowsLaunch SPECTRUM_OF[SP_MAX_LOG2 + 1] = {
    nullptr, launch_spectrum<1, false>, launch_spectrum<2, false>, launch_spectrum<3, false>, launch_spectrum<4, false>,
    launch_spectrum<5, false>, launch_spectrum<6, false>, launch_spectrum<7, false>, nullptr,   // 256: always a row a workgroup
    launch_spectrum<9, false>, launch_spectrum<10, false>, launch_spectrum<11, false>};

// Up to three rows a CU go one to a workgroup (see group_rows), all in flight
// at once; more share workgroups.  theta_shift of 50 rows of 64, 256 and 1024:
// 4.6, 6.4 and 9.1 us (shared: 6.5, 9.2 and 11.6), of 768 rows 5.8, 9.3 and 20.5
// (6.8, 10.7 and 23), of 2000 rows of 256: 17.6 (15.4); the spectrum of 200
// rows of 8, 128 and 512: 2.4, 4.1 and 4.6 us (4.8, 5.3 and 6.0).  Up to twice
// as many where a shared workgroup is a long chain (the shortest rows, a thread
// each; 1000 rows of 8: 5.4 us against 7.5) or a small part of the chip (1000 rows
// of 128 and 256: 7.8 and 10.4 against 9.8 and 11.6; of 512: 17 against 15).
// Rows of 2048 have all of a workgroup's threads either way (50 rows: 12.6 us,
// 12.1).
constexpr int64_t FEW_ROWS = 768, FEW_SAMPLES = 1 << 18;
constexpr int FEW_MAX_LOG2 = 10;
constexpr RowsLaunch SHIFT_FEW[FEW_MAX_LOG2 + 1] = {
    nullptr, launch_shift<1, true>, launch_shift<2, true>, launch_shift<3, true>, launch_shift<4, true>,
    launch_shift<5, true>, launch_shift<6, true>, launch_shift<7, true>, launch_shift<8, true>, launch_shift<9, true>,
    launch_shift<10, true>};
constexpr RowsLaunch SPECTRUM_FEW[FEW_MAX_LOG2 + 1] = {
    nullptr, launch_spectrum<1, true>, launch_spectrum<2, true>, launch_spectrum<3, true>, launch_spectrum<4, true>,
    launch_spectrum<5, true>, launch_spectrum<6, true>, launch_spectrum<7, true>, launch_spectrum<8, true>,
    launch_spectrum<9, true>, launch_spectrum<10, true>};

bool few_rows(int n_theta, int64_t n_rows)
{
    const bool twice = n_theta <= 8 || (n_theta >= 128 && n_rows * n_theta <= FEW_SAMPLES);
    return n_theta <= 1 << FEW_MAX_LOG2 && n_rows <= (twice ? 2 * FEW_ROWS : FEW_ROWS);
}

// The spectrum takes a row to a workgroup for more: its registers let four rows
// of 1024 run on a CU, and once the rows' bytes are what it takes (from 2^22
// samples on) small workgroups, which start and end by themselves, keep the
// loads and stores going where shared ones do so in turns.  769 rows of 1024:
// 14.1 us, 15.8 shared; 8192 of 512: 44.5 (47.2), 20000: 118 (124); 8192 of 1024:
// 101 (103).  Between the two the shared ones' shorter exchange is ahead: 2300
// rows of 512 and 1024 15.7 and 27.2 us against 17.0 and 30.2.  256 samples, half
// a wave: 1300, 4000 and 12000 rows 7.4, 14.7 and 31.6 us, 8.4, 17.0 and 34.1
// shared; of 128, 4000 rows 10.4 against 9.4.
constexpr int64_t LONE_ROWS = 1024, LONE_SAMPLES = 1 << 22;

bool lone_spectrum(int n_theta, int64_t n_rows)
{
    if (n_theta < 256 || n_theta > 1 << FEW_MAX_LOG2) return few_rows(n_theta, n_rows);
    return n_theta == 256 || n_rows <= LONE_ROWS || n_rows * n_theta >= LONE_SAMPLES;
}

// theta_shift on validated arguments (n_theta a power of two in range).
int shift_rows(const double *in, double *out, int n_theta, int64_t n_rows, const double *rho_dev, double rho,
               int order, const int64_t *row_map, hipStream_t st)
{
    const RowsLaunch *launch = few_rows(n_theta, n_rows) ? SHIFT_FEW : SHIFT_OF;
    return launch[__builtin_ctz(n_theta)]({in, out, rho_dev, rho, order, row_map, n_rows}, st);
}

// Row copies through a row map (negative entries dropped): the unshifted
// layer of the globalized mesh.
__global__ void __launch_bounds__(256) k_copy_rows(const double *in, double *out, const int64_t *row_map,
                                                   int64_t n_rows, int N)
{
    const int64_t per = (int64_t)N * 2;   // double2 per row
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_rows * per) return;
    const int64_t row = i / per, e = i - row * per;
    const int64_t orow = row_map[row];
    if (orow < 0) return;
    reinterpret_cast<double2 *>(out)[orow * per + e] = reinterpret_cast<const double2 *>(in)[i];
}

}  // namespace
}  // namespace ms

using namespace ms;

extern "C" int globalize_workspace_size(int32_t n_theta, int32_t n_s, int32_t n_max, size_t *bytes)
{
    if (!bytes || n_theta < 1 || n_s < 0 || n_max < 0) return fail(MS_E_ARG, "globalize_workspace_size: bad argument");
    const size_t grid = (size_t)n_s * n_theta * 32;
    const size_t map = (size_t)(n_max + 1) * n_s * 8;
    *bytes = ((grid + 255) & ~(size_t)255) + ((map + 255) & ~(size_t)255);
    return MS_OK;
}

extern "C" int globalize_manifold(const double *grid_dev, const double *s_host, int32_t n_theta, int32_t n_s,
                                  int32_t n_max, double omega, double lambda, const map_params_t *map,
                                  double *out_dev, int64_t out_rows_cap, double *s_out_host, int64_t *n_rows_out,
                                  void *ws, size_t ws_bytes, void *stream)
{
    if (!s_host || !map || !n_rows_out || n_s < 1 || n_max < 0 || (!grid_dev) || (!s_out_host))
        return fail(MS_E_ARG, "globalize_manifold: bad argument");
    if (n_theta < 2 || n_theta > (1 << SP_MAX_LOG2) || (n_theta & (n_theta - 1)))
        return fail(MS_E_ARG, "globalize_manifold: n_theta must be a power of two in [2, 2048]");
    if (map->n_periods != 1 && map->n_periods != -1)
        return fail(MS_E_ARG, "globalize_manifold: map->n_periods must be +1 (unstable) or -1 (stable)");
    if (!(lambda > 0.0) || !isfinite(lambda) || !isfinite(omega))
        return fail(MS_E_ARG, "globalize_manifold: need lambda > 0 and a finite omega");
    for (int k = 0; k < n_s; ++k)
        if (!isfinite(s_host[k]) || (k > 0 && !(s_host[k] > s_host[k - 1])))
            return fail(MS_E_ARG, "globalize_manifold: s must be finite and strictly increasing");
    const int d = map->n_periods;
    // the rows (n, k) and their s values, sorted by s (s = 0 kept once)
    struct Entry { double s; int n, k; };
    std::vector<Entry> ent;
    for (int n = 0; n <= n_max; ++n)
        for (int k = 0; k < n_s; ++k) {
            if (n > 0 && s_host[k] == 0.0) continue;
            ent.push_back({pow(lambda, (double)(d * n)) * s_host[k], n, k});
        }
    std::stable_sort(ent.begin(), ent.end(), [](const Entry &a, const Entry &b) { return a.s < b.s; });
    const int64_t M = (int64_t)ent.size();
    *n_rows_out = M;
    if (!out_dev || out_rows_cap < M) return fail(MS_E_CAPACITY, "globalize_manifold: output holds too few rows");
    size_t need = 0;
    int rc = globalize_workspace_size(n_theta, n_s, n_max, &need);
    if (rc) return rc;
    if (!ws || ws_bytes < need) return fail(MS_E_WORKSPACE, "globalize_manifold: workspace too small");
    std::vector<int64_t> rmap((size_t)(n_max + 1) * n_s, -1);
    for (int64_t r = 0; r < M; ++r) {
        rmap[(size_t)ent[r].n * n_s + ent[r].k] = r;
        s_out_host[r] = ent[r].s;
    }
    double *P = (double *)ws;
    int64_t *rmap_dev = (int64_t *)((char *)ws + (((size_t)n_s * n_theta * 32 + 255) & ~(size_t)255));
    hipStream_t st = (hipStream_t)stream;
    MS_HIP(hipMemcpyAsync(rmap_dev, rmap.data(), rmap.size() * 8, hipMemcpyHostToDevice, st));
    MS_HIP(hipStreamSynchronize(st));   // rmap is a host vector of this call
    const int64_t n_states = (int64_t)n_s * n_theta;
    hipLaunchKernelGGL(k_copy_rows, dim3((unsigned)ceil_div(n_states * 2, 256)), dim3(256), 0, st, grid_dev, out_dev,
                       rmap_dev, (int64_t)n_s, (int)n_theta);
    MS_HIP(hipGetLastError());
    if (n_max > 0) MS_HIP(hipMemcpyAsync(P, grid_dev, (size_t)n_states * 32, hipMemcpyDeviceToDevice, st));
    for (int n = 1; n <= n_max; ++n) {
        // P <- F^d(P) = F^(d n)(grid), then W(theta_i, lambda^(d n) s_k) = P shifted by -d n omega
        if ((rc = pertbp_map(P, P, n_states, map, stream))) return rc;
        if ((rc = shift_rows(P, out_dev, n_theta, n_s, nullptr, -(double)(d * n) * omega, 0,
                             rmap_dev + (size_t)n * n_s, st)))
            return rc;
    }
    return MS_OK;
}

extern "C" int theta_spectrum(const double *in_dev, double *out_dev, int32_t n_theta, int64_t n_rows, void *stream)
{
    if (n_rows < 0 || (n_rows > 0 && (!in_dev || !out_dev))) return fail(MS_E_ARG, "theta_spectrum: bad argument");
    if (n_theta < 2 || n_theta > (1 << SP_MAX_LOG2) || (n_theta & (n_theta - 1)))
        return fail(MS_E_ARG, "theta_spectrum: n_theta must be a power of two in [2, 2048]");
    if (n_rows > 0x7fffffff) return fail(MS_E_ARG, "theta_spectrum: too many rows for one launch");
    if (n_rows == 0) return MS_OK;
    const RowsLaunch *launch = lone_spectrum(n_theta, n_rows) ? SPECTRUM_FEW : SPECTRUM_OF;
    return launch[__builtin_ctz(n_theta)]({in_dev, out_dev, nullptr, 0.0, 0, nullptr, n_rows}, (hipStream_t)stream);
}

extern "C" int theta_shift(const double *in_dev, double *out_dev, int32_t n_theta, int64_t n_rows,
                           const double *rho_dev, double rho, int32_t order, void *stream)
{
    if (n_rows < 0 || (n_rows > 0 && (!in_dev || !out_dev))) return fail(MS_E_ARG, "theta_shift: bad argument");
    if (n_theta < 2 || n_theta > (1 << SP_MAX_LOG2) || (n_theta & (n_theta - 1)))
        return fail(MS_E_ARG, "theta_shift: n_theta must be a power of two in [2, 2048]");
    if (order < 0 || order > 2) return fail(MS_E_ARG, "theta_shift: order must be 0, 1 or 2");
    if (!rho_dev && !isfinite(rho)) return fail(MS_E_ARG, "theta_shift: rho must be finite");
    if (n_rows > 0x7fffffff) return fail(MS_E_ARG, "theta_shift: too many rows for one launch");
    if (n_rows == 0) return MS_OK;
    return shift_rows(in_dev, out_dev, n_theta, n_rows, rho_dev, rho, order, nullptr, (hipStream_t)stream);
}

extern "C" int theta_interp(const double *rows_dev, int32_t n_theta, int64_t n_rows, const int64_t *row_dev,
                            const double *theta_dev, int64_t n_query, double *out_dev, void *stream)
{
    if (n_query < 0 || n_rows < 0 || n_theta < 1 ||
        (n_query > 0 && (!rows_dev || !row_dev || !theta_dev || !out_dev)))
        return fail(MS_E_ARG, "theta_interp: bad argument");
    if (n_query == 0) return MS_OK;
    hipStream_t st = (hipStream_t)stream;
    const int N = (int)n_theta;
    // A block's table and offsets cost some 8 us: short rows repay them only
    // with many queries for each block (129 samples, 5000 queries: 11 to 16
    // against 9 us; 256, 20000: 16 against 33; 256 and 300, 500: 5.5 and 6.0
    // against 5.1 and 5.5, 4096: 7.6 and 8.4 against 9.4 and 10.7), the shortest
    // never (64 samples, 20000 queries: 15 against 17; 33, 65536: 47 and 47).  An
    // odd length's table has two numbers a sample (319 and 511 samples, 4096
    // queries of as many rows: 13.9 and 17.2 against 10.6 and 14.8, of one row 11.7
    // and 11.9 against 10.0 and 13.0; 8192 of one row 13.5 and 15.6 against 16.3
    // and 21.5).
    const bool odd = (N & 1) != 0;
    if (N > IP_MAX_N || N < 64 || (N < 256 && n_query < 16384) || (N < 320 && n_query < 2048) ||
        (odd && N < 512 && n_query <= 4096)) {
        const int64_t blocks = ceil_div(n_query, 4);
        if (blocks > 0x7fffffff) return fail(MS_E_ARG, "theta_interp: too many queries for one launch");
        hipLaunchKernelGGL(k_theta_interp_plain, dim3((unsigned)blocks), dim3(256), 0, st, rows_dev, N, n_rows, row_dev,
                           theta_dev, n_query, out_dev);
        MS_HIP(hipGetLastError());
        return MS_OK;
    }
    InterpArgs g;
    g.in = rows_dev;
    g.rows = row_dev;
    g.theta = theta_dev;
    g.out = out_dev;
    g.n_rows = n_rows;
    g.nq = n_query;
    g.N = N;
    g.slice = g.per_slice = g.bins = g.shift = 0;
    const size_t table = (size_t)(odd ? 16 : 8) * N;
    // Grouped by rows where the rows do not stay in the caches (8 MB: twice
    // an XCD's L2) and are read more than once: 2048 rows of 2048, 4096 queries:
    // 39 us against 42; 4096 rows, 8192 queries: 56 against 78; 300 rows of 1024,
    // 65536 queries: 118 against 171; but 300 rows of 512: 94 against 60, 128 of
    // 2048: 173 against 149.  The grouping's own 9 us want some 5 million samples:
    // 1000 rows of 300, 512 and 1024, 4096 queries: 16.4, 18.3 and 22.6 against
    // 8.6, 12.4 and 21.3; of 700, 8192 queries: 20.3 against 25.5.
    const bool grouped = n_query >= 4096 && n_query >= 2 * n_rows && n_rows > (8 << 20) / (32 * N) &&
                         n_query * N >= (int64_t)5 << 20;
    int64_t blocks;
    size_t lds = table;
    int threads = IP_BLOCK;
    if (grouped) {
        const int64_t slices = ceil_div(n_query, (int64_t)IP_SLICE);
        g.slice = (int)ceil_div(n_query, slices);
        g.share = (int)std::max<int64_t>(32, ceil_div(g.slice, 256));
        g.per_slice = (int)ceil_div(g.slice, g.share);
        while ((((n_rows > 0 ? n_rows : 1) - 1) >> g.shift) >= IP_MAX_BINS) ++g.shift;
        g.bins = n_rows > 0 ? (int)((n_rows - 1) >> g.shift) + 1 : 1;
        lds = std::max(table, (size_t)g.bins * 4);
        blocks = slices * g.per_slice;
    } else {
        threads = n_query >= 16384 ? 1024 : 256;     // few queries: spread over the CUs, a table each
        const int w = threads / 64;
        g.share = (int)std::min<int64_t>(IP_MAX_Q, w * ceil_div(n_query, w * (int64_t)(262144 / threads)));
        blocks = ceil_div(n_query, g.share);
    }
    if (blocks > 0x7fffffff) return fail(MS_E_ARG, "theta_interp: too many queries for one launch");
    const dim3 grid((unsigned)blocks), block((unsigned)threads);
    if (odd && grouped) hipLaunchKernelGGL((k_theta_interp<true, true>), grid, block, lds, st, g);
    else if (odd) hipLaunchKernelGGL((k_theta_interp<true, false>), grid, block, lds, st, g);
    else if (grouped) hipLaunchKernelGGL((k_theta_interp<false, true>), grid, block, lds, st, g);
    else hipLaunchKernelGGL((k_theta_interp<false, false>), grid, block, lds, st, g);
    MS_HIP(hipGetLastError());
    return MS_OK;
}
