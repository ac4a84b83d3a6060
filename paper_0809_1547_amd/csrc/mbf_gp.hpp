// Bound states of the dimensionless Gross-Pitaevskii equation of the random
// laser (the oscillation condition gain = loss with gain saturation, finite
// gain bandwidth and a quadratic trap from the high-Q modes, Gross-Pitaevskii
// section, Eq. g5):
//
//     -phi'' + tau^2 phi + phi^3 = E phi,     phi(tau) > 0, phi -> 0 at |tau| -> inf,
//
// for a batch of nonlinear eigenvalues E > 1, and the normalised spectrum of
// each solution (its Fourier transform, Eq. s1 and Fig. 5: waist and peak).
//
// Discretisation: M interior points tau_i = -L + (i+1) h, h = 2L/(M+1),
// phi = 0 at tau = +-L, second differences.  Each E is solved by one wave: a
// semi-implicit gradient flow
//     (A + diag(phi_k^2) - E + 1/ds) phi_{k+1} = phi_k / ds,   ds = 1/E
// (A = -d2 + tau^2; an M-matrix, so phi stays positive), then Newton steps
//     (A + diag(3 phi^2) - E) delta = -(A phi + phi^3 - E phi)
// until the update is below 1e-13 of max phi.  A solve is a chain of some 405
// tridiagonal systems, bound by the latency of each.  The spectrum is
//     phit(nu) = (h / 2 pi) sum_i phi_i cos(nu tau_i),  S(nu) = phit(nu)^2
// on nu_k = k dnu; its peak is S(0) and its waist w = sigma_nu / (2 pi),
// sigma_nu^2 the second moment of the symmetric spectrum (S_0 + 2 sum_{k>=1}
// weights), so that a Gaussian S ~ exp(-nu^2 / (8 pi^2 w^2)) has waist w.
#pragma once

#include "mbf_kernels.hpp"

namespace mbf {

constexpr int kGpThreads = 256;        // of k_gp_stats
constexpr int kGpMaxM = 1023;          // interior points (64 lanes of at most 16 rows)

// Sum over the workgroup in a fixed order, returned to every thread.
__device__ __forceinline__ double gp_sum(double x, double* sh) {
    const int t = (int)threadIdx.x;
    x = wave_sum(x);
    __syncthreads();
    if ((t & 63) == 0) sh[t >> 6] = x;
    __syncthreads();
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < kGpThreads / 64; ++w) r += sh[w];
    return r;
}

__device__ __forceinline__ double gp_max(double x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o, 64));
    return x;
}

// 1 / x to within an ulp: the hardware's estimate and two Newton-Raphson steps.
// A correctly rounded division scales its operands and fixes the last bit
// besides, twice the chain; the solutions' errors are no larger without (against
// 64-bit reference solutions 1.0e-15 here, 1.6e-15 with divisions).
__device__ __forceinline__ double gp_rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// Tridiagonal solve of a wave: b the diagonal, s every off-diagonal entry
// between rows of the system, d the right-hand side on entry and the solution
// on exit.  Lane l holds rows R l .. R l + R - 1 in registers; rows at M and
// beyond are identity rows.  Partition method (Wang, ACM TOMS 7, 1981): each
// lane eliminates its rows against the lane before's last unknown and its
// own, which leaves one row per lane; parallel cyclic reduction solves those
// 64 in six exchanges between lanes.  Latency-bound, so nothing waits on
// memory or at a barrier: one elimination of R rows and six exchanges where
// cyclic reduction over all 1024 rows in LDS took ten levels, two divisions a
// row and twenty barriers (a system of 1023 rows 18.9 us; now 1.7 us).
template <int R>
__device__ __forceinline__ void gp_tridiag(const double (&b)[R], double (&d)[R], double s, int M) {
    const int lane = (int)(threadIdx.x & 63u);
    const int rows = M - lane * R;                    // rows of the system from this lane's first on
    const auto up = [&](int r) { return r + 1 < rows ? s : 0.0; };   // entry (r, r+1) = (r+1, r)
    double ib[R], f[R], g[R];
    ib[0] = gp_rcp(b[0]);
    f[0] = lane > 0 && rows > 0 ? s : 0.0;
    double bl = b[0];
#pragma unroll
    for (int r = 1; r < R; ++r) {
        const double c = up(r - 1), m = c * ib[r - 1];
        bl = fma(-m, c, b[r]);
        ib[r] = gp_rcp(bl);
        d[r] = fma(-m, d[r - 1], d[r]);
        f[r] = -m * f[r - 1];
    }
    g[R - 2] = up(R - 2);
#pragma unroll
    for (int r = R - 3; r >= 0; --r) {
        const double m = up(r) * ib[r + 1];
        d[r] = fma(-m, d[r + 1], d[r]);
        f[r] = fma(-m, f[r + 1], f[r]);
        g[r] = -m * g[r + 1];
    }
    // rows r < R-1:  f y(l-1) + x_r / ib + g y(l) = d;  the last row with the
    // next lane's first row put in
    const double cn = up(R - 1);
    const double d0 = __shfl_down(d[0] * ib[0], 1, 64), f0 = __shfl_down(f[0] * ib[0], 1, 64),
                 g0 = __shfl_down(g[0] * ib[0], 1, 64);
    const double ir = gp_rcp(fma(-cn, f0, bl));
    double A = f[R - 1] * ir, C = -cn * g0 * ir, y = fma(-cn, d0, d[R - 1]) * ir;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        // entries that would reach past the ends are 0
        const double Al = __shfl_up(A, o, 64), Cl = __shfl_up(C, o, 64), yl = __shfl_up(y, o, 64);
        const double Ah = __shfl_down(A, o, 64), Ch = __shfl_down(C, o, 64), yh = __shfl_down(y, o, 64);
        const double iv = gp_rcp(fma(-C, Ah, fma(-A, Cl, 1.0)));
        y = fma(-C, yh, fma(-A, yl, y)) * iv;
        A = -A * Al * iv;
        C = -C * Ch * iv;
    }
    const double yl = __shfl_up(y, 1, 64);
#pragma unroll
    for (int r = 0; r < R - 1; ++r) d[r] = fma(-f[r], yl, fma(-g[r], y, d[r])) * ib[r];
    d[R - 1] = y;
}

struct GpArgs {
    const double* E;       // n_E eigenvalues
    int M;                 // interior points (3 .. kGpMaxM)
    double L;              // half-width of the tau window
    int n_nu;              // spectrum points nu_k = k dnu
    double dnu;
    int flow_iters;        // gradient-flow steps before Newton
    int newton_iters;      // Newton steps at most
    double* phi;           // n_E x M
    double* spec;          // n_E x n_nu
    double* stats;         // n_E x kGpStats
};

// stats per E: N = h sum phi^2, w, p = S(0), phi(0) (largest sample), max
// residual |A phi + phi^3 - E phi|, Newton steps taken, 1 when converged
constexpr int kGpStats = 7;

// Whether E lies below every eigenvalue of A: all pivots of A - E are positive
// (rarely asked: every lane takes the M divisions one after another).
__device__ __attribute__((noinline)) bool gp_no_bound_state(double E, int M, double L, double h, double ih2) {
    double d = 0.0;
    for (int i = 0; i < M; ++i) {
        const double tau = -L + (double)(i + 1) * h;
        d = 2.0 * ih2 + tau * tau - E - (i > 0 ? ih2 * ih2 / d : 0.0);
        if (!(d > 0.0)) return false;
    }
    return true;
}

// The bound state of one E: phi and all statistics but the spectrum's.  R rows
// a lane, 64 R >= M; a workgroup is one wave, so few E still take a CU each.
template <int R>
__global__ void __launch_bounds__(64) k_gp_solve(GpArgs g) {
    const int lane = (int)threadIdx.x;
    const int e = (int)blockIdx.x;
    const double E = g.E[e];
    const int M = g.M;
    const int i0 = lane * R;
    const double h = 2.0 * g.L / (double)(M + 1);
    const double ih2 = 1.0 / (h * h);
    const double ids = 1.0 / (1.0 / E);
    // initial profile: the near-threshold Gaussian for E < 3, Thomas-Fermi above
    double ph[R], t2[R], b[R], d[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double tau = -g.L + (double)(i0 + r + 1) * h;
        t2[r] = tau * tau;
        const double v = E < 3.0 ? sqrt(sqrt(2.0) * (E - 1.0)) * exp(-0.5 * tau * tau) : sqrt(fmax(E - tau * tau, 0.0) + 1e-3);
        ph[r] = i0 + r < M ? v : 0.0;
    }
    // gradient flow
    for (int it = 0; it < g.flow_iters; ++it) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            b[r] = i0 + r < M ? 2.0 * ih2 + t2[r] + ph[r] * ph[r] - E + ids : 1.0;
            ph[r] *= ids;
        }
        gp_tridiag<R>(b, ph, -ih2, M);
    }
    // A phi + phi^3 - E phi at row r; pl, pr: phi beside the lane's rows (zero
    // past the ends)
    const auto F = [&ph, &t2, i0, M, ih2, E](int r, double pl, double pr) {
        const double p = ph[r], l = r > 0 ? ph[r > 0 ? r - 1 : 0] : pl, q = r < R - 1 ? ph[r < R - 1 ? r + 1 : r] : pr;
        return i0 + r < M ? (2.0 * p - l - q) * ih2 + t2[r] * p + p * p * p - E * p : 0.0;
    };
    const auto below = [lane](double x) { const double v = __shfl_up(x, 1, 64); return lane == 0 ? 0.0 : v; };
    const auto above = [lane](double x) { const double v = __shfl_down(x, 1, 64); return lane == 63 ? 0.0 : v; };
    // Newton
    int steps = 0;
    int converged = 0;
    bool decayed = false;
    for (int it = 0; it < g.newton_iters; ++it) {
        const double pl = below(ph[R - 1]), pr = above(ph[0]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            b[r] = i0 + r < M ? 2.0 * ih2 + t2[r] + 3.0 * ph[r] * ph[r] - E : 1.0;
            d[r] = -F(r, pl, pr);
        }
        gp_tridiag<R>(b, d, -ih2, M);
        double dmax = 0.0, pmax = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ph[r] += d[r];
            dmax = fmax(dmax, fabs(d[r]));
            pmax = fmax(pmax, fabs(ph[r]));
        }
        dmax = gp_max(dmax);
        pmax = gp_max(pmax);
        steps = it + 1;
        // where the box has no bound state phi decays, and its steps end among the
        // subnormal numbers, whose rounding is as large as they are: zero is the
        // state then.  (A bound state that the flow missed stays unconverged.)
        if (pmax < 2.2250738585072014e-308 && !decayed) {
            decayed = true;
            if (gp_no_bound_state(E, M, g.L, h, ih2)) {
#pragma unroll
                for (int r = 0; r < R; ++r) ph[r] = 0.0;
            }
        }
        if (dmax <= 1e-13 * pmax) {
            converged = 1;
            break;
        }
    }
    // residual, norm, output profile
    double res = 0.0, nrm = 0.0, pk = 0.0;
    const double pl = below(ph[R - 1]), pr = above(ph[0]);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double p = ph[r];
        res = fmax(res, fabs(F(r, pl, pr)));
        nrm += p * p;
        pk = fmax(pk, p);
        if (i0 + r < M) g.phi[(int64_t)e * M + i0 + r] = p;
    }
    res = gp_max(res);
    pk = gp_max(pk);
    nrm = h * wave_sum(nrm);
    if (lane == 0) {
        double* st = g.stats + (int64_t)e * kGpStats;
        st[0] = nrm;
        st[3] = pk;
        st[4] = res;
        st[5] = (double)steps;
        st[6] = (double)converged;
    }
}

// Spectra of eight solutions at 64 frequencies a workgroup.  A cosine costs two
// orders of magnitude more than the multiplication that uses it, so a lane
// forms the cosines of its frequency once for eight solutions, and once for
// tau and -tau.  The rows go to the 16 waves in turn, eight at a time, held
// one a lane and solution and broadcast from there (scalar loads of them miss
// the scalar cache at every row: 388 us); the waves' sums are added in order.
// 256 solutions of 1023 rows at 512 frequencies take 34 us, where one
// frequency and solution a thread, each with its own cosines, took about 500.
constexpr int kGpSpecE = 8, kGpSpecWaves = 16;

__global__ void __launch_bounds__(64 * kGpSpecWaves) k_gp_spec(const double* __restrict__ phi, double* __restrict__ spec,
                                                              int n_E, int M, double L, int k0, int n_nu, double dnu) {
    __shared__ double sum[kGpSpecE][64];
    const int lane = (int)(threadIdx.x & 63u);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const unsigned k = (unsigned)k0 + blockIdx.x * 64u + (unsigned)lane;
    const int e0 = (int)blockIdx.y * kGpSpecE;
    const double nu = (double)k * dnu, h = 2.0 * L / (double)(M + 1);
    const double* const row = phi + (int64_t)min(e0 + (lane >> 3), n_E - 1) * M;
    const int half = (M + 1) / 2;                     // rows with tau <= 0
    double acc[kGpSpecE];
#pragma unroll
    for (int q = 0; q < kGpSpecE; ++q) acc[q] = 0.0;
    for (int i0 = 8 * w; i0 < half; i0 += 8 * kGpSpecWaves) {
        const int i = i0 + (lane & 7), o = M - 1 - i;
        double p = 0.0;                               // phi(tau) + phi(-tau)
        if (i < half) p = row[i] + (o > i ? row[o] : 0.0);
        for (int u = 0; u < 8; ++u) {
            const double c = cos(nu * (-L + (double)(i0 + u + 1) * h));
#pragma unroll
            for (int q = 0; q < kGpSpecE; ++q) {
                const int from = 8 * q + u;
                const double pq = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(p), from),
                                                   __builtin_amdgcn_readlane(__double2loint(p), from));
                acc[q] = fma(pq, c, acc[q]);
            }
        }
    }
    for (int v = 0; v < kGpSpecWaves; ++v) {
        if (v == w) {
#pragma unroll
            for (int q = 0; q < kGpSpecE; ++q) sum[q][lane] = (v == 0 ? 0.0 : sum[q][lane]) + acc[q];
        }
        __syncthreads();
    }
    if (w < kGpSpecE && e0 + w < n_E && k < (unsigned)n_nu) {
        const double f = sum[w][lane] * (h / (2.0 * 3.14159265358979323846));
        spec[(int64_t)(e0 + w) * n_nu + k] = f * f;
    }
}

// Waist and peak of each spectrum.
__global__ void __launch_bounds__(kGpThreads) k_gp_stats(GpArgs g) {
    __shared__ double sh[kGpThreads / 64];
    const int t = (int)threadIdx.x;
    const int e = (int)blockIdx.x;
    const double* S = g.spec + (int64_t)e * g.n_nu;
    double s0 = 0.0, s2 = 0.0;
    for (int k = t; k < g.n_nu; k += kGpThreads) {
        const double nu = (double)k * g.dnu;
        const double wgt = k == 0 ? 1.0 : 2.0;    // the spectrum is even in nu
        s0 += wgt * S[k];
        s2 += wgt * S[k] * nu * nu;
    }
    s0 = gp_sum(s0, sh);
    s2 = gp_sum(s2, sh);
    if (t == 0) {
        double* st = g.stats + (int64_t)e * kGpStats;
        st[1] = s0 > 0.0 ? sqrt(s2 / s0) / (2.0 * 3.14159265358979323846) : 0.0;
        st[2] = S[0];
    }
}

// Queue the solves of n eigenvalues, their spectra and statistics.  Rows a
// lane: the fewest that hold M rows on 64 lanes (fewer rows, a shorter chain).
inline void gp_launch(const GpArgs& g, int n, hipStream_t st) {
    const dim3 gs((unsigned)n), tb(64);
    if (g.M <= 64 * 4) hipLaunchKernelGGL(k_gp_solve<4>, gs, tb, 0, st, g);
    else if (g.M <= 64 * 8) hipLaunchKernelGGL(k_gp_solve<8>, gs, tb, 0, st, g);
    else hipLaunchKernelGGL(k_gp_solve<16>, gs, tb, 0, st, g);
    // a launch holds fewer than 2^32 threads along x
    constexpr int kSlice = 1 << 27;
    for (int64_t k0 = 0; k0 < g.n_nu; k0 += kSlice) {
        const int nk = (int)(g.n_nu - k0 < kSlice ? g.n_nu - k0 : kSlice);
        hipLaunchKernelGGL(k_gp_spec, dim3((unsigned)((nk - 1) / 64 + 1), (unsigned)((n + kGpSpecE - 1) / kGpSpecE)),
                           dim3(64 * kGpSpecWaves), 0, st, g.phi, g.spec, n, g.M, g.L, (int)k0, g.n_nu, g.dnu);
    }
    hipLaunchKernelGGL(k_gp_stats, dim3((unsigned)n), dim3(kGpThreads), 0, st, g);
}

}  // namespace mbf
