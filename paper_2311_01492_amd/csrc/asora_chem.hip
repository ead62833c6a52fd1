// Hydrogen chemistry step (Section 2.1): the time-averaged solution of the
// chemistry equation over a step dt for the time-averaged rate Gamma, with
// the electron density iterated per cell.  Elementwise over the grid: 44
// bytes per cell move (Gamma, n_H FP32; y0, the previous <y> FP64 in; <y>,
// y(dt) FP64 and <y> FP32 out), one thread per cell, grid-stride.
// The FP64 exponentials of the n_e passes set its time (a wave takes as many
// passes as its slowest cell), then the fields.  250^3 cells half ionized, 10
// Myr: 303 us with the library's expm1 and exp in every pass and a count's
// atomics from every wave (all to one address: 12 ns each); 258 with one
// exponential for both; 178 with the secant in the passes, a cell's loads one
// cell ahead and an atomic per work-group, 32 waves a CU.
//
// Carried in the neutral fraction y = 1 - x_HII:
//   rate = Gamma + n_e (C_H + alpha_H),  y_eq = n_e alpha_H / rate,
//   <y>  = y_eq + (y0 - y_eq) (1 - e^-u) / u,  y(dt) = y_eq + (y0 - y_eq) e^-u,
//   u = rate dt,  n_e = n_H (1 - <y>), starting from n_H (1 - y0).
#include <hip/hip_runtime.h>

#include "asora_internal.h"

#include "asora_dev.h"

namespace asora {

namespace {

constexpr int kChemThreads = 512;

struct ChemArgs {
    long n;
    const float *gamma, *nH;
    const double *y0, *y_prev;
    double *y_avg, *y_end;
    float *y_avg32;
    double dt, inv_dt, alpha, c_h, ne_rtol, conv_rtol;
    int max_iter;
    unsigned long long *changed;   // cells whose <y> moved by more than conv_rtol relative (may be NULL)
    unsigned long long *unconverged;   // cells whose n_e iteration hit max_iter
};

// One n_e pass: <y>, and what y(dt) follows from (end_of_step).
struct Pass {
    double y_eq;
    double u;      // general form
    double p;      // e^-u = 2^k (1 + p)
    int k;
    bool general;
};

// 1/x to the last bits, for x well within the normal range.
__device__ __forceinline__ double recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// The exponential serves both the average and y(dt): -u = k ln 2 + r with
// |r| <= ln 2 / 2, p = e^r - 1 from its series' fit (relative error 2e-18 before
// rounding), 1 - e^-u = (1 - 2^k) - 2^k p without cancellation for small u.  The
// two quotients by the rate share one reciprocal and are corrected by their
// remainders, so that they are as good as divisions.
__device__ __forceinline__ double time_average(double gamma, double n_e, double y0, double dt, double inv_dt,
                                               double alpha, double c_h, Pass &P)
{
    const double rate = gamma + n_e * (c_h + alpha);
    const double u = rate * dt, a = n_e * alpha;
    P.u = u;
    P.general = !(rate > 1e-280 && rate < 1e280 && u > 1e-280 && u < 1e280);
    if (P.general) {   // no rate, or far out of range
        P.y_eq = rate > 0.0 ? a / rate : 1.0;
        // (1 - e^-u) / u; 1 at u = 0
        return P.y_eq + (y0 - P.y_eq) * (u > 0.0 ? -expm1(-u) / u : 1.0);
    }
    const double inv = recip(rate), inv_u = inv * inv_dt;
    double y_eq = a * inv;
    y_eq = fma(fma(-y_eq, rate, a), inv, y_eq);
    const double v = u < 800.0 ? u : 800.0;   // e^-800 is 0
    const double kf = rint(v * -ASORA_K64(1.4426950408889634));
    double r = fma(-kf, ASORA_K64(0.693147180559663), -v);   // (41 bits: the product is exact)
    r = fma(-kf, ASORA_K64(2.8235290563031577e-13), r);
    double p = ASORA_K64(2.090212378204763e-09);
    p = ASORA_HORNER(p, r, 2.510891805611665e-08);
    p = ASORA_HORNER(p, r, 2.7557348756596875e-07);
    p = ASORA_HORNER(p, r, 2.7557244761575786e-06);
    p = ASORA_HORNER(p, r, 2.4801587186627587e-05);
    p = ASORA_HORNER(p, r, 0.00019841269885487796);
    p = ASORA_HORNER(p, r, 0.0013888888888988144);
    p = ASORA_HORNER(p, r, 0.008333333333321782);
    p = ASORA_HORNER(p, r, 0.04166666666666635);
    p = ASORA_HORNER(p, r, 0.16666666666666677);
    p = fma(p, r, 0.5);
    p = fma(p * r, r, r);
    P.k = (int)kf;
    P.p = p;
    P.y_eq = y_eq;
    const double s = ldexp(1.0, P.k);
    const double q = (1.0 - s) - s * p;
    double frac = q * inv_u;
    frac = fma(fma(-frac, u, q), inv_u, frac);
    return y_eq + (y0 - y_eq) * frac;
}

__device__ __forceinline__ double end_of_step(double y0, const Pass &P)
{
    return P.y_eq + (y0 - P.y_eq) * (P.general ? exp(-P.u) : ldexp(1.0 + P.p, P.k));
}

__global__ __launch_bounds__(kChemThreads) void chem_kernel(ChemArgs A)
{
    unsigned int changed = 0, unconverged = 0;
    // the next cell's values are loaded before this one's passes
    const long step = (long)gridDim.x * blockDim.x;
    long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    float g_n = 0.f, h_n = 0.f;
    double y0_n = 0.0, yp_n = 0.0;
    auto fetch = [&](long j) {
        if (j < A.n) {
            g_n = A.gamma[j];
            h_n = A.nH[j];
            y0_n = A.y0[j];
            if (A.y_prev) yp_n = A.y_prev[j];
        }
    };
    fetch(i);
    for (; i < A.n; i += step) {
        const double g = (double)g_n, nH = (double)h_n, y0 = y0_n;
        // n_e from the previous pass's <y> when there is one: the same fixed
        // point, reached in fewer passes
        const double yp = A.y_prev ? yp_n : y0;
        fetch(i + step);
        double ya = yp;
        Pass P;
        P.y_eq = y0;
        P.u = 0.0;
        P.general = true;   // max_iter 0: y(dt) is y0
        int it = 0;
        // Fixed-point passes y -> T(y), from the second on with the secant's
        // estimate of the fixed point.  Only where the passes shrink the
        // distance by half or more by themselves: the passes that a cell with a
        // slower map runs out of are counted as before.  Converged is a pass
        // that moves y by less than ne_rtol, accelerated or not.
        double y_b = 0.0, T_b = 0.0;   // the pass before
        for (; it < A.max_iter; ++it) {
            const double T = time_average(g, nH * (1.0 - ya), y0, A.dt, A.inv_dt, A.alpha, A.c_h, P);
            const double d = T - ya;
            double next = T;
            const bool done = fabs(d) <= A.ne_rtol * T;
            if (!done && it > 0) {
                const double slope = (T - T_b) * recip(ya - y_b);
                const double s = ya + d * recip(1.0 - slope);
                if (fabs(slope) < 0.5 && s > 0.0 && s < 1.0) next = s;
            }
            y_b = ya;
            T_b = T;
            ya = next;
            if (done) break;
        }
        const double ye = end_of_step(y0, P);
        if (it == A.max_iter) ++unconverged;
        A.y_avg[i] = ya;
        A.y_end[i] = ye;
        A.y_avg32[i] = (float)ya;
        if (A.y_prev && fabs(ya - yp) > A.conv_rtol * ya) ++changed;
    }
    // one atomic per work-group for each count: they go to one address, 12 ns
    // each, and all at the end
    __shared__ unsigned int sum[2];
    if (threadIdx.x < 2) sum[threadIdx.x] = 0;
    __syncthreads();
    unsigned int c = changed, u = unconverged;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        c += __shfl_xor(c, o, 64);
        u += __shfl_xor(u, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        if (c) atomicAdd(&sum[0], c);
        if (u) atomicAdd(&sum[1], u);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (A.changed && sum[0]) atomicAdd(A.changed, (unsigned long long)sum[0]);
        if (sum[1]) atomicAdd(A.unconverged, (unsigned long long)sum[1]);
    }
}

// Start of a time step: <y> := y0 (FP64 copy and FP32 for the ray tracing);
// counters cleared (by a kernel: no memset node if the caller records it).
__global__ __launch_bounds__(kChemThreads) void chem_prepare_kernel(long n, const double *y0, double *y_avg,
                                                                    float *y_avg32, unsigned long long *cnt)
{
    if (blockIdx.x == 0 && threadIdx.x < 2) cnt[threadIdx.x] = 0;
    for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
        const double y = y0[i];
        if (y_avg) y_avg[i] = y;
        y_avg32[i] = (float)y;
    }
}

__global__ void chem_clear_kernel(unsigned long long *cnt)
{
    if (threadIdx.x < 2) cnt[threadIdx.x] = 0;
}

}  // namespace

hipError_t launch_chem_prepare(hipStream_t st, long n, const double *y0, double *y_avg, float *y_avg32,
                               unsigned long long *cnt, int n_cu)
{
    long blocks = (n + kChemThreads - 1) / kChemThreads;
    if (blocks > (long)n_cu * 16) blocks = (long)n_cu * 16;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(chem_prepare_kernel, dim3((unsigned)blocks), dim3(kChemThreads), 0, st, n, y0, y_avg,
                       y_avg32, cnt);
    return hipGetLastError();
}

hipError_t launch_chem_clear(hipStream_t st, unsigned long long *cnt)
{
    hipLaunchKernelGGL(chem_clear_kernel, dim3(1), dim3(64), 0, st, cnt);
    return hipGetLastError();
}

hipError_t launch_chemistry(hipStream_t st, const ChemLaunch &L)
{
    ChemArgs A;
    A.n = L.n;
    A.gamma = L.gamma;
    A.nH = L.nH;
    A.y0 = L.y0;
    A.y_prev = L.y_prev;
    A.y_avg = L.y_avg;
    A.y_end = L.y_end;
    A.y_avg32 = L.y_avg32;
    A.dt = L.dt;
    A.inv_dt = 1.0 / L.dt;
    A.alpha = L.alpha;
    A.c_h = L.c_h;
    A.ne_rtol = L.ne_rtol;
    A.conv_rtol = L.conv_rtol;
    A.max_iter = L.max_iter;
    A.changed = L.changed;
    A.unconverged = L.unconverged;
    long blocks = (L.n + kChemThreads - 1) / kChemThreads;
    const long cap = (long)L.n_cu * 4;   // grid-stride beyond 32 waves per CU
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(chem_kernel, dim3((unsigned)blocks), dim3(kChemThreads), 0, st, A);
    return hipGetLastError();
}

}  // namespace asora
