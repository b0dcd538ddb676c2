// One-dimensional growing domain (Sec. 3.1.2, Example 1): batched float64
// IMEX solves with a growth function rho(t), the misfit at T, and the C ABI
// of include/rdbayes_growth1d.h.
//
// Sixteen lanes per item, four items per wavefront.  Lane L of an item owns
// the M = ceil(n / 16) neighbouring rows L M .. L M + M - 1 of both
// tridiagonal systems (u and v), so n <= 128 cells fit; rows past n carry
// zeros and no coupling.  Each lane eliminates inside its rows (forward, then
// backward, which leaves its first row as a function of its own last row and
// of the last row of the lane before), the sixteen last rows form a
// tridiagonal system that four levels of parallel cyclic reduction solve with
// lane shifts inside a 16-lane row, and the lane's other rows follow by
// substitution: 20 operations per row and system plus 26 per level, where
// cyclic reduction over all rows takes 16 per row, system and each of its six
// levels and an LDS round trip with a barrier per level.  The fields stay in
// registers for the whole horizon; only the data and the results touch HBM.
//
// What bounds it: FP64 issue; at 4096 items, one wavefront per SIMD, vector
// instructions are active in 0.85 of the cycles.  Measured, n = 100, 1000 steps
// of 4096 items: 1.17 to 1.21 ms; cyclic reduction over all rows by one wavefront
// per item 7.46 ms.

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <hip/hip_runtime.h>

#include "../../include/rdbayes_growth1d.h"
#include "rd_device.hpp"
#include "rd_sampler.hpp"

namespace rd {
namespace g1d {

constexpr int kLanes = 16;  // lanes of an item (a DPP row)

struct Args {
    int n, n_steps, law, obs;
    double inv_tau, tau, inv_T, rho_T;
    double a, b, g, d;
    double inv_2s2;           // 1 / (2 sigma^2)
    const double *u0, *v0;    // [n]
    const double *y;          // [2][n] or null
    const double *beta;       // [m][beta_stride] (polynomial law)
    int beta_stride;
    const int *need;          // [m] or null: 0 = do not solve
    int m;
    double *u_out, *v_out;    // [m][n] or null
    double *phi;              // [m] or null
    int *status;              // [m] or null
};

// 1/x from the hardware estimate refined by two Newton steps (e = 1 - x r,
// r <- r + r e); each step squares the relative error, so the result is
// within an ulp or two for the positive, well-scaled pivots of these
// diagonally dominant systems.
__device__ inline double recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}

// rho(t) and rho'(t).  Polynomial: Horner in s = t / T with beta_4 fixed by
// rho(T) = rho_T; the data laws of eq. (grates).
__device__ inline void growth(const Args &a, double b1, double b2, double b3, double b4, double t,
                              double &rho, double &drho)
{
    if (a.law == G1D_LAW_POLY) {
        const double s = t * a.inv_T;
        rho = 1.0 + s * (b1 + s * (b2 + s * (b3 + s * b4)));
        drho = (b1 + s * (2.0 * b2 + s * (3.0 * b3 + s * 4.0 * b4))) * a.inv_T;
    } else if (a.law == G1D_LAW_EXP) {
        rho = exp(0.001 * t);
        drho = 0.001 * rho;
    } else {
        const double K = exp(0.6);
        const double e = exp(0.01 * t);
        const double D = 1.0 + (e - 1.0) / K;
        rho = e / D;
        drho = 0.01 * e * (1.0 - 1.0 / K) / (D * D);
    }
}

// The value of the lane kBy before (after) this one in its item, zero past
// the item's ends.
template <int kBy>
__device__ __forceinline__ double before(double v)
{
    return dpp_f64<0x110 + kBy, 0xF>(v);
}
template <int kBy>
__device__ __forceinline__ double after(double v)
{
    return dpp_f64<0x100 + kBy, 0xF>(v);
}

// One level of cyclic reduction on the rows a x- + b x + c x+ = d of the two
// systems, x-, x+ the unknowns kBy lanes away.
template <int kBy>
__device__ __forceinline__ void pcr_level(double (&a)[2], double (&b)[2], double (&c)[2],
                                          double (&d)[2])
{
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const double rb = recip(b[s]);
        const double ar = a[s] * rb, cr = c[s] * rb, dr = d[s] * rb;
        const double am = before<kBy>(ar), cm = before<kBy>(cr), dm = before<kBy>(dr);
        const double ap = after<kBy>(ar), cp = after<kBy>(cr), dp = after<kBy>(dr);
        b[s] = fma(-a[s], cm, fma(-c[s], ap, b[s]));
        d[s] = fma(-a[s], dm, fma(-c[s], dp, d[s]));
        a[s] = -a[s] * am;
        c[s] = -c[s] * cp;
    }
}

// Sum over the lanes of an item, in its last lane.
__device__ __forceinline__ double item_sum(double x)
{
    x += before<1>(x);
    x += before<2>(x);
    x += before<4>(x);
    x += before<8>(x);
    return x;
}

// The pivots of the forward pass.  kExcess: as the pivot less the coupling to
// the next row, e, which is what stays of the diagonal when the neighbours'
// couplings are taken out: the row's own excess and the part of the previous
// row's, all positive, where b - c^2 / b of the full diagonals cancels it out of
// 2 k.  From five rows a lane that cancellation shows (r.m.s. error of u against
// long double, 1000 steps, n = 100 / 128: full diagonals 5.8e-14 / 7.7e-14, this
// 4.0e-14 / 4.3e-14, cyclic reduction over all rows 4.9e-14 / 5.8e-14); below, full
// diagonals are no further off than cyclic reduction (n = 64: 4.5e-14 for 4.9e-14),
// and this takes 4 to 7 % longer at n = 48 and 64.
template <int M>
__global__ __launch_bounds__(64) void k_g1d_solve(Args a)
{
    constexpr bool kExcess = M > 4;
    const int lane = threadIdx.x & (kLanes - 1), sub = threadIdx.x / kLanes;
    const int item = blockIdx.x * (64 / kLanes) + sub;
    const int n = a.n, i0 = lane * M;
    int st = item < a.m ? 0 : RD_ST_OUT_OF_PRIOR;
    // x[0] = u, x[1] = v; cpl: 1 where row j couples to row j + 1; nb: number
    // of neighbours; src: source terms (all zero in rows past n)
    double x[2][M], cpl[M], nb[M], src[2][M];
    const double left = lane > 0 && i0 < n ? 1.0 : 0.0;
#pragma unroll
    for (int j = 0; j < M; ++j) {
        const int i = i0 + j;
        const bool in = i < n;
        x[0][j] = in ? a.u0[i] : 0.0;
        x[1][j] = in ? a.v0[i] : 0.0;
        cpl[j] = i + 1 < n ? 1.0 : 0.0;
        nb[j] = cpl[j] + (in && i > 0 ? 1.0 : 0.0);
        src[0][j] = in ? a.g * a.a : 0.0;
        src[1][j] = in ? a.g * a.b : 0.0;
    }
    double b1 = 0.0, b2 = 0.0, b3 = 0.0, b4 = 0.0;
    if (a.law == G1D_LAW_POLY && st == 0) {
        const double *bp = a.beta + (size_t)item * a.beta_stride;
        b1 = bp[0];
        b2 = bp[1];
        b3 = bp[2];
        b4 = a.rho_T - 1.0 - b1 - b2 - b3;
    }
    if (st == 0 && a.need && !a.need[item])
        st = RD_ST_OUT_OF_PRIOR;
    const double nn = (double)n * (double)n;
    for (int k = 0; k < a.n_steps && __any(st == 0); ++k) {
        if (st == 0) {  // (all or none of an item's lanes)
            double rho, drho;
            growth(a, b1, b2, b3, b4, (double)k * a.tau, rho, drho);
            if (!(rho > 0.0)) {
                st = RD_ST_OUT_OF_PRIOR;
            } else {
                const double rr = recip(rho);
                const double base = fma(drho, rr, a.inv_tau);
                double kk[2];
                kk[0] = nn * rr * rr;
                kk[1] = a.d * kk[0];
                // rows after the forward pass: x_j = dr + fr x_left + cr x_{j+1}
                double cr[2][M], dr[2][M], fr[2][M], c[2], b[2], d[2], f[2], e[2];
                f[0] = kk[0] * left;
                f[1] = kk[1] * left;
#pragma unroll
                for (int j = 0; j < M; ++j) {
                    const double gu = a.g * x[0][j];
                    double bj[2], dj[2];
                    bj[0] = fma(-gu, x[1][j], base + a.g);
                    bj[1] = fma(gu, x[0][j], base);
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        dj[s] = fma(x[s][j], a.inv_tau, src[s][j]);
                        if constexpr (kExcess) {
                            bj[s] = j > 0 ? fma(cr[s][j - 1], e[s], bj[s]) : bj[s] + f[s];
                        } else {
                            bj[s] = fma(kk[s], nb[j], bj[s]);
                            if (j > 0)
                                bj[s] = fma(-c[s], cr[s][j - 1], bj[s]);
                        }
                        if (j > 0) {  // c: coupling of row j - 1 to this one
                            dj[s] = fma(c[s], dr[s][j - 1], dj[s]);
                            f[s] = c[s] * fr[s][j - 1];
                        }
                        c[s] = kk[s] * cpl[j];
                        e[s] = bj[s];
                        if constexpr (kExcess)
                            bj[s] += c[s];
                        if (j < M - 1) {
                            const double rb = recip(bj[s]);
                            cr[s][j] = c[s] * rb;
                            dr[s][j] = dj[s] * rb;
                            fr[s][j] = f[s] * rb;
                        }
                        b[s] = bj[s];
                        d[s] = dj[s];
                    }
                }
                // the first row in terms of x_left and the last row:
                // x_0 = A + B x_left + E x_last; the next lane's closes the
                // equation of this lane's last row
                double aa[2], cc[2];
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    double A = 0.0, B = 0.0, E = 1.0;
#pragma unroll
                    for (int j = M - 2; j >= 0; --j) {
                        A = fma(cr[s][j], A, dr[s][j]);
                        B = fma(cr[s][j], B, fr[s][j]);
                        E = cr[s][j] * E;
                    }
                    const double An = after<1>(A), Bn = after<1>(B), En = after<1>(E);
                    aa[s] = -f[s];
                    b[s] = fma(-c[s], Bn, b[s]);
                    cc[s] = -c[s] * En;
                    d[s] = fma(c[s], An, d[s]);
                }
                pcr_level<1>(aa, b, cc, d);
                pcr_level<2>(aa, b, cc, d);
                pcr_level<4>(aa, b, cc, d);
                pcr_level<8>(aa, b, cc, d);
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    x[s][M - 1] = d[s] * recip(b[s]);
                    const double xl = before<1>(x[s][M - 1]);
#pragma unroll
                    for (int j = M - 2; j >= 0; --j)
                        x[s][j] = fma(cr[s][j], x[s][j + 1], fma(fr[s][j], xl, dr[s][j]));
                }
            }
        }
    }
    double acc = 0.0;
    bool bad = false;
    if (item < a.m) {
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const int i = i0 + j;
            if (i < n) {
                bad = bad || !isfinite(x[0][j]) || !isfinite(x[1][j]);
                if (a.u_out) {
                    a.u_out[(size_t)item * n + i] = x[0][j];
                    a.v_out[(size_t)item * n + i] = x[1][j];
                }
                if (a.y) {
                    if (a.obs & 1) {
                        const double e = a.y[i] - x[0][j];
                        acc += e * e;
                    }
                    if (a.obs & 2) {
                        const double e = a.y[n + i] - x[1][j];
                        acc += e * e;
                    }
                }
            }
        }
    }
    const bool any_bad = (__ballot(bad) >> (kLanes * sub)) & 0xFFFFull;
    if (st == 0 && any_bad)
        st = RD_ST_NONFINITE;
    acc = item_sum(acc);
    if (lane == kLanes - 1 && item < a.m) {
        if (a.status)
            a.status[item] = st;
        if (a.phi)
            a.phi[item] = st == 0 ? acc * a.inv_2s2 : INFINITY;
    }
}

hipError_t launch_solve(const Args &a, hipStream_t s)
{
    if (a.m <= 0)
        return hipSuccess;
    // the fewest rows per lane that hold n cells
    const dim3 grid((a.m + 64 / kLanes - 1) / (64 / kLanes)), block(64);
    switch ((a.n + kLanes - 1) / kLanes) {
    case 1: hipLaunchKernelGGL(k_g1d_solve<1>, grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL(k_g1d_solve<2>, grid, block, 0, s, a); break;
    case 3: hipLaunchKernelGGL(k_g1d_solve<3>, grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL(k_g1d_solve<4>, grid, block, 0, s, a); break;
    case 5: hipLaunchKernelGGL(k_g1d_solve<5>, grid, block, 0, s, a); break;
    case 6: hipLaunchKernelGGL(k_g1d_solve<6>, grid, block, 0, s, a); break;
    case 7: hipLaunchKernelGGL(k_g1d_solve<7>, grid, block, 0, s, a); break;
    case 8: hipLaunchKernelGGL(k_g1d_solve<8>, grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace g1d
}  // namespace rd

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------

using namespace rd;

extern "C" int32_t rd_set_error(int32_t code, const char *msg);

namespace {

int32_t fail(int32_t code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    return rd_set_error(code, buf);
}

#define G1D_TRY(expr)                                                                  \
    do {                                                                               \
        hipError_t e_ = (expr);                                                        \
        if (e_ != hipSuccess)                                                          \
            return fail(RD_EHIP, "%s: %s", #expr, hipGetErrorString(e_));              \
    } while (0)

}  // namespace

struct g1d_problem {
    g1d_desc desc{};
    int device = 0;
    double *u0 = nullptr, *v0 = nullptr, *y = nullptr;
    uint64_t *ctr = nullptr;      // [2] sampler step counter, step of trace row 0
    double *phi_prop = nullptr;   // [max][4]
    int *inside = nullptr;        // [max]
    double *ll_prop = nullptr;    // [max]
    int *status = nullptr;        // [max]
};

namespace {

g1d::Args base_args(const g1d_problem *p)
{
    const g1d_desc &d = p->desc;
    g1d::Args a{};
    a.n = d.n;
    a.n_steps = d.n_steps;
    a.law = d.law;
    a.obs = d.obs;
    a.tau = d.tau;
    a.inv_tau = 1.0 / d.tau;
    a.inv_T = 1.0 / ((double)d.n_steps * d.tau);
    a.rho_T = d.rho_T;
    a.a = d.theta[0];
    a.b = d.theta[1];
    a.g = d.theta[2];
    a.d = d.theta[3];
    a.inv_2s2 = p->y ? 1.0 / (2.0 * d.sigma * d.sigma) : 0.0;
    a.u0 = p->u0;
    a.v0 = p->v0;
    a.y = p->y;
    a.beta_stride = 3;
    return a;
}

void release(g1d_problem *p)
{
    hipFree(p->u0);
    hipFree(p->v0);
    hipFree(p->y);
    hipFree(p->ctr);
    hipFree(p->phi_prop);
    hipFree(p->inside);
    hipFree(p->ll_prop);
    hipFree(p->status);
}

int32_t check_batch(const g1d_problem *p, int32_t n, const double *beta)
{
    if (!p)
        return fail(RD_EINVAL, "problem is NULL");
    if (n < 0 || n > p->desc.max_batch)
        return fail(RD_EINVAL, "n = %d outside [0, max_batch = %d]", n, p->desc.max_batch);
    if (n > 0 && p->desc.law == G1D_LAW_POLY && !beta)
        return fail(RD_EINVAL, "beta is required with the polynomial growth law");
    return RD_OK;
}

}  // namespace

extern "C" int32_t g1d_init(const g1d_desc *d, g1d_problem **out)
{
    if (!d || !out)
        return fail(RD_EINVAL, "desc and out are required");
    *out = nullptr;
    if (d->n < 2 || d->n > G1D_MAX_N)
        return fail(RD_EINVAL, "n = %d outside [2, %d]", d->n, G1D_MAX_N);
    if (d->n_steps < 0 || !(d->tau > 0.0) || !isfinite(d->tau))
        return fail(RD_EINVAL, "n_steps must be >= 0 and tau > 0");
    if (d->law < G1D_LAW_POLY || d->law > G1D_LAW_LOGISTIC)
        return fail(RD_EINVAL, "law %d unknown", d->law);
    if (d->law == G1D_LAW_POLY && !(d->rho_T > 0.0))
        return fail(RD_EINVAL, "rho_T must be > 0");
    for (int i = 0; i < 4; ++i)
        if (!isfinite(d->theta[i]))
            return fail(RD_EINVAL, "theta must be finite");
    if (!d->u0 || !d->v0)
        return fail(RD_EINVAL, "u0 and v0 are required");
    if (d->y && ((d->obs & 3) == 0 || (d->obs & ~3) != 0 || !(d->sigma > 0.0)))
        return fail(RD_EINVAL, "with data, obs must be 1, 2 or 3 and sigma > 0");
    if (d->max_batch < 1)
        return fail(RD_EINVAL, "max_batch must be >= 1");
    for (int i = 0; i < 3; ++i) {
        if (d->prior_kind[i] != RD_PRIOR_UNIFORM && d->prior_kind[i] != RD_PRIOR_NORMAL)
            return fail(RD_EINVAL, "prior_kind[%d] unknown", i);
        if (d->prior_kind[i] == RD_PRIOR_NORMAL && !(d->prior_sd[i] > 0.0))
            return fail(RD_EINVAL, "prior_sd[%d] must be > 0", i);
        if (d->prior_kind[i] == RD_PRIOR_UNIFORM && !(d->lo[i] <= d->hi[i]))
            return fail(RD_EINVAL, "lo[%d] > hi[%d]", i, i);
        if (!(d->step[i] >= 0.0))
            return fail(RD_EINVAL, "step[%d] must be >= 0", i);
    }
    int device = 0;
    G1D_TRY(hipGetDevice(&device));
    g1d_problem *p = new g1d_problem;
    p->desc = *d;
    p->desc.u0 = p->desc.v0 = p->desc.y = nullptr;  // host arrays are read during the call only
    p->device = device;
    const size_t n = (size_t)d->n, mb = (size_t)d->max_batch;
    hipError_t e = hipSuccess;
    if (e == hipSuccess) e = hipMalloc(&p->u0, n * sizeof(double));
    if (e == hipSuccess) e = hipMalloc(&p->v0, n * sizeof(double));
    if (e == hipSuccess && d->y) e = hipMalloc(&p->y, 2 * n * sizeof(double));
    if (e == hipSuccess) e = hipMalloc(&p->ctr, 2 * sizeof(uint64_t));
    if (e == hipSuccess) e = hipMalloc(&p->phi_prop, 4 * mb * sizeof(double));
    if (e == hipSuccess) e = hipMalloc(&p->inside, mb * sizeof(int));
    if (e == hipSuccess) e = hipMalloc(&p->ll_prop, mb * sizeof(double));
    if (e == hipSuccess) e = hipMalloc(&p->status, mb * sizeof(int));
    if (e != hipSuccess) {
        release(p);
        delete p;
        return fail(RD_ENOMEM, "device allocation failed: %s", hipGetErrorString(e));
    }
    e = hipMemcpy(p->u0, d->u0, n * sizeof(double), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(p->v0, d->v0, n * sizeof(double), hipMemcpyHostToDevice);
    if (e == hipSuccess && d->y)
        e = hipMemcpy(p->y, d->y, 2 * n * sizeof(double), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        release(p);
        delete p;
        return fail(RD_EHIP, "copy to device failed: %s", hipGetErrorString(e));
    }
    *out = p;
    return RD_OK;
}

extern "C" int32_t g1d_destroy(g1d_problem *p)
{
    if (!p)
        return RD_OK;
    hipDeviceSynchronize();
    release(p);
    delete p;
    return RD_OK;
}

extern "C" int32_t g1d_forward_batch(g1d_problem *p, int32_t n, const double *beta, double *u,
                                     double *v, int32_t *status, void *stream)
{
    int32_t r = check_batch(p, n, beta);
    if (r != RD_OK)
        return r;
    if (n > 0 && (!u || !v))
        return fail(RD_EINVAL, "u and v are required");
    g1d::Args a = base_args(p);
    a.beta = beta;
    a.m = n;
    a.u_out = u;
    a.v_out = v;
    a.status = status;
    a.y = nullptr;
    G1D_TRY(g1d::launch_solve(a, (hipStream_t)stream));
    return RD_OK;
}

extern "C" int32_t g1d_log_likelihood_batch(g1d_problem *p, int32_t n, const double *beta,
                                            double *phi, int32_t *status, void *stream)
{
    int32_t r = check_batch(p, n, beta);
    if (r != RD_OK)
        return r;
    if (!p->y)
        return fail(RD_EINVAL, "the problem has no data y");
    if (n > 0 && !phi)
        return fail(RD_EINVAL, "phi is required");
    g1d::Args a = base_args(p);
    a.beta = beta;
    a.m = n;
    a.phi = phi;
    a.status = status;
    G1D_TRY(g1d::launch_solve(a, (hipStream_t)stream));
    return RD_OK;
}

extern "C" int32_t g1d_mcmc_step_batch(g1d_problem *p, rd_chains *c, int32_t n_steps,
                                       void *stream)
{
    if (!p)
        return fail(RD_EINVAL, "problem is NULL");
    if (!c)
        return fail(RD_EINVAL, "chains is NULL");
    if (c->n_chains < 0 || c->n_chains > p->desc.max_batch)
        return fail(RD_EINVAL, "n_chains %d outside [0, max_batch = %d]", c->n_chains,
                    p->desc.max_batch);
    if (!c->phi || !c->loglik)
        return fail(RD_EINVAL, "chains->phi and chains->loglik are required");
    if (c->trace && c->trace_rows < 0)
        return fail(RD_EINVAL, "chains->trace_rows < 0");
    if (!p->y || p->desc.law != G1D_LAW_POLY)
        return fail(RD_EINVAL, "sampling needs data y and the polynomial growth law");
    if (n_steps < 0)
        return fail(RD_EINVAL, "n_steps < 0");
    if (n_steps == 0 || c->n_chains == 0) {
        c->step += (uint64_t)n_steps;
        return RD_OK;
    }
    hipStream_t s = (hipStream_t)stream;
    const g1d_desc &d = p->desc;
    SamplerArgs sa{};
    sa.n = c->n_chains;
    sa.seed = c->seed;
    sa.ctr = p->ctr;
    sa.cfg.free_mask = 0x7u;
    sa.cfg.use_chol = 0;
    sa.cfg.any_normal = 0;
    for (int i = 0; i < 3; ++i) {
        sa.cfg.lo[i] = d.lo[i];
        sa.cfg.hi[i] = d.hi[i];
        sa.cfg.step[i] = d.step[i];
        sa.cfg.prior_kind[i] = d.prior_kind[i];
        sa.cfg.prior_mean[i] = d.prior_mean[i];
        sa.cfg.prior_sd[i] = d.prior_sd[i];
        if (d.prior_kind[i] == RD_PRIOR_NORMAL)
            sa.cfg.any_normal = 1;
    }
    // The fourth coordinate is carried unchanged and only has to lie in a
    // box that holds every value.
    sa.cfg.lo[3] = -INFINITY;
    sa.cfg.hi[3] = INFINITY;
    sa.cfg.step[3] = 0.0;
    sa.cfg.prior_kind[3] = RD_PRIOR_UNIFORM;
    sa.cfg.prior_sd[3] = 1.0;
    sa.cfg.turing = 0;
    sa.phi = c->phi;
    sa.loglik = c->loglik;
    sa.phi_prop = p->phi_prop;
    sa.theta_prop = nullptr;
    sa.inside = p->inside;
    sa.loglik_prop = p->ll_prop;
    sa.n_accept = c->n_accept;
    sa.n_solves = c->n_solves;
    sa.trace = c->trace;
    sa.trace_rows = c->trace_rows;
    g1d::Args a = base_args(p);
    a.beta = p->phi_prop;
    a.beta_stride = 4;
    a.need = p->inside;
    a.m = c->n_chains;
    a.phi = p->ll_prop;
    a.status = p->status;
    G1D_TRY(launch_set_ctr(p->ctr, c->step, c->trace_step0, s));
    for (int k = 0; k < n_steps; ++k) {
        G1D_TRY(launch_propose(sa, s));
        G1D_TRY(g1d::launch_solve(a, s));
        G1D_TRY(launch_accept(sa, s));
        G1D_TRY(launch_advance_ctr(p->ctr, s));
    }
    c->step += (uint64_t)n_steps;
    return RD_OK;
}
