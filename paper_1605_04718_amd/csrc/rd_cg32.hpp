// FP64 solve of 32x32 items by plain CG: a workgroup of four wavefronts per
// item, every array in registers.
//
// Lane l of wave w owns columns 2j, 2j + 1 (j = l % 16) of rows
// 8w + 2 (l / 16) and the next: with a row of the grid in the 16 lanes of one
// DPP row, the west and east neighbours come from row shifts, whose lanes
// without a source keep their own value (the mirror ghost).  The rows above and
// below go through LDS.
//
// Bound by the latency of one iteration, a chain of stencil, sum, division,
// update, sum, division (the 1024 cells are 4 per lane, and a chain of an MCMC
// run is one item): hence four waves rather than one or two, the sums by
// matrix instructions (four 4x4 products with ones and one trip through LDS for
// the workgroup, against six DPP steps before the trip and four after), two
// barriers per iteration instead of three (the new residual's rows are exchanged
// at the barrier of its norm, and each lane advances the direction of the rows
// beside its own by itself, with the same operations as their owner), and a
// loop with one way out, which keeps its vectors in place.
//
// Measured, us per step near the posterior (11.4 iterations) at 1 / 256 / 600 /
// 1500 items, rtol 1e-10: 9.1 / 9.3 / 16.3 / 28.5.  With p in LDS and strips of
// 8 cells per lane: 21.5 / 22.2 / 26.2 / 35.7, of 4: 18.1 / 18.6 / 25.9 / 42.8.
// 0.60 us an iteration and 1.1 us a set-up.  Three waves per SIMD (162 VGPRs);
// four spill, and with the sums by 16x16 products an item took 18 us.
#pragma once

namespace rd {
namespace cg32 {

constexpr int N = 32, NW = 4, T = NW * kWave;

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// Own cells: [row][column].
struct Cells {
    double v[2][2];
};
// Columns 2j, 2j + 1 of the rows above and below the own ones.
struct Halo {
    f64x2 n, s;
};

struct Lds {
    double x[3][N][N];  // rows of the field and of two increments (set-up)
    double r[N][N];     // rows of the residual
    double sums[7][4 * NW];  // of the set-up
    double pq[1][4 * NW], rr[1][4 * NW], last[1][4 * NW];
};

struct Ctx {
    Lds &s;
    int row, col, up, down, put_at, get_at;
    bool first;  // first lane of a 4x4 block
    __device__ explicit Ctx(Lds &lds) : s(lds)
    {
        const int lane = threadIdx.x & (kWave - 1);
        const int wave = wave_index();
        first = lane < 16 && lane % 4 == 0;
        put_at = 4 * wave + lane / 4 % 4;
        get_at = lane % 4 + 4 * (lane / 16);
        row = 8 * wave + 2 * (lane >> 4);
        col = 2 * (lane & 15);
        up = row > 0 ? row - 1 : row;  // mirror ghosts
        down = row + 2 < N ? row + 2 : row + 1;
    }
    __device__ __forceinline__ void put(double (*a)[N], const Cells &c) const
    {
#pragma unroll
        for (int k = 0; k < 2; ++k)
            *(f64x2 *)&a[row + k][col] = f64x2{c.v[k][0], c.v[k][1]};
    }
    __device__ __forceinline__ Halo halo(const double (*a)[N]) const
    {
        return Halo{*(const f64x2 *)&a[up][col], *(const f64x2 *)&a[down][col]};
    }
};

// Value of the lane before (kCtrl row_shr:1) or after (row_shl:1) in the row of
// 16; `own` where there is none.
template <int kCtrl>
__device__ __forceinline__ double beside(double own, double src)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(own), __double2loint(src), kCtrl, 0xf,
                                               0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(own), __double2hiint(src), kCtrl, 0xf,
                                               0xf, false);
    return __hiloint2double(hi, lo);
}

// As beside(), 0 where there is none.
template <int kCtrl>
__device__ __forceinline__ double shifted(double src)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(src), kCtrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(src), kCtrl, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// f(k, m, own, west, east, north, south) for each own cell.
template <typename F>
__device__ __forceinline__ void sweep(const Cells &c, const Halo &h, F &&f)
{
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const double a = c.v[k][0], b = c.v[k][1];
        const double w = beside<0x111>(a, b), e = beside<0x101>(b, a);
        const double na = k ? c.v[0][0] : h.n[0], nb = k ? c.v[0][1] : h.n[1];
        const double sa = k ? h.s[0] : c.v[1][0], sb = k ? h.s[1] : c.v[1][1];
        f(k, 0, a, w, b, na, sa);
        f(k, 1, b, a, e, nb, sb);
    }
}

// Sum of the four differences to the neighbours, -h^2 Lap_h.
__device__ __forceinline__ double diffs(double o, double w, double e, double n, double s)
{
    return ((o - w) + (o - e)) + ((o - s) + (o - n));
}

// A product of four 4x4 blocks with ones: block b (lanes with l / 4 % 4 == b)
// holds its factor's row l % 4, column l / 16, and gets row l / 16 of the
// result, so that two products leave the sum of a block's 16 lanes in each of
// them.
template <int M>
__device__ __forceinline__ void block_totals(double (&v)[M])
{
#pragma unroll
    for (int l = 0; l < 2; ++l)
#pragma unroll
        for (int m = 0; m < M; ++m)
            v[m] = __builtin_amdgcn_mfma_f64_4x4x4f64(v[m], 1.0, 0.0, 0, 0, 0);
}

// Sums over the workgroup in two halves, a barrier between them: the 16 block
// totals go to LDS, and each lane reads the one that its place in a block asks
// for.
template <int M>
__device__ __forceinline__ void put_sums(const Ctx &x, double (&v)[M], double (*slots)[4 * NW])
{
    block_totals(v);
    if (x.first)
#pragma unroll
        for (int m = 0; m < M; ++m)
            slots[m][x.put_at] = v[m];
}

template <int M>
__device__ __forceinline__ void get_sums(const Ctx &x, double (&v)[M],
                                         const double (*slots)[4 * NW])
{
#pragma unroll
    for (int m = 0; m < M; ++m)
        v[m] = slots[m][x.get_at];
    block_totals(v);
}

__device__ __forceinline__ void put_sum(const Ctx &x, double v, double (*slot)[4 * NW])
{
    double a[1] = {v};
    put_sums(x, a, slot);
}

__device__ __forceinline__ double get_sum(const Ctx &x, const double (*slot)[4 * NW])
{
    double a[1];
    get_sums(x, a, slot);
    return a[0];
}

// A condition that is the same in every lane, as a scalar.
__device__ __forceinline__ bool all_same(bool c)
{
    return __builtin_amdgcn_ballot_w64(c) != 0;
}

// 1 / d and n / d to an ulp: a reciprocal refined twice and the quotient once,
// so that the reciprocal is off the path that waits for the numerator.  Not for
// denormal d, whose reciprocal overflows: below kTiny the callers divide.
constexpr double kTiny = 1e-290;
__device__ __forceinline__ double recip(double d)
{
    double y = __builtin_amdgcn_rcp(d);
    y = fma(y, fma(-d, y, 1.0), y);
    return fma(y, fma(-d, y, 1.0), y);
}

__device__ __forceinline__ double quotient(double n, double d, double rd)
{
    const double q = n * rd;
    return fma(fma(-d, q, n), rd, q);
}

struct Species {
    double c;         // c' / h^2
    double src;       // source
    double e0;        // constant part of the reaction + dilution diagonal
    double gam;
    double inv_dt, rtol2;
    int maxit;
};

// CG for the increment d of one implicit step of species kSp (0: u, 1: v),
//   (1/dt + e) x' - c' Lap_h x' = x/dt + src,  x' = x + d,
// e from the level-n fields (e_u = 2r + g (1 - u v), e_v = 2r + g u^2), o the
// other species' field.  h1, h2: the increments of the last two steps; the start
// vector is none (npred 0), the minimal-residual step along h1 (1), or the
// Galerkin one over both (2), as in the tiled solver.  The stopping test is
// |r| <= rtol |b| on the updated residual; `quiet` tells whether the step's
// first residual met it.
template <int kSp>
__device__ __forceinline__ int cg(const Ctx &x, const Species &p, const Cells &f, const Cells &o,
                                  const Cells &h1, const Cells &h2, int npred, Cells &d,
                                  int &it_acc, int &quiet)
{
    Lds &s = x.s;
    Cells r, q1, q2, sig;
    x.put(s.x[0], f);
    if (npred >= 1)
        x.put(s.x[1], h1);
    if (npred == 2)
        x.put(s.x[2], h2);
    __syncthreads();
    double bb = 0.0, rr = 0.0;
    // r0 = b - A x = src - e x - c t(x): the 1/dt terms cancel exactly
    sweep(f, x.halo(s.x[0]), [&](int k, int m, double own, double w, double e, double n, double so) {
        const double ov = o.v[k][m];
        const double er = kSp == 0 ? fma(-p.gam, own * ov, p.e0) : fma(p.gam, ov * ov, p.e0);
        const double b = fma(own, p.inv_dt, p.src);
        const double res = fma(-p.c, diffs(own, w, e, n, so), fma(-er, own, p.src));
        sig.v[k][m] = er + p.inv_dt;
        r.v[k][m] = res;
        bb = fma(b, b, bb);
        rr = fma(res, res, rr);
    });
    auto apply = [&](const Cells &h, const double (*rows)[N], Cells &q) {
        sweep(h, x.halo(rows), [&](int k, int m, double own, double w, double e, double n,
                                   double so) {
            q.v[k][m] = fma(sig.v[k][m], own, p.c * diffs(own, w, e, n, so));
        });
    };
    auto dot = [&](const Cells &a, const Cells &b) {
        return fma(a.v[0][0], b.v[0][0], a.v[0][1] * b.v[0][1]) +
               fma(a.v[1][0], b.v[1][0], a.v[1][1] * b.v[1][1]);
    };
    double w1 = 0.0, w2 = 0.0;
    if (npred == 2) {
        apply(h1, s.x[1], q1);
        apply(h2, s.x[2], q2);
        double t[7] = {bb, rr, dot(h1, q1), dot(h2, q1), dot(h2, q2), dot(h1, r), dot(h2, r)};
        put_sums(x, t, s.sums);
        __syncthreads();
        get_sums(x, t, s.sums);
        bb = t[0];
        rr = t[1];
        const double g11 = t[2], g12 = t[3], g22 = t[4], b1 = t[5], b2 = t[6];
        const double det = g11 * g22 - g12 * g12;
        if (all_same(g11 > 0.0 && g22 > 0.0 && finite(det) && det > 1e-12 * g11 * g22 &&
                     finite(b1) && finite(b2))) {
            const double n1 = b1 * g22 - b2 * g12, n2 = b2 * g11 - b1 * g12;
            if (all_same(det > kTiny)) {
                const double rd = recip(det);
                w1 = quotient(n1, det, rd);
                w2 = quotient(n2, det, rd);
            } else {
                w1 = n1 / det;
                w2 = n2 / det;
            }
        } else if (all_same(g11 > 0.0 && finite(b1))) {
            w1 = b1 / g11;  // the pair is (nearly) dependent: h1 alone
        }
    } else if (npred == 1) {
        apply(h1, s.x[1], q1);
        double t[4] = {bb, rr, dot(r, q1), dot(q1, q1)};
        put_sums(x, t, s.sums);
        __syncthreads();
        get_sums(x, t, s.sums);
        bb = t[0];
        rr = t[1];
        if (all_same(t[3] > 0.0 && finite(t[2])))
            w1 = t[2] / t[3];
    } else {
        double t[2] = {bb, rr};
        put_sums(x, t, s.sums);
        __syncthreads();
        get_sums(x, t, s.sums);
        bb = t[0];
        rr = t[1];
    }
    const double tol2 = p.rtol2 * bb;
    quiet = !all_same(rr > tol2);
    if (!all_same(finite(bb) && finite(rr)))
        return kStNonfinite;
    double rp = 0.0;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            double dv = 0.0, rv = r.v[k][m];
            if (npred >= 1) {
                dv = w1 * h1.v[k][m];
                rv = fma(-w1, q1.v[k][m], rv);
            }
            if (npred == 2) {
                dv = fma(w2, h2.v[k][m], dv);
                rv = fma(-w2, q2.v[k][m], rv);
            }
            d.v[k][m] = dv;
            r.v[k][m] = rv;
            rp = fma(rv, rv, rp);
        }
    x.put(s.r, r);
    put_sum(x, rp, s.rr);
    __syncthreads();
    Halo ph = x.halo(s.r);
    rr = get_sum(x, s.rr);
    Cells pv = r;
    // The diagonal of the neighbour-sum form; where the row shift has no source
    // it gives 0, and the mirror ghost goes into the diagonal.
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        sig.v[k][0] += (x.col == 0 ? 3.0 : 4.0) * p.c;
        sig.v[k][1] += (x.col == N - 2 ? 3.0 : 4.0) * p.c;
    }
    int st = 0, it = 0;
    // One way out of the loop: after a breakdown the rest of its iteration
    // still runs, on a direction and an increment that nothing uses.  (rr > tol2
    // is false of a NaN.)
    bool go = all_same(rr > tol2 && finite(rr)) && p.maxit > 0;
    while (go) {
        Cells &q = q1;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const double a = pv.v[k][0], b = pv.v[k][1];
            const double na = k ? pv.v[0][0] : ph.n[0], nb = k ? pv.v[0][1] : ph.n[1];
            const double sa = k ? ph.s[0] : pv.v[1][0], sb = k ? ph.s[1] : pv.v[1][1];
            q.v[k][0] = fma(-p.c, (shifted<0x111>(b) + b) + (sa + na), sig.v[k][0] * a);
            q.v[k][1] = fma(-p.c, (a + shifted<0x101>(a)) + (sb + nb), sig.v[k][1] * b);
        }
        put_sum(x, dot(pv, q), s.pq);
        const bool tiny = !all_same(rr > kTiny);
        double rrr = recip(rr);
        RD_PIN(rrr);  // here, not after the barrier
        __syncthreads();
        const double pq = get_sum(x, s.pq);
        if (!all_same(pq > 0.0))
            st = kStBreakdown;
        if (!all_same(finite(pq)))
            st = kStNonfinite;
        const double al = tiny ? rr / pq : quotient(rr, pq, recip(pq));
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int m = 0; m < 2; ++m)
                r.v[k][m] = fma(-al, q.v[k][m], r.v[k][m]);
        x.put(s.r, r);
        put_sum(x, dot(r, r), s.rr);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                d.v[k][m] = fma(al, pv.v[k][m], d.v[k][m]);
                RD_PIN(d.v[k][m]);
            }
        __syncthreads();
        const Halo rh = x.halo(s.r);
        const double rn = get_sum(x, s.rr);
        it += st == 0;
        const double bt = tiny ? rn / rr : quotient(rn, rr, rrr);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int m = 0; m < 2; ++m)
                pv.v[k][m] = fma(bt, pv.v[k][m], r.v[k][m]);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            ph.n[m] = fma(bt, ph.n[m], rh.n[m]);
            ph.s[m] = fma(bt, ph.s[m], rh.s[m]);
        }
        rr = rn;
        go = all_same(rr > tol2 && finite(rr)) && st == 0 && it < p.maxit;
    }
    if (!st)
        st = !all_same(finite(rr)) ? kStNonfinite : all_same(rr > tol2) ? kStNotConverged : 0;
    it_acc += it;
    return st;
}

// All steps of item c (see the tiled solver for the scheme and for the
// steady-state stop).
__device__ __forceinline__ void solve_item(const SolveArgs &a, int c, const GridDev &gd, const Ctx &x)
{
    const double th[4] = {a.theta[4 * c], a.theta[4 * c + 1], a.theta[4 * c + 2],
                          a.theta[4 * c + 3]};
    const double inv_dt = 1.0 / a.dt, n2 = (double)N * N, decay = gd.decay;
    Cells u, v, du, dv, hu1 = {}, hu2 = {}, hv1 = {}, hv2 = {};
    auto each = [&](auto &&f) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int m = 0; m < 2; ++m)
                f(k, m, (x.row + k) * N + x.col + m);
    };
    each([&](int k, int m, int i) {
        u.v[k][m] = ((const double *)gd.u0)[i];
        v.v[k][m] = ((const double *)gd.v0)[i];
    });
    Species pu{0.0, th[2] * th[0], gd.dil + th[2], th[2], inv_dt, a.rtol2, a.maxit};
    Species pv{0.0, th[2] * th[1], gd.dil, th[2], inv_dt, a.rtol2, a.maxit};
    double rho_m2 = 1.0;
    int st = 0, steps = 0, itu = 0, itv = 0, quiet_u = 0, quiet_v = 0, last_u = 0, last_v = 0;
    bool steady = false;
    for (int s = 0; s < a.n_steps; ++s, rho_m2 *= decay) {
        pu.c = rho_m2 * n2;
        pv.c = th[3] * rho_m2 * n2;
        // the pair costs a second product, so it is taken only after a solve
        // of two iterations or more; none while a field does not move
        const int npu = (s == 0 || quiet_u) ? 0 : (s == 1 || last_u < 2) ? 1 : 2;
        const int npv = (s == 0 || quiet_v) ? 0 : (s == 1 || last_v < 2) ? 1 : 2;
        const int itu0 = itu, itv0 = itv;
        st = cg<0>(x, pu, u, v, hu1, hu2, npu, du, itu, quiet_u);
        if (st)
            break;
        st = cg<1>(x, pv, v, u, hv1, hv2, npv, dv, itv, quiet_v);
        if (st)
            break;
        steps = s + 1;
        double moved = 0.0;
        each([&](int k, int m, int) {
            u.v[k][m] += du.v[k][m];
            v.v[k][m] += dv.v[k][m];
            moved += du.v[k][m] * du.v[k][m] + dv.v[k][m] * dv.v[k][m];
        });
        hu2 = hu1;
        hu1 = du;
        hv2 = hv1;
        hv1 = dv;
        if (a.steady_tt > 0.0) {
            put_sum(x, moved, x.s.last);
            __syncthreads();
            const double thr = a.steady_tt * (double)N;
            steady = all_same(get_sum(x, x.s.last) < thr * thr);
            if (steady)
                break;
        }
        last_u = itu - itu0;
        last_v = itv - itv0;
    }
    if (!st && !steady && a.steady_tt > 0.0)
        st = kStNotSteady;  // the cap came first
    const size_t off = (size_t)c * a.out_stride;
    double phi = 0.0;
    each([&](int k, int m, int i) {
        if (a.u_out)
            ((double *)a.u_out)[off + i] = u.v[k][m];
        if (a.v_out)
            ((double *)a.v_out)[off + i] = v.v[k][m];
        if (a.phi && gd.y) {
            const double e = gd.y[i] - u.v[k][m];
            phi = fma(e, e, phi);
        }
    });
    if (a.phi) {
        __syncthreads();  // the step size's last readers are done
        put_sum(x, phi, x.s.last);
        __syncthreads();
        phi = get_sum(x, x.s.last);
        if (threadIdx.x == 0)
            a.phi[c] = (st != 0 || !gd.y || !finite(phi)) ? __builtin_inf() : phi * gd.inv_2s2;
    }
    if (threadIdx.x == 0) {
        a.status[c] = st;
        if (a.steps_out)
            a.steps_out[c] = steps;
        if (a.iters) {
            a.iters[2 * c] = itu;
            a.iters[2 * c + 1] = itv;
        }
    }
}

__global__ __launch_bounds__(T, 3) void k_solve_cg32(SolveArgs a)
{
    __shared__ __attribute__((aligned(16))) Lds lds;
    __shared__ int s_item;
    const Ctx x(lds);
    for (int item = next_item(a.queue, &s_item); item < a.n_items;
         item = next_item(a.queue, &s_item)) {
        const int c = uniform(a.order ? a.order[item] : item);
        if (!a.need || uniform(a.need[c])) {
            const int gid = item_grid(a, c);
            if (gid >= 0 && uniform(a.grids[gid].n) == N)
                solve_item(a, c, a.grids[gid], x);
        }
    }
}

}  // namespace cg32
}  // namespace rd
