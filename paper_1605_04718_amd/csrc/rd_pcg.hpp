// Resident FP32 solve with a spectral preconditioner (64 x 64 and 128 x 128).
//
// The increment systems (sigma + c L) d = r0 of a time step (L the 5-point
// Neumann Laplacian times h^2, sigma = 1/dt + e(x)) differ from their
// constant-coefficient mean (sbar + c L) only by the spread of the reaction
// diagonal about its mean, a few per cent to a few tens of per cent of 1/dt.
// The cosine transform (DCT-II) diagonalises that mean operator on the cell
// grid, so CG preconditioned with
//   z = Q^T [ (Q r Q^T) / (sbar + c (lam_q + lam_k)) ] Q
// reaches the tolerance in one or two iterations where plain CG needs 10 to
// 100 (condition number up to 1 + 8 c dt, 160 at 128 x 128 with d = 50 and
// dt = 2.5e-4).  The four N x N x N products of one application run on the
// matrix cores in FP16 with FP32 accumulation: a preconditioner only chooses
// the search direction, and its FP16 rounding (2^-11 relative) limits the
// contraction per iteration to about 0.05, not the accuracy of the solve.
// Residuals, increments and the operator stay FP32, dot products, step
// lengths and the stopping test FP64, and the fields FP64.
//
// Layout: one workgroup of W = N / 16 waves per item; wave w owns rows
// 16 w .. 16 w + 15, lane l the C = N / 64 columns C l .. C l + C - 1 of each
// (R = 16 C cells per thread).  Vertical neighbours are the thread's own
// registers, horizontal ones a DPP lane shift, so a stencil pass reads no
// LDS; only the rows above and below a wave's strip come from another wave.
//
// Global slot of a workgroup: the fields X_u, X_v in FP64, then the last two
// increments of each species in FP32.
//
// What bounds it (128 x 128, cycles of a 120 k-cycle IMEX step near the
// posterior): the passes over the slot's fields and increments (residuals
// 28 k, predictor 52 k, fold 13 k; 1.3 MB per step from L2 and the memory-side
// cache, 7 TB/s over the chip), not the transforms (10 k per application).
#pragma once

namespace rd {
namespace pcg {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kRows = 16;  // rows per wave: one matrix-core tile

// Reduction slots (FP64, W each): the predictor's 8 sums, then |r|^2, r.z,
// p.q and the misfit or step size.  No two consecutive reductions share one.
template <int W>
struct RedSlots {
    static constexpr int gram = 0, rr = 8 * W, rz = 9 * W, pq = 10 * W, misc = 11 * W,
                         total = 12 * W;
};

template <int N>
struct Layout {
    static constexpr int C = N / 64;      // columns per lane
    static constexpr int W = N / kRows;   // waves per item
    static constexpr int T = 64 * W;      // threads per item
    static constexpr int R = kRows * C;   // cells per thread
    static constexpr int KS = N / 32;     // 32-wide slices of a contraction
    static constexpr int SN = N + 8;      // stride of the FP16 row buffers
    static constexpr int ZN = N + 4;      // stride of the FP32 rows of z
};

// LDS of a workgroup.  qf / qt: Q and Q^T as matrix-core fragments (tile of
// 16 rows, 32-wide slice, lane, 8 values: a fragment is one conflict-free
// 16-byte read).  x, y: the FP16 arrays of the transform stages, padded so
// that the 16 rows a fragment touches start in different banks.
template <int N>
struct Lds {
    _Float16 qf[N * N];
    _Float16 qt[N * N];
    _Float16 x[N * Layout<N>::SN];
    _Float16 y[N * Layout<N>::SN];
    float lam[N];  // 2 - 2 cos(pi k / N)
    double red[RedSlots<Layout<N>::W>::total];
    int item;
};

// Lanes of one wave exchange data through LDS without a workgroup barrier:
// LDS operations of a wave complete in order, and this keeps the compiler
// from moving them across.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Ends a group of unrolled cells: nothing moves across, so the loads and
// conversions of later cells do not pile up in registers.
__device__ __forceinline__ void group_end()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// An offset whose use the compiler cannot hoist: otherwise the per-row
// addresses of every global array stay live through the time loop.
__device__ __forceinline__ int opaque(int o)
{
    asm volatile("" : "+v"(o));
    return o;
}

// Makes the values of an array opaque between two passes: otherwise the
// compiler keeps the FP64 conversions of one pass in registers for the next.
template <int R>
__device__ __forceinline__ void repin(float (&v)[R])
{
#pragma unroll
    for (int i = 0; i < R; ++i)
        RD_PIN(v[i]);
}

// Value of the lane to the west / east; zero at the wave's ends, which are
// the domain's edges.
__device__ __forceinline__ float from_west(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ float from_east(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                 0x130, 0xF, 0xF, true));
}
__device__ __forceinline__ double from_west(double v) { return dpp_f64<0x138, 0xF>(v); }
__device__ __forceinline__ double from_east(double v) { return dpp_f64<0x130, 0xF>(v); }

// Fragments of Q, Q^T and the eigenvalues (once per workgroup).
template <int N>
__device__ void init_tables(Lds<N> &s)
{
    constexpr int KS = Layout<N>::KS, T = Layout<N>::T;
    const float nrm = sqrtf(2.0f / (float)N);
    for (int t = threadIdx.x; t < N * N; t += T) {
        const int e = t & 7, l = (t >> 3) & 63, f = t >> 9;
        const int row = (f / KS) * 16 + (l & 15), col = (f % KS) * 32 + 8 * (l >> 4) + e;
        // Q[k][i] = nrm cos(pi k (2 i + 1) / 2N), row 0 scaled by 1/sqrt(2);
        // the angle is reduced exactly in integers
        const float qv = cospif((float)((row * (2 * col + 1)) % (4 * N)) / (float)(2 * N)) *
                         (row == 0 ? sqrtf(1.0f / (float)N) : nrm);
        const float tv = cospif((float)((col * (2 * row + 1)) % (4 * N)) / (float)(2 * N)) *
                         (col == 0 ? sqrtf(1.0f / (float)N) : nrm);
        s.qf[t] = (_Float16)qv;
        s.qt[t] = (_Float16)tv;
    }
    for (int k = threadIdx.x; k < N; k += T)
        s.lam[k] = 2.0f - 2.0f * cospif((float)k / (float)N);
    __syncthreads();
}

// Row r (0 .. 15) of wave w's part of z: rows 0-7 lie in the wave's own part
// of x, rows 8-15 in its part of y (both are free when z is formed).
template <int N>
__device__ __forceinline__ float *z_row(Lds<N> &s, int w, int r)
{
    _Float16 *base = (r < 8 ? s.x : s.y) + w * kRows * Layout<N>::SN;
    return (float *)base + (r & 7) * Layout<N>::ZN;
}

__device__ __forceinline__ f32x4 mfma(half8 a, half8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// One transform stage of a wave: for each of the N / 16 tiles of the table m
// the 16 x 16 product with the wave's own 16 rows a (kTableFirst: the table
// gives the result's rows, otherwise its columns), handed to f(tile, acc).
// The next tile's fragments are read during the present one's products.
template <int N, bool kTableFirst, typename F>
__device__ __forceinline__ void product(const _Float16 *m, const half8 (&a)[Layout<N>::KS], F &&f)
{
    constexpr int KS = Layout<N>::KS, NT = Layout<N>::W;
    const _Float16 *ml = m + lane_here() * 8;
    half8 b[2][KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        b[0][ks] = *(const half8 *)&ml[ks * 512];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        if (nt + 1 < NT) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                b[(nt + 1) & 1][ks] = *(const half8 *)&ml[((nt + 1) * KS + ks) * 512];
        }
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            acc = kTableFirst ? mfma(b[nt & 1][ks], a[ks], acc) : mfma(a[ks], b[nt & 1][ks], acc);
        f(nt, acc);
        group_end();
    }
}

// z = M^-1 r (own cells; the rows also stay in LDS for the neighbours after
// the caller's next barrier).  scale: power of two that brings r near 1;
// cs = c / sbar; out = 1 / (scale sbar).
//
// Every wave transforms its own 16 rows of r (stage 1), then works on its own
// 16 horizontal modes k for both vertical transforms (stages 2, 3), then on
// its own 16 rows again (stage 4), so that only the two changes of owner need
// a workgroup barrier.  A fragment holds row l % 16, columns 8 (l / 16) .. + 7
// of its slice for either operand; the result holds column l % 16, rows
// 4 (l / 16) .. + 3, and the operands are placed so that those four values
// are neighbours in the next stage's rows.
template <int N>
__device__ __forceinline__ void apply_precond(Lds<N> &s, const float (&r)[Layout<N>::R],
                                              float (&z)[Layout<N>::R], float scale, float cs,
                                              float out, int w)
{
    using L = Layout<N>;
    constexpr int C = L::C, KS = L::KS, SN = L::SN;
    const int lane = lane_here(), lr = lane & 15, lq = lane >> 4;
    _Float16 *xo = s.x + w * kRows * SN;  // own 16 rows
    _Float16 *yo = s.y + w * kRows * SN;
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
#pragma unroll
        for (int c = 0; c < C; ++c)
            xo[k * SN + lane * C + c] = (_Float16)(r[k * C + c] * scale);
        if (k % 4 == 3)
            group_end();
    }
    wave_sync();
    half8 a[KS];
    auto rows = [&](const _Float16 *x) {  // the fragments of 16 rows
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            a[ks] = *(const half8 *)&x[lr * SN + ks * 32 + lq * 8];
    };
    // stage 1: T[j][k] = sum_i r[j][i] Q[k][i], own rows j -> y[k][j]
    rows(xo);
    product<N, false>(s.qf, a, [&](int nt, f32x4 acc) {
        const half4 h = {(_Float16)acc[0], (_Float16)acc[1], (_Float16)acc[2], (_Float16)acc[3]};
        *(half4 *)&s.y[(nt * 16 + lr) * SN + w * kRows + lq * 4] = h;
    });
    __syncthreads();
    // stage 2: U[q][k] = sum_j Q[q][j] T[j][k], own modes k, divided by
    // 1 + cs (lam_q + lam_k) -> y[k][q] in place
    rows(yo);
    wave_sync();
    const float base = fmaf(cs, s.lam[w * kRows + lr], 1.0f);
    product<N, true>(s.qf, a, [&](int nt, f32x4 acc) {
        const f32x4 lam = *(const f32x4 *)&s.lam[nt * 16 + lq * 4];
        half4 h;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            h[i] = (_Float16)(acc[i] * __builtin_amdgcn_rcpf(fmaf(cs, lam[i], base)));
        *(half4 *)&yo[lr * SN + nt * 16 + lq * 4] = h;
    });
    wave_sync();
    // stage 3: V[j][k] = sum_q Q[q][j] U[q][k], own modes k -> x[j][k]
    rows(yo);
    product<N, false>(s.qt, a, [&](int nt, f32x4 acc) {
        const half4 h = {(_Float16)acc[0], (_Float16)acc[1], (_Float16)acc[2], (_Float16)acc[3]};
        *(half4 *)&s.x[(nt * 16 + lr) * SN + w * kRows + lq * 4] = h;
    });
    __syncthreads();
    // stage 4: z[j][i] = sum_k V[j][k] Q[k][i], own rows j
    rows(xo);
    wave_sync();
    float *zr = z_row<N>(s, w, lr);
    product<N, true>(s.qt, a, [&](int nt, f32x4 acc) {
        acc *= out;
        *(f32x4 *)&zr[nt * 16 + lq * 4] = acc;
    });
    wave_sync();
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const float *p = z_row<N>(s, w, k) + lane * C;
#pragma unroll
        for (int c = 0; c < C; ++c)
            z[k * C + c] = p[c];
    }
}

// f(index, own, t) for every own cell, t = sum over the neighbours of
// (own - neighbour); hs, hn: the rows below and above the strip.  The
// differences are formed, not the neighbours' sum: for a smooth p the sum's
// rounding, scaled by 4 c, is the same in many cells at once and would act on
// the smooth part of the increment (measured: relative error 1.3e-6 instead
// of 4e-8 after 100 steps of 128 x 128 prior draws).
template <int N, typename F>
__device__ __forceinline__ void stencil(const float (&p)[Layout<N>::R],
                                        const float (&hs)[Layout<N>::C],
                                        const float (&hn)[Layout<N>::C], F &&f)
{
    constexpr int C = Layout<N>::C;
    const bool east_edge = lane_here() == 63;
    float ds[C];
#pragma unroll
    for (int c = 0; c < C; ++c)
        ds[c] = p[c] - hs[c];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        float de[C];  // east neighbour - own, zero across the domain's edge
#pragma unroll
        for (int c = 0; c < C - 1; ++c)
            de[c] = p[k * C + c + 1] - p[k * C + c];
        de[C - 1] = from_east(p[k * C]) - p[k * C + C - 1];
        de[C - 1] = east_edge ? 0.0f : de[C - 1];
        const float dw = from_west(de[C - 1]);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const float own = p[k * C + c];
            const float dn = (k < kRows - 1 ? p[(k + 1) * C + c] : hn[c]) - own;
            f(k * C + c, own, ((c > 0 ? de[c - 1] : dw) - de[c]) + (ds[c] - dn));
            ds[c] = dn;
        }
        if ((k * C) % 4 == 4 - C)
            group_end();
    }
}

// Scalars of one species' system.
struct System {
    double inv_dt, c, src, e0, g;  // e = e0 - g u v (u) or e0 + g u^2 (v)
};

template <int N>
struct Ctx {
    using L = Layout<N>;
    Lds<N> &s;
    double *xs;          // X_u, X_v (slot)
    float *hs;           // increments [species][buffer]
    int w, o, os, on;    // wave, own / south / north row offsets of this lane

    __device__ double *field(int sp) const { return xs + (size_t)sp * (N * N); }
    __device__ float *h(int sp, int k) const { return hs + (size_t)(2 * sp + k) * (N * N); }

    __device__ Ctx(Lds<N> &lds, void *slot) : s(lds)
    {
        xs = (double *)slot;
        hs = (float *)(xs + 2 * N * N);
        w = wave_index();
        const int lane = threadIdx.x & 63;
        o = (w * kRows) * N + lane * L::C;
        // mirror rows at the domain's edges: the strip's own edge row
        os = w > 0 ? o - N : o;
        on = w < L::W - 1 ? o + kRows * N : o + (kRows - 1) * N;
    }
};

// Residual of the level-n field, r = src - e x - c t(x) in FP64 rounded once,
// sg = sigma = 1/dt + e, and this thread's sums of b^2, r^2 and e.  kSp = 1
// also advances u by its increment du (whose system is solved by then; the v
// system uses u of level n, which is read here for the last time) and
// records du in h_u.
template <int N, int kSp>
__device__ __forceinline__ void residual(const Ctx<N> &x, const System &y,
                                         float (&r)[Layout<N>::R], float (&sg)[Layout<N>::R],
                                         double &bb, double &rr, double &es,
                                         const float (&du)[Layout<N>::R], float *h_u)
{
    using L = Layout<N>;
    constexpr int C = L::C;
    const double *own = x.field(kSp), *oth = x.field(1 - kSp);
    double *adv = x.field(0);
    const int lane = lane_here(), o = opaque(x.o);
    double cnt[C];
#pragma unroll
    for (int c = 0; c < C; ++c)
        cnt[c] = 4.0 - (c == 0 && lane == 0 ? 1.0 : 0.0) - (c == C - 1 && lane == 63 ? 1.0 : 0.0);
    // kG rows of both fields are loaded while the kG rows before them are
    // worked on
    constexpr int kG = 4;
    double cur[C], so[C], nx[2][kG][C], ot[2][kG][C];
    auto load = [&](int k0, double (&nn)[kG][C], double (&oo)[kG][C]) {
#pragma unroll
        for (int j = 0; j < kG; ++j)
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int k = k0 + j;
                nn[j][c] = k < kRows - 1 ? own[o + (k + 1) * N + c] : own[x.on + c];
                oo[j][c] = oth[o + k * N + c];
            }
    };
#pragma unroll
    for (int c = 0; c < C; ++c) {
        cur[c] = own[o + c];
        so[c] = own[x.os + c];
    }
    load(0, nx[0], ot[0]);
    bb = rr = es = 0.0;
#pragma unroll
    for (int k0 = 0; k0 < kRows; k0 += kG) {
        const int ph = (k0 / kG) & 1;
        if (k0 + kG < kRows)
            load(k0 + kG, nx[ph ^ 1], ot[ph ^ 1]);
#pragma unroll
        for (int j = 0; j < kG; ++j) {
            const int k = k0 + j;
            const double ww = from_west(cur[C - 1]), ee = from_east(cur[0]);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const double xc = cur[c], sc = ot[ph][j][c];
                const double wv = c > 0 ? cur[c - 1] : ww;
                const double ev = c < C - 1 ? cur[c + 1] : ee;
                const double t = fma(cnt[c], xc, -((wv + ev) + (so[c] + nx[ph][j][c])));
                const double e = kSp == 0 ? fma(-y.g, xc * sc, y.e0) : fma(y.g, sc * sc, y.e0);
                const double res = fma(-y.c, t, fma(-e, xc, y.src));
                const double b = fma(xc, y.inv_dt, y.src);
                bb = fma(b, b, bb);
                rr = fma(res, res, rr);
                es += e;
                float rf = (float)res, sf = (float)(y.inv_dt + e);
                RD_PIN(rf);
                RD_PIN(sf);
                RD_PIN(bb);
                RD_PIN(rr);
                RD_PIN(es);
                if constexpr (kSp == 1) {
                    const float dk = du[k * C + c];
                    adv[o + k * N + c] = sc + (double)dk;
                    h_u[o + k * N + c] = dk;
                }
                r[k * C + c] = rf;
                sg[k * C + c] = sf;
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                so[c] = cur[c];
                cur[c] = nx[ph][j][c];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        group_end();
    }
}

// Preconditioned CG for the increment d of one species; r, sg from
// residual().  h1, h2: the increments of the last two steps; npred is the
// number of them that the start vector d0 = w1 h1 + w2 h2 uses, with the
// Galerkin weights (h_i, r0 - A d0) = 0 (the start of least energy-norm
// error over their span).  The stopping test is |r| <= rtol |b| on the
// recursively updated residual.
template <int N>
__device__ int solve(const Ctx<N> &x, const System &y, float (&r)[Layout<N>::R],
                     const float (&sg)[Layout<N>::R], float (&d)[Layout<N>::R], double bb,
                     double rr, double es, const float *h1, const float *h2, int npred,
                     double rtol2, int maxit, int &it_acc, int &quiet)
{
    using L = Layout<N>;
    using RS = RedSlots<L::W>;
    constexpr int C = L::C, R = L::R, W = L::W;
    double *red = x.s.red;
    const float cf = uniform((float)y.c);
    float p[R], q[R];
    if (npred > 0) {
        float s1[C], n1[C], s2[C], n2[C];
        double g11 = 0.0, g12 = 0.0, g22 = 0.0, b1 = 0.0, b2 = 0.0;
        const int o = opaque(x.o);
#pragma unroll
        for (int k = 0; k < kRows; ++k)
#pragma unroll
            for (int c = 0; c < C; ++c) {
                p[k * C + c] = h1[o + k * N + c];
                d[k * C + c] = 0.0f;
            }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            s1[c] = h1[x.os + c];
            n1[c] = h1[x.on + c];
            s2[c] = n2[c] = 0.0f;
        }
        if (npred > 1) {
#pragma unroll
            for (int k = 0; k < kRows; ++k)
#pragma unroll
                for (int c = 0; c < C; ++c)
                    d[k * C + c] = h2[o + k * N + c];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                s2[c] = h2[x.os + c];
                n2[c] = h2[x.on + c];
            }
        }
        stencil<N>(p, s1, n1, [&](int i, float own, float t5) {
            float w = fmaf(cf, t5, sg[i] * own);  // (A h1) at the cell
            RD_PIN(w);
            g11 = fma((double)own, (double)w, g11);
            g12 = fma((double)d[i], (double)w, g12);
            b1 = fma((double)own, (double)r[i], b1);
            RD_PIN(g11);
            RD_PIN(g12);
            RD_PIN(b1);
        });
        repin(d);
        repin(r);
        stencil<N>(d, s2, n2, [&](int i, float own, float t5) {
            float w = fmaf(cf, t5, sg[i] * own);  // (A h2) at the cell
            RD_PIN(w);
            g22 = fma((double)own, (double)w, g22);
            b2 = fma((double)own, (double)r[i], b2);
            RD_PIN(g22);
            RD_PIN(b2);
        });
        double v8[8] = {bb, rr, es, g11, g12, g22, b1, b2};
        block_sum_n<W>(v8, red + RS::gram, x.w);
        bb = v8[0];
        rr = v8[1];
        es = v8[2];
        g11 = v8[3];
        g12 = v8[4];
        g22 = v8[5];
        b1 = v8[6];
        b2 = v8[7];
        quiet = uniform((int)!(rr > rtol2 * bb));
        double w1 = 0.0, w2 = 0.0;
        const double det = g11 * g22 - g12 * g12;
        if (g11 > 0.0 && g22 > 0.0 && finite(det) && det > 1e-12 * g11 * g22 && finite(b1) &&
            finite(b2)) {
            w1 = (b1 * g22 - b2 * g12) / det;
            w2 = (b2 * g11 - b1 * g12) / det;
        } else if (g11 > 0.0 && finite(b1)) {
            w1 = b1 / g11;  // one increment only, or a (nearly) dependent pair
        }
        const float W1 = uniform((float)w1), W2 = uniform((float)w2);
        if (finite(rr)) {
            repin(p);
            repin(r);
            repin(d);
            // r0 - A d0 from the stencil of d0 itself, so that r is the
            // residual of the rounded d0 (and A h1, A h2 need no registers)
#pragma unroll
            for (int i = 0; i < R; ++i)
                d[i] = fmaf(W1, p[i], W2 * d[i]);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                s1[c] = fmaf(W1, s1[c], W2 * s2[c]);
                n1[c] = fmaf(W1, n1[c], W2 * n2[c]);
            }
            double t = 0.0;
            stencil<N>(d, s1, n1, [&](int i, float own, float t5) {
                float v = r[i] - fmaf(cf, t5, sg[i] * own);
                RD_PIN(v);
                r[i] = v;
                t = fma((double)v, (double)v, t);
                RD_PIN(t);
            });
            repin(r);
            rr = block_sum<W>(t, red + RS::rr, x.w);
        }
    } else {
        double v3[3] = {bb, rr, es};
        block_sum_n<W>(v3, red + RS::gram, x.w);
        bb = v3[0];
        rr = v3[1];
        es = v3[2];
        quiet = uniform((int)!(rr > rtol2 * bb));
#pragma unroll
        for (int i = 0; i < R; ++i)
            d[i] = 0.0f;
    }
    const double tol2 = rtol2 * bb;
    int st = (finite(bb) && finite(rr)) ? 0 : kStNonfinite;
    int it = 0;
    // mean of sigma; the preconditioner stays positive definite whatever the
    // reaction term does
    double sbar = y.inv_dt + es * (1.0 / ((double)N * N));
    if (!(sbar > 0.25 * y.inv_dt) || !finite(sbar))
        sbar = y.inv_dt;
    const float cs = uniform((float)(y.c / sbar));
    double rz_old = 1.0;
    float ps[C], pn[C];
    while (st == 0 && rr > tol2) {
        if (it >= maxit) {
            st = kStNotConverged;
            break;
        }
        // power of two near the r.m.s. residual (the FP16 stages see values
        // near 1; one coefficient can hold all of |r|, at most N)
        int ex = uniform(__builtin_amdgcn_frexp_exp(rr * (1.0 / ((double)N * N)))) >> 1;
        ex = ex < -100 ? -100 : ex > 100 ? 100 : ex;
        const float scale = ldexpf(1.0f, -ex);
        const float out = uniform((float)(ldexp(1.0, ex) / sbar));
        apply_precond<N>(x.s, r, q, scale, cs, out, x.w);  // z in q
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < R; ++i)
            t = fma((double)r[i], (double)q[i], t);
        repin(r);
        repin(q);
        const double rz = block_sum<W>(t, red + RS::rz, x.w);  // (z is visible now)
        if (!finite(rz)) {
            st = kStNonfinite;
            break;
        }
        // the neighbours' edge rows of p are formed here from their z
        const float *zs = (x.w > 0 ? z_row<N>(x.s, x.w - 1, kRows - 1) : z_row<N>(x.s, 0, 0)) +
                          (threadIdx.x & 63) * C;
        const float *zn = (x.w < W - 1 ? z_row<N>(x.s, x.w + 1, 0)
                                       : z_row<N>(x.s, W - 1, kRows - 1)) +
                          (threadIdx.x & 63) * C;
        if (it == 0) {
#pragma unroll
            for (int i = 0; i < R; ++i)
                p[i] = q[i];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                ps[c] = zs[c];
                pn[c] = zn[c];
            }
        } else {
            const float bt = uniform((float)(rz / rz_old));
#pragma unroll
            for (int i = 0; i < R; ++i)
                p[i] = fmaf(bt, p[i], q[i]);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                ps[c] = fmaf(bt, ps[c], zs[c]);
                pn[c] = fmaf(bt, pn[c], zn[c]);
            }
        }
        rz_old = rz;
        t = 0.0;
        stencil<N>(p, ps, pn, [&](int i, float own, float t5) {
            float w = fmaf(cf, t5, sg[i] * own);
            RD_PIN(w);
            q[i] = w;
            t = fma((double)own, (double)w, t);
            RD_PIN(t);
        });
        repin(p);
        repin(q);
        const double pq = block_sum<W>(t, red + RS::pq, x.w);
        if (!finite(pq)) {
            st = kStNonfinite;
            break;
        }
        if (!(pq > 0.0)) {
            st = kStBreakdown;
            break;
        }
        const float a = uniform((float)(rz / pq));
        t = 0.0;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            d[i] = fmaf(a, p[i], d[i]);
            const float v = fmaf(-a, q[i], r[i]);
            r[i] = v;
            t = fma((double)v, (double)v, t);
        }
        repin(r);
        rr = block_sum<W>(t, red + RS::rr, x.w);
        ++it;
        if (!finite(rr)) {
            st = kStNonfinite;
            break;
        }
    }
    it_acc += it;
    return st;
}

// One item: all IMEX steps, then the outputs and the misfit.
template <int N>
__device__ void solve_item(const SolveArgs &a, int c, const GridDev &gd, Lds<N> &s, void *slot)
{
    using L = Layout<N>;
    constexpr int C = L::C, R = L::R, W = L::W, NN = N * N;
    const Ctx<N> x(s, slot);
    const double th0 = a.theta[4 * c], th1 = a.theta[4 * c + 1], th2 = a.theta[4 * c + 2],
                 th3 = a.theta[4 * c + 3];
    {
        const float *u0 = (const float *)gd.u0 + x.o, *v0 = (const float *)gd.v0 + x.o;
#pragma unroll
        for (int k = 0; k < kRows; ++k)
#pragma unroll
            for (int cc = 0; cc < C; ++cc) {
                const int i = k * N + cc;  // stored as [hi | lo]
                x.field(0)[x.o + i] = (double)u0[i] + (double)u0[NN + i];
                x.field(1)[x.o + i] = (double)v0[i] + (double)v0[NN + i];
            }
    }
    __syncthreads();  // the rows of the neighbouring waves are in place
    const double inv_dt = uniform(1.0 / a.dt);
    const double decay = gd.decay;
    double rho_m2 = 1.0;
    int st = 0, steps = 0, itu = 0, itv = 0, quiet = 0;  // (bit sp)
    float r[R], sg[R], d[R];
    double bb, rr, es;
    for (int n = 0; n < a.n_steps; ++n, rho_m2 = uniform(rho_m2 * decay)) {
        // buffer n & 1 holds the increment of step n - 2 and receives this one
        const int kn = n & 1, np = n < 2 ? n : 2;
        int sp = 0;
        for (; sp < 2; ++sp) {
            System y;
            y.inv_dt = inv_dt;
            y.c = uniform((sp ? th3 : 1.0) * rho_m2 * (double)NN);
            y.src = uniform(th2 * (sp ? th1 : th0));
            y.e0 = uniform(sp ? gd.dil : gd.dil + th2);
            y.g = uniform(th2);
            if (sp == 0)
                residual<N, 0>(x, y, r, sg, bb, rr, es, d, nullptr);
            else  // (d still holds the increment of u)
                residual<N, 1>(x, y, r, sg, bb, rr, es, d, x.h(0, kn));
            int it = 0, still = 0;
            st = solve<N>(x, y, r, sg, d, bb, rr, es, x.h(sp, kn ^ 1), x.h(sp, kn),
                          (quiet >> sp) & 1 ? 0 : np, a.rtol2, a.maxit, it, still);
            quiet = (quiet & ~(1 << sp)) | (still << sp);
            itu += sp == 0 ? it : 0;
            itv += sp == 1 ? it : 0;
            if (st)
                break;
        }
        if (st) {
            if (sp == 1) {
                // the step is not taken: u goes back to level n
#pragma unroll 1
                for (int k = 0; k < kRows; ++k)
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) {
                        const int i = x.o + k * N + cc;
                        x.field(0)[i] -= (double)x.h(0, kn)[i];
                    }
            }
            break;
        }
        const int o = opaque(x.o);
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
#pragma unroll
            for (int cc = 0; cc < C; ++cc) {
                const int i = o + k * N + cc;
                const float dk = d[k * C + cc];
                x.field(1)[i] += (double)dk;
                x.h(1, kn)[i] = dk;
            }
        }
        steps = n + 1;
        if (a.steady_tt > 0.0) {
            double acc = 0.0;
#pragma unroll 1
            for (int k = 0; k < kRows; ++k)
#pragma unroll
                for (int cc = 0; cc < C; ++cc) {
                    const int i = x.o + k * N + cc;
                    const double du = x.h(0, kn)[i], dv = x.h(1, kn)[i];
                    acc += du * du + dv * dv;
                }
            const double thr = a.steady_tt * (double)N;
            if (block_sum<W>(acc, s.red + RedSlots<W>::misc, x.w) < thr * thr)
                break;
            if (n + 1 == a.n_steps)
                st = kStNotSteady;  // the cap came first
        } else {
            __syncthreads();  // the fields of this level are in place
        }
    }
    if (a.n_steps == 0 && a.steady_tt > 0.0)
        st = kStNotSteady;
    const size_t off = (size_t)c * a.out_stride;
    double sum = 0.0;
#pragma unroll 4
    for (int k = 0; k < kRows; ++k)
#pragma unroll
        for (int cc = 0; cc < C; ++cc) {
            const int i = x.o + k * N + cc;
            const double u = x.field(0)[i];
            if (a.u_out)
                ((float *)a.u_out)[off + i] = (float)u;
            if (a.v_out)
                ((float *)a.v_out)[off + i] = (float)x.field(1)[i];
            if (a.phi && gd.y) {
                const double e = gd.y[i] - u;
                sum = fma(e, e, sum);
            }
        }
    if (a.phi) {
        sum = block_sum<W>(sum, s.red + RedSlots<W>::gram, x.w);
        if (threadIdx.x == 0)
            a.phi[c] = (st != 0 || !gd.y || !finite(sum)) ? __builtin_inf() : sum * gd.inv_2s2;
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

template <int N>
__global__ __launch_bounds__(Layout<N>::T, N == 128 ? 2 : 4) void k_solve_pcg(SolveArgs a)
{
    __shared__ __attribute__((aligned(16))) Lds<N> s;
    init_tables<N>(s);
    void *slot = (char *)a.gws + (size_t)blockIdx.x * a.gws_stride;
    for (int item = next_item(a.queue, &s.item); item < a.n_items;
         item = next_item(a.queue, &s.item)) {
        const int c = uniform(a.order ? a.order[item] : item);
        if (!a.need || uniform(a.need[c])) {
            const int gid = item_grid(a, c);
            if (gid >= 0)
                solve_item<N>(a, c, a.grids[gid], s, slot);
        }
    }
}

template <int N>
constexpr size_t slot_bytes()
{
    return (size_t)N * N * (2 * sizeof(double) + 4 * sizeof(float));
}

}  // namespace pcg
}  // namespace rd
