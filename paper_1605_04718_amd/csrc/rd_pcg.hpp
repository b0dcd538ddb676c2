// Solves with a spectral preconditioner: one workgroup per item at 32 x 32,
// 64 x 64 and 128 x 128, a group of four workgroups at 256 x 256, in FP32 and
// FP64.
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
// The iteration's vectors and operator are FP32, its dot products, step
// lengths and stopping test FP64; residuals are evaluated in FP64 from FP64
// fields.  FP32 problems take the increment that this gives.  FP64 problems
// add it to an FP64 field, evaluate the residual of the implicit system for
// that field in FP64, and solve for a further correction until that true
// residual meets the tolerance (iterative refinement; the tolerance then
// bounds the evaluated residual, not a recursively updated one).  FP64 items
// that leave the range of FP32 corrections are left to plain CG in FP64
// (out_of_range).
//
// Layout: strip s of an item is K whole rows, lane l of it the C columns
// C l .. C l + C - 1 (R = K C cells per thread).  A wave is one strip, at
// 32 x 32 two.  Vertical neighbours are the thread's own
// registers, horizontal ones a DPP lane shift, so a stencil pass reads no
// LDS; only the rows above and below a wave's strip come from another wave.
//
// Global slot of a workgroup: the fields X_u, X_v in FP64, then the last two
// increments of each species in FP32.
//
// What bounds it, from counters: at 32 x 32 and 64 x 64 the issue of vector
// instructions (active in 0.95 and 0.82 of the SIMDs' cycles).  At 128 x 128,
// with every CU busy, the passes over the slots: 1.19 MB per IMEX step from the
// memory-side cache, 7.1 TB/s over the chip, where a kernel that only walks 256
// such slots, half of them written, gets 8.2 (vector instructions, 2 000 per
// wave for the set-up of a system and 1 800 per iteration, 0.53); an item alone,
// or the 64 of an FP64 batch, the latency of its passes.  512 items of 128 x 128
// near the posterior, 500 steps: 43.2 ms, plain CG 89.5; 64 FP64 items, 40
// steps: 4.38 ms, plain CG with streamed arrays 144.
#pragma once

namespace rd {
namespace pcg {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// N x N cells, W waves per workgroup, K rows per strip, G workgroups per item.
template <int N_, int W_, int K_, int G_>
struct Shape {
    static constexpr int N = N_, W = W_, K = K_, G = G_;
    static constexpr int LW = N < 64 ? N : 64;    // lanes of a strip
    static constexpr int C = N / LW;              // columns per lane
    static constexpr int R = K * C;               // cells per thread
    static constexpr int T = 64 * W;              // threads per workgroup
    static constexpr int M = N / G;               // rows of one workgroup
    static constexpr int ST = M / K;              // strips of one workgroup
    static constexpr int KS = N / 32;             // 32-wide slices of a contraction
    static constexpr int NT = N / 16;             // 16-row tiles of a table
    static constexpr int SN = N + 8;              // stride of the FP16 row buffers
    static constexpr int ZN = N + 4;              // stride of the FP32 rows of z
    static constexpr int cells = M * N;           // cells of one workgroup
    static_assert(ST * LW == T, "strips cover the workgroup");
};
// 32^2: two waves of 2 x 8 rows take 9.9 us per step for one item and 26.8 for
// 2000; one wave of 2 x 16 rows 13.5 and 26.4, four of 2 x 4 rows 8.8 and
// 33.5.  128^2: eight waves of 16 rows 43 ms for 512 items of 500 steps;
// sixteen of 8 rows, whose 128 registers do not hold a strip, 64.
using S32 = Shape<32, 2, 8, 1>;
using S64 = Shape<64, 4, 16, 1>;
using S128 = Shape<128, 8, 16, 1>;

// Reduction slots (FP64, W each): the predictor's 8 sums of each species,
// then |r|^2, r.z, p.q, the true residual of a refinement, the step size and
// the misfit.  A sum is write, barrier, read, so a wave may write the next
// sum while another still reads this one: no two consecutive reductions share
// a slot (the step size follows a true residual or |r|^2 at once).
template <int W>
struct RedSlots {
    static constexpr int gram = 0, rr = 16 * W, rz = 17 * W, pq = 18 * W, truth = 19 * W,
                         step = 20 * W, misfit = 21 * W, total = 22 * W;
};

// LDS of a workgroup.  qf / qt: Q and Q^T as matrix-core fragments (tile of
// 16 rows, 32-wide slice, lane, 8 values: a fragment is one conflict-free
// 16-byte read).  x, y: the FP16 arrays of the transform stages, padded so
// that the 16 rows a fragment touches start in different banks.
template <class S>
struct Lds {
    _Float16 qf[S::N * S::N];
    _Float16 qt[S::N * S::N];
    _Float16 x[S::N * S::SN];
    _Float16 y[S::N * S::SN];
    float lam[S::N];  // 2 - 2 cos(pi k / N)
    double red[RedSlots<S::W>::total];
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

// Values whose use the compiler cannot hoist: otherwise the per-row addresses
// of every global array stay live through the time loop.
__device__ __forceinline__ unsigned opaque(unsigned o)
{
    asm volatile("" : "+v"(o));
    return o;
}
template <typename T>
__device__ __forceinline__ T *opaque(T *p)
{
    asm volatile("" : "+s"(p));
    return p;
}

// C neighbouring values at a 32-bit lane offset (in values) from a
// wave-uniform row pointer: one access of up to 16 bytes whose address is the
// scalar row pointer plus the one lane offset.
template <int C, typename T>
__device__ __forceinline__ void load_cols(const T *row, unsigned off, T (&v)[C])
{
    constexpr int V = C * sizeof(T) > 16 ? 16 / sizeof(T) : C;
    typedef T vec __attribute__((ext_vector_type(V)));
    typedef __attribute__((address_space(1))) vec gvec;  // (global, not flat)
#pragma unroll
    for (int c = 0; c < C; c += V) {
        const vec t = *(const gvec *)((const char *)(row + c) + off * (unsigned)sizeof(T));
#pragma unroll
        for (int j = 0; j < V; ++j)
            v[c + j] = t[j];
    }
}
template <int C, typename T>
__device__ __forceinline__ void store_cols(T *row, unsigned off, const T (&v)[C])
{
    constexpr int V = C * sizeof(T) > 16 ? 16 / sizeof(T) : C;
    typedef T vec __attribute__((ext_vector_type(V)));
    typedef __attribute__((address_space(1))) vec gvec;  // (global, not flat)
#pragma unroll
    for (int c = 0; c < C; c += V) {
        vec t;
#pragma unroll
        for (int j = 0; j < V; ++j)
            t[j] = v[c + j];
        *(gvec *)((char *)(row + c) + off * (unsigned)sizeof(T)) = t;
    }
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

// Value of the lane to the west / east (zero at the wave's ends).
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

// Sums of up to four values over a wave at once: exchanging halves, then
// quarters, between pairs of values leaves row m of the wave (lanes 16 m ..)
// with the partial sums of value {0, 2, 1, 3}[m], and four row shifts add
// them up in the row's last lane: 21 instructions for four values, where one
// value alone takes 18.
__device__ __forceinline__ double swap_add32(double a, double b)
{
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi =
        __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) +
           __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
}
__device__ __forceinline__ double swap_add16(double a, double b)
{
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi =
        __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) +
           __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
}

// The wave's totals of M values into slot[M][W].
template <int W, int M>
__device__ __forceinline__ void wave_totals(const double (&v)[M], double *slot, int w)
{
    const int lane = lane_here(), row = lane >> 4;
    if constexpr (M < 3) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const double t = wave_sum_last_lane(v[m]);
            if (lane == kLastLane)
                slot[m * W + w] = t;
        }
    } else {
        const int m = row == 1 ? 2 : row == 2 ? 1 : row;
#pragma unroll
        for (int m0 = 0; m0 < M; m0 += 4) {
            const double a = swap_add32(v[m0], m0 + 1 < M ? v[m0 + 1] : 0.0);
            const double b = swap_add32(m0 + 2 < M ? v[m0 + 2] : 0.0, m0 + 3 < M ? v[m0 + 3] : 0.0);
            double t = swap_add16(a, b);
            t += dpp_f64<0x111, 0xF>(t);  // row_shr:1, 2, 4, 8
            t += dpp_f64<0x112, 0xF>(t);
            t += dpp_f64<0x114, 0xF>(t);
            t += dpp_f64<0x118, 0xF>(t);
            if ((lane & 15) == 15 && m0 + m < M)
                slot[(m0 + m) * W + w] = t;
        }
    }
}

// Workgroup sums of M values; every wave gets them in the same order of
// additions.
template <int W, int M>
__device__ __forceinline__ void group_sum(double (&v)[M], double *slot, int w)
{
    wave_totals<W>(v, slot, w);
    __syncthreads();
    slots_sum<W>(v, slot);
}

// Q[k][i] = nrm cos(pi k (2 i + 1) / 2N), row 0 scaled by 1/sqrt(2); the
// angle is reduced exactly in integers.
template <int N>
__device__ __forceinline__ float dct(int k, int i)
{
    return cospif((float)((k * (2 * i + 1)) % (4 * N)) / (float)(2 * N)) *
           sqrtf((k == 0 ? 1.0f : 2.0f) / (float)N);
}

// Row and column of value t of a table in fragment order.
template <class S>
__device__ __forceinline__ void fragment_entry(int t, int &row, int &col)
{
    const int e = t & 7, l = (t >> 3) & 63, f = t >> 9;
    row = (f / S::KS) * 16 + (l & 15);
    col = (f % S::KS) * 32 + 8 * (l >> 4) + e;
}

// Fragments of Q, Q^T and the eigenvalues (once per workgroup).
template <class S>
__device__ void init_tables(Lds<S> &s)
{
    for (int t = threadIdx.x; t < S::N * S::N; t += S::T) {
        int row, col;
        fragment_entry<S>(t, row, col);
        s.qf[t] = (_Float16)dct<S::N>(row, col);
        s.qt[t] = (_Float16)dct<S::N>(col, row);
    }
    for (int k = threadIdx.x; k < S::N; k += S::T)
        s.lam[k] = 2.0f - 2.0f * cospif((float)k / (float)S::N);
    __syncthreads();
}

// Row j of z: of the 16 rows of a tile the first 8 lie in the tile's own
// part of x, the others in its part of y (both are free when z is formed).
template <class S>
__device__ __forceinline__ float *z_row(Lds<S> &s, int j)
{
    _Float16 *base = (j & 8 ? s.y : s.x) + (j >> 4) * 16 * S::SN;
    return (float *)base + (j & 7) * S::ZN;
}

__device__ __forceinline__ f32x4 mfma(half8 a, half8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ half4 to_half(f32x4 v)
{
    return half4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
}

// One transform stage of a wave: for each of the table's tiles the 16 x 16
// product with the wave's 16 rows a (kTableFirst: the table gives the
// result's rows, otherwise its columns), handed to f(tile, acc).  The next
// tile's fragments are read during the present one's products.
template <class S, bool kTableFirst, typename F>
__device__ __forceinline__ void product(const _Float16 *m, const half8 (&a)[S::KS], F &&f)
{
    constexpr int KS = S::KS, NT = S::NT;
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

// What a thread knows of its place and its item's arrays.
template <class S>
struct Ctx {
    using Sh = S;
    Lds<S> &s;
    double *xs;       // fields (slot)
    float *hs;        // increments [species][buffer]
    int w;            // wave
    unsigned o;       // this lane's offset from row(k) of its wave
    unsigned os, on;  // offsets of the rows below and above the strip

    __device__ Ctx(Lds<S> &lds, void *slot, int n_fields) : s(lds)
    {
        xs = (double *)slot;
        hs = (float *)(xs + (size_t)n_fields * S::cells);
        w = wave_index();
        const int st = strip(), col = lane() * S::C;
        o = S::LW == 64 ? col : (st % (64 / S::LW)) * S::K * S::N + col;
        // mirror rows at the domain's edges: the strip's own edge row
        os = (st > 0 ? st * S::K - 1 : 0) * S::N + col;
        on = (st < S::ST - 1 ? (st + 1) * S::K : S::M - 1) * S::N + col;
    }
    // Offset of row k of this wave('s first strip) in an array.
    __device__ int row(int k) const { return (w * (64 / S::LW) * S::K + k) * S::N; }
    __device__ int strip() const { return S::LW == 64 ? w : (int)threadIdx.x / S::LW; }
    __device__ int lane() const { return (int)threadIdx.x % S::LW; }
    __device__ double *field(int k) const { return opaque(xs + (size_t)k * S::cells); }
    __device__ float *h(int sp, int k) const { return opaque(hs + (size_t)(2 * sp + k) * S::cells); }
    __device__ size_t cell0() const { return 0; }  // first cell of the workgroup's rows

    // Sums over the item's threads; also a barrier of the item.
    template <int M>
    __device__ void sum(double (&v)[M], int slot)
    {
        group_sum<S::W>(v, s.red + slot, w);
    }
    __device__ double sum1(double v, int slot)
    {
        double t[1] = {v};
        sum(t, slot);
        return t[0];
    }
    __device__ void sync() { __syncthreads(); }
    __device__ bool failed() const { return false; }
    __device__ bool leader() const { return threadIdx.x == 0; }
    // Rows below and above the strip of a field, an increment, and z.
    __device__ void halo(int k, double (&lo)[S::C], double (&hi)[S::C]) const
    {
        load_cols(field(k), opaque(os), lo);
        load_cols(field(k), opaque(on), hi);
    }
    __device__ void halo(int sp, int k, float (&lo)[S::C], float (&hi)[S::C]) const
    {
        load_cols(h(sp, k), opaque(os), lo);
        load_cols(h(sp, k), opaque(on), hi);
    }
    __device__ void halo_z(float (&lo)[S::C], float (&hi)[S::C]) const
    {
        const int st = strip(), l = lane() * S::C;
        const float *a = z_row<S>(s, st > 0 ? st * S::K - 1 : 0) + l;
        const float *b = z_row<S>(s, st < S::ST - 1 ? (st + 1) * S::K : S::N - 1) + l;
#pragma unroll
        for (int c = 0; c < S::C; ++c) {
            lo[c] = a[c];
            hi[c] = b[c];
        }
    }
    // z = r (no preconditioner)
    __device__ void set_z(const float (&r)[S::R]) const
    {
#pragma unroll
        for (int k = 0; k < S::K; ++k)
#pragma unroll
            for (int c = 0; c < S::C; ++c)
                z_row<S>(s, strip() * S::K + k)[lane() * S::C + c] = r[k * S::C + c];
    }
    // A group of workgroups also hands its edge rows to its neighbours.
    __device__ void put_edge(int, int, const double (&)[S::C]) const {}
    __device__ void put_edge(int, int, int, const float (&)[S::C]) const {}
    __device__ void put_edge_z(const float (&)[S::R]) const {}
};

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
template <class S>
__device__ __forceinline__ void apply_precond(const Ctx<S> &x, const float (&r)[S::R],
                                              float (&z)[S::R], float scale, float cs, float out)
{
    constexpr int C = S::C, KS = S::KS, SN = S::SN;
    static_assert(S::NT == S::W, "one row tile per wave");
    Lds<S> &s = x.s;
    const int lane = lane_here(), lr = lane & 15, lq = lane >> 4;
    const int st = x.strip();
    {
        _Float16 *xo = s.x + st * S::K * SN + x.lane() * C;
#pragma unroll
        for (int k = 0; k < S::K; ++k) {
#pragma unroll
            for (int c = 0; c < C; ++c)
                xo[k * SN + c] = (_Float16)(r[k * C + c] * scale);
            if (k % 4 == 3)
                group_end();
        }
    }
    wave_sync();
    half8 a[KS];
    auto rows = [&](const _Float16 *p) {  // the fragments of 16 rows
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            a[ks] = *(const half8 *)&p[lr * SN + ks * 32 + lq * 8];
    };
    const int t0 = x.w * 16;
    // stage 1: T[j][k] = sum_i r[j][i] Q[k][i], own rows j -> y[k][j]
    rows(s.x + t0 * SN);
    product<S, false>(s.qf, a, [&](int nt, f32x4 acc) {
        *(half4 *)&s.y[(nt * 16 + lr) * SN + t0 + lq * 4] = to_half(acc);
    });
    __syncthreads();
    // stage 2: U[q][k] = sum_j Q[q][j] T[j][k], own modes k, divided by
    // 1 + cs (lam_q + lam_k) -> y[k][q] in place
    rows(s.y + t0 * SN);
    wave_sync();
    const float base = fmaf(cs, s.lam[t0 + lr], 1.0f);
    product<S, true>(s.qf, a, [&](int nt, f32x4 acc) {
        const f32x4 lam = *(const f32x4 *)&s.lam[nt * 16 + lq * 4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            acc[i] *= __builtin_amdgcn_rcpf(fmaf(cs, lam[i], base));
        *(half4 *)&s.y[(t0 + lr) * SN + nt * 16 + lq * 4] = to_half(acc);
    });
    wave_sync();
    // stage 3: V[j][k] = sum_q Q[q][j] U[q][k], own modes k -> x[j][k]
    rows(s.y + t0 * SN);
    product<S, false>(s.qt, a, [&](int nt, f32x4 acc) {
        *(half4 *)&s.x[(nt * 16 + lr) * SN + t0 + lq * 4] = to_half(acc);
    });
    __syncthreads();
    // stage 4: z[j][i] = sum_k V[j][k] Q[k][i], own rows j
    rows(s.x + t0 * SN);
    wave_sync();
    float *zr = z_row<S>(s, t0 + lr);
    product<S, true>(s.qt, a, [&](int nt, f32x4 acc) {
        acc *= out;
        *(f32x4 *)&zr[nt * 16 + lq * 4] = acc;
    });
    wave_sync();
#pragma unroll
    for (int k = 0; k < S::K; ++k) {
        const float *p = z_row<S>(s, st * S::K + k) + x.lane() * C;
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
// of 2.5e-8 after 100 steps of 128 x 128 prior draws).
template <class S, typename F>
__device__ __forceinline__ void stencil(const float (&p)[S::R], const float (&hs)[S::C],
                                        const float (&hn)[S::C], F &&f)
{
    constexpr int C = S::C, K = S::K;
    const bool east_edge = (lane_here() & (S::LW - 1)) == S::LW - 1;
    float ds[C];
#pragma unroll
    for (int c = 0; c < C; ++c)
        ds[c] = p[c] - hs[c];
#pragma unroll
    for (int k = 0; k < K; ++k) {
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
            const float dn = (k < K - 1 ? p[(k + 1) * C + c] : hn[c]) - own;
            f(k * C + c, own, ((c > 0 ? de[c - 1] : dw) - de[c]) + (ds[c] - dn));
            ds[c] = dn;
        }
        if ((k * C) % 4 == 4 - C || C == 4)
            group_end();
    }
}

// Scalars of one species' system.
struct System {
    double inv_dt, c, src, e0, g;  // e = e0 - g u v (u) or e0 + g u^2 (v)
};

// Residual of the level-n field, r = src - e x - c t(x) in FP64 rounded once,
// sg = sigma = 1/dt + e, and this thread's sums of b^2, r^2 and e.
// fo, ft: field buffers of this species and of the other one.
// kAdvance: the other species is one increment d behind (its system of the
// step that it belongs to is solved; u of level n is read here for the last
// time in the v system, v is first read at its new level in the next u
// system): it is advanced on the way, and d recorded in increment buffer hb.
template <int kSp, bool kAdvance, class X>
__device__ __forceinline__ void residual(const X &x, const System &y, int fo, int ft,
                                         float (&r)[X::Sh::R], float (&sg)[X::Sh::R], double &bb,
                                         double &rr, double &es, const float (&d)[X::Sh::R],
                                         int hb)
{
    using S = typename X::Sh;
    constexpr int C = S::C, N = S::N, K = S::K, R = S::R;
    const double *own = x.field(fo) + x.row(0);
    double *oth = x.field(ft) + x.row(0);
    float *hd = x.h(1 - kSp, hb) + x.row(0);
    const int lane = lane_here() & (S::LW - 1);
    const unsigned o = opaque(x.o);
    double cnt[C];
#pragma unroll
    for (int c = 0; c < C; ++c)
        cnt[c] = 4.0 - (c == 0 && lane == 0 ? 1.0 : 0.0) -
                 (c == C - 1 && lane == S::LW - 1 ? 1.0 : 0.0);
    // kG rows of both fields are loaded while the kG rows before them are
    // worked on
    constexpr int kG = K <= 4 || R <= 16 || C >= 4 ? 2 : 4;
    double cur[C], so[C], last[C], nx[2][kG][C], ot[2][kG][C];
    auto load = [&](int k0, double (&nn)[kG][C], double (&oo)[kG][C]) {
#pragma unroll
        for (int j = 0; j < kG; ++j) {
            const int k = k0 + j;
            if (k < K - 1) {
                load_cols(own + (k + 1) * N, o, nn[j]);
            } else {
#pragma unroll
                for (int c = 0; c < C; ++c)
                    nn[j][c] = last[c];
            }
            load_cols(oth + k * N, o, oo[j]);
        }
    };
    x.halo(fo, so, last);
    load_cols(own, o, cur);
    load(0, nx[0], ot[0]);
    bb = rr = es = 0.0;
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += kG) {
        const int ph = (k0 / kG) & 1;
        if (k0 + kG < K)
            load(k0 + kG, nx[ph ^ 1], ot[ph ^ 1]);
#pragma unroll
        for (int j = 0; j < kG; ++j) {
            const int k = k0 + j;
            double ww = from_west(cur[C - 1]), ee = from_east(cur[0]);
            if constexpr (S::LW < 64) {  // the strips of a wave are not neighbours here
                ww = lane == 0 ? 0.0 : ww;
                ee = lane == S::LW - 1 ? 0.0 : ee;
            }
            double xn[C];
            float dk[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int i = k * C + c;
                double xc = cur[c], sc = ot[ph][j][c];
                dk[c] = d[i];
                if constexpr (kAdvance && kSp == 0)  // v is read at its new level
                    sc += (double)dk[c];
                const double wv = c > 0 ? cur[c - 1] : ww;
                const double ev = c < C - 1 ? cur[c + 1] : ee;
                const double t = fma(cnt[c], xc, -((wv + ev) + (so[c] + nx[ph][j][c])));
                const double e = kSp == 0 ? fma(-y.g, xc * sc, y.e0) : fma(y.g, sc * sc, y.e0);
                const double res = fma(-y.c, t, fma(-e, xc, y.src));
                const double b = fma(xc, y.inv_dt, y.src);
                bb = fma(b, b, bb);
                rr = fma(res, res, rr);
                if (c == 0)  // (any good mean of sigma will do)
                    es += e;
                float rf = (float)res, sf = (float)(y.inv_dt + e);
                RD_PIN(rf);
                RD_PIN(sf);
                RD_PIN(bb);
                RD_PIN(rr);
                RD_PIN(es);
                if constexpr (kAdvance)
                    xn[c] = kSp == 0 ? sc : sc + (double)dk[c];
                r[i] = rf;
                sg[i] = sf;
            }
            if constexpr (kAdvance) {
                store_cols(oth + k * N, o, xn);
                store_cols(hd + k * N, o, dk);
                if (k == 0 || k == K - 1) {
                    x.put_edge(ft, k, xn);
                    x.put_edge(1 - kSp, hb, k, dk);
                }
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

// Own cells of a slot array.
template <class X>
__device__ __forceinline__ void load_strip(const X &x, const float *a, float (&v)[X::Sh::R])
{
    using S = typename X::Sh;
    const float *row = a + x.row(0);
    const unsigned o = opaque(x.o);
#pragma unroll
    for (int k = 0; k < S::K; ++k) {
        float t[S::C];
        load_cols(row + k * S::N, o, t);
#pragma unroll
        for (int c = 0; c < S::C; ++c)
            v[k * S::C + c] = t[c];
    }
}

// The scalars of one solve that its passes share.
struct Scalars {
    double bb, rr, sbar, rtol2, floor2;
    int maxit, it;
};

// Start vector d0 = w1 h1 + w2 h2 from the increments of the last two steps
// (npred of them), with the Galerkin weights (h_i, r0 - A d0) = 0: the start
// of least energy-norm error over their span.  r becomes the residual of d0.
// On entry bb, rr hold this thread's sums and es its sum of e; on return v
// holds the item's.  `quiet`: r0 itself met the tolerance.
template <class X>
__device__ __forceinline__ void start(X &x, const System &y, int sp, int kn, int npred,
                                      float (&r)[X::Sh::R], const float (&sg)[X::Sh::R],
                                      float (&d)[X::Sh::R], double es, Scalars &v, int &quiet)
{
    using S = typename X::Sh;
    using RS = RedSlots<S::W>;
    constexpr int C = S::C, R = S::R, K = S::K, N = S::N;
    const float cf = uniform((float)y.c);
    if (npred > 0) {
        float p[R], s1[C], n1[C], s2[C], n2[C];
        double g11 = 0.0, g12 = 0.0, g22 = 0.0, b1 = 0.0, b2 = 0.0;
        load_strip(x, x.h(sp, kn ^ 1), p);
#pragma unroll
        for (int i = 0; i < R; ++i)
            d[i] = 0.0f;
        x.halo(sp, kn ^ 1, s1, n1);
#pragma unroll
        for (int c = 0; c < C; ++c)
            s2[c] = n2[c] = 0.0f;
        if (npred > 1) {
            load_strip(x, x.h(sp, kn), d);
            x.halo(sp, kn, s2, n2);
        }
        stencil<S>(p, s1, n1, [&](int i, float own, float t5) {
            float w = fmaf(cf, t5, sg[i] * own);  // (A h1) at the cell
            RD_PIN(w);
            g11 = fma((double)own, (double)w, g11);
            g12 = fma((double)d[i], (double)w, g12);
            b1 = fma((double)own, (double)r[i], b1);
            b2 = fma((double)d[i], (double)r[i], b2);
            RD_PIN(g11);
            RD_PIN(g12);
            RD_PIN(b1);
            RD_PIN(b2);
        });
        repin(d);
        repin(r);
        stencil<S>(d, s2, n2, [&](int i, float own, float t5) {
            float w = fmaf(cf, t5, sg[i] * own);  // (A h2) at the cell
            RD_PIN(w);
            g22 = fma((double)own, (double)w, g22);
            RD_PIN(g22);
        });
        double v8[8] = {v.bb, v.rr, es, g11, g12, g22, b1, b2};
        x.sum(v8, RS::gram + 8 * sp * S::W);
        v.bb = v8[0];
        v.rr = v8[1];
        es = v8[2];
        g11 = v8[3];
        g12 = v8[4];
        g22 = v8[5];
        b1 = v8[6];
        b2 = v8[7];
        quiet = uniform((int)!(v.rr > v.rtol2 * v.bb));
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
        if (finite(v.rr)) {
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
            stencil<S>(d, s1, n1, [&](int i, float own, float t5) {
                float w = r[i] - fmaf(cf, t5, sg[i] * own);
                RD_PIN(w);
                r[i] = w;
                t = fma((double)w, (double)w, t);
                RD_PIN(t);
            });
            repin(r);
            v.rr = x.sum1(t, RS::rr);
        }
    } else {
        double v3[3] = {v.bb, v.rr, es};
        x.sum(v3, RS::gram + 8 * sp * S::W);
        v.bb = v3[0];
        v.rr = v3[1];
        es = v3[2];
        quiet = uniform((int)!(v.rr > v.rtol2 * v.bb));
#pragma unroll
        for (int i = 0; i < R; ++i)
            d[i] = 0.0f;
    }
    // mean of sigma; the preconditioner stays positive definite whatever the
    // reaction term does
    v.sbar = y.inv_dt + es * (1.0 / ((double)N * S::LW));
    if (!(v.sbar > 0.25 * y.inv_dt) || !finite(v.sbar))
        v.sbar = y.inv_dt;
}

// Preconditioned CG: d += A^-1 r until |r|^2 <= stop2 (r is updated
// recursively).  Returns RD status bits; st, if it is set, before any iteration.
template <class X>
__device__ __forceinline__ int pcg(X &x, const System &y, float (&r)[X::Sh::R],
                                   const float (&sg)[X::Sh::R], float (&d)[X::Sh::R],
                                   double stop2, Scalars &v, int st = 0)
{
    using S = typename X::Sh;
    using RS = RedSlots<S::W>;
    constexpr int C = S::C, R = S::R, N = S::N;
    const float cf = uniform((float)y.c);
    const float cs = uniform((float)(y.c / v.sbar));
    // The stiffest mode leaves stage 2 divided by 1 + 8 cs.  Where that takes
    // it below the normal FP16 numbers (2^-14), the stages run scaled up by
    // 2^kHead, which puts the largest value, N times the r.m.s. one, just below
    // the largest FP16, and the iteration converges up to 8 c dt = 3e7, as far
    // as plain CG in FP32 does; without it, from 3e7 on (at 1e7 in 21 to 90
    // iterations) it does not.
    constexpr int kHead = N == 32 ? 10 : N == 64 ? 9 : N == 128 ? 8 : 7;
    constexpr int kStiff = 0x45000000;  // the bits of 2048.0f
    float p[R], q[R], ps[C], pn[C];
    double rz_old = 1.0;
    st = (finite(v.bb) && finite(v.rr)) || st ? st : kStNonfinite;
    bool first = true;
    while (st == 0 && v.rr > stop2) {
        if (x.failed()) {
            st = kStGroupTimeout;
            break;
        }
        if (v.it >= v.maxit) {
            st = kStNotConverged;
            break;
        }
        // power of two near the r.m.s. residual (the FP16 stages see values
        // near 1; one coefficient can hold all of |r|, at most N), less head
        int ex = uniform(__builtin_amdgcn_frexp_exp(v.rr * (1.0 / ((double)N * N)))) >> 1;
        ex = (ex < -100 ? -100 : ex > 100 ? 100 : ex) -
             (__float_as_int(cs) > kStiff ? kHead : 0);
        const float scale = ldexpf(1.0f, -ex);
        const float out = uniform((float)(ldexp(1.0, ex) / v.sbar));
        if (v.maxit >= kPlainCap) {
            apply_precond(x, r, q, scale, cs, out);  // z in q
        } else {
            x.set_z(r);
#pragma unroll
            for (int i = 0; i < R; ++i)
                q[i] = r[i];
        }
        x.put_edge_z(q);
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < R; ++i)
            t = fma((double)r[i], (double)q[i], t);
        repin(r);
        repin(q);
        const double rz = x.sum1(t, RS::rz);  // (z is visible now)
        if (!finite(rz)) {
            st = kStNonfinite;
            break;
        }
        // the neighbours' edge rows of p are formed here from their z
        float zs[C], zn[C];
        x.halo_z(zs, zn);
        if (first) {
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
        first = false;
        rz_old = rz;
        t = 0.0;
        stencil<S>(p, ps, pn, [&](int i, float own, float t5) {
            float w = fmaf(cf, t5, sg[i] * own);
            RD_PIN(w);
            q[i] = w;
            t = fma((double)own, (double)w, t);
            RD_PIN(t);
        });
        repin(p);
        repin(q);
        const double pq = x.sum1(t, RS::pq);
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
            const float w = fmaf(-a, q[i], r[i]);
            r[i] = w;
            t = fma((double)w, (double)w, t);
        }
        repin(r);
        v.rr = x.sum1(t, RS::rr);
        ++v.it;
        if (!finite(v.rr))
            st = kStNonfinite;
    }
    if (x.failed())
        st = kStGroupTimeout;
    return st;
}

// FP64 problems: a system that the FP32 corrections cannot be relied on for,
// because the right-hand side's size leaves their range (with it the residuals,
// 1e-15 as large, and the products of the fields in sigma), or because it is so
// stiff that the preconditioner helps little and the FP32 operator's rounding
// reaches the smooth part.  Such items are solved again from the start by plain
// CG in FP64.  Measured at rtol 1e-12, iterations of two steps of 64 x 64, 128 x
// 128 and 256 x 256 from rough fields, here | plain: 8 c dt = 1e6 57, 47, 57 |
// 1100 to 4000; 1e7 235, 122, 157; 3e7 623, 432, 279; 1e8 more than 4000.
template <class S>
__device__ __forceinline__ bool out_of_range(const System &y, const Scalars &v)
{
    constexpr double cells = (double)S::N * S::N;
    return finite(v.bb) && v.bb > 0.0 &&
           (v.bb < 0x1p-80 * cells || v.bb > 0x1p80 * cells || 8.0 * y.c > 0x1p24 * v.sbar);
}

// FP64 problems.  Adds the correction d to the new field fn (kFirst: to the
// level-n field fo) and to the increment in buffer hb.
template <class X>
__device__ __forceinline__ void correct(const X &x, int sp, int fo, int fn, bool first,
                                        const float (&d)[X::Sh::R], int hb)
{
    using S = typename X::Sh;
    constexpr int C = S::C, N = S::N;
    const double *from = x.field(first ? fo : fn) + x.row(0);
    double *to = x.field(fn) + x.row(0);
    float *hd = x.h(sp, hb) + x.row(0);
    const unsigned o = opaque(x.o);
#pragma unroll
    for (int k = 0; k < S::K; ++k) {
        double yn[C];
        float hn[C];
        load_cols(from + k * N, o, yn);
        if (first) {
#pragma unroll
            for (int c = 0; c < C; ++c)
                hn[c] = 0.0f;
        } else {
            load_cols(hd + k * N, o, hn);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            yn[c] += (double)d[k * C + c];
            hn[c] += d[k * C + c];
        }
        store_cols(to + k * N, o, yn);
        store_cols(hd + k * N, o, hn);
        if (k == 0 || k == S::K - 1) {
            x.put_edge(fn, k, yn);
            x.put_edge(sp, hb, k, hn);
        }
        if (k % 4 == 3)
            group_end();
    }
}

// FP64 problems: residual of the implicit system for the new field,
// r = src + (x - x') / dt - e x' - c t(x'), e from the level-n fields, and
// this thread's sum of r^2.
template <class X>
__device__ __forceinline__ double true_residual(const X &x, const System &y, int sp, int fo, int ft,
                                                int fn, float (&r)[X::Sh::R])
{
    using S = typename X::Sh;
    constexpr int C = S::C, N = S::N, K = S::K;
    const double *nw = x.field(fn) + x.row(0), *own = x.field(fo) + x.row(0),
                 *oth = x.field(ft) + x.row(0);
    const int lane = lane_here() & (S::LW - 1);
    const unsigned o = opaque(x.o);
    double cur[C], so[C], last[C], rr = 0.0;
    x.halo(fn, so, last);
    load_cols(nw, o, cur);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        double no[C], xos[C], scs[C];
        load_cols(own + k * N, o, xos);
        load_cols(oth + k * N, o, scs);
        if (k < K - 1) {
            load_cols(nw + (k + 1) * N, o, no);
        } else {
#pragma unroll
            for (int c = 0; c < C; ++c)
                no[c] = last[c];
        }
        const double ww = from_west(cur[C - 1]), ee = from_east(cur[0]);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const double xo = xos[c], sc = scs[c], xc = cur[c];
            const double dw = c > 0 ? xc - cur[c - 1] : lane == 0 ? 0.0 : xc - ww;
            const double de = c < C - 1 ? xc - cur[c + 1] : lane == S::LW - 1 ? 0.0 : xc - ee;
            const double t = (dw + de) + ((xc - so[c]) + (xc - no[c]));
            const double e = sp == 0 ? fma(-y.g, xo * sc, y.e0) : fma(y.g, sc * sc, y.e0);
            double res = fma(-y.c, t, fma(-e, xc, fma(xo - xc, y.inv_dt, y.src)));
            rr = fma(res, res, rr);
            float rf = (float)res;
            RD_PIN(rf);
            RD_PIN(rr);
            r[k * C + c] = rf;
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            so[c] = cur[c];
            cur[c] = no[c];
        }
        if (k % 4 == 3)
            group_end();
    }
    return rr;
}

// Squared tolerance of an FP64 system.  A residual of the preconditioned
// iteration is smooth where plain CG's is rough, and the same norm of it
// stands for a larger error of the field (A is 1/dt on the smooth part, up to
// 8 c on the rough one): a twentieth of the caller's tolerance gives the
// accuracy that plain CG had at it, but not below the rounding of the
// evaluated residual (squared, of |b|: a field of the size of the present one,
// rounded to FP64, through the operator, 2^-53 (1 + 8 c dt) / 2, a few times).
__device__ __forceinline__ double fp64_floor2(double c_dt)
{
    return 6.4e-29 * (1.0 + c_dt) * (1.0 + c_dt);
}
__device__ __forceinline__ double fp64_rtol2(double rtol2, double floor2)
{
    return fmax(0.0025 * rtol2, fmin(rtol2, floor2));
}

// FP32 problems: the residual that u is solved to.  As above, and the smooth
// error shows in u, whose operator is the weaker one; half the tolerance takes
// it below plain CG's, down to 1e-8, from where the FP32 output's rounding
// covers it.  Measured, relative error of u against 64 bits, 12 sets of 10
// prior draws of 32 x 32, 446 steps, rtol 1e-7: plain CG 6.4e-7 to 2.6e-6, at
// the caller's tolerance 1.0e-6 to 2.5e-6, at half of it 3.8e-7 to 1.2e-6; 5000
// growing items 54.0 against 52.7 us per step.  (Plain CG under a cap: as asked.)
__device__ __forceinline__ double fp32_rtol2(double rtol2, int sp, int maxit)
{
    return sp || maxit < kPlainCap ? rtol2 : fmax(fmin(rtol2, 1e-16), 0.25 * rtol2);
}

// Corrections of an FP64 system after its first solve: refined until the
// evaluated residual meets the tolerance.  One that has stopped falling although
// every correction converged is accepted only at the rounding of its evaluation
// (a tolerance below that); elsewhere the item goes to plain CG (an operator
// within 1e-8 of a singular one, whose solution is so much larger than the
// present field that it sets the rounding).
template <class X>
__device__ __forceinline__ int refine(X &x, const System &y, int sp, int fo, int ft, int fn,
                                      float (&r)[X::Sh::R], const float (&sg)[X::Sh::R],
                                      float (&d)[X::Sh::R], Scalars &v, int hb)
{
    using S = typename X::Sh;
    bool first = true;
    double best = __builtin_inf();
    int stalled = 0;
    for (;;) {
        correct(x, sp, fo, fn, first, d, hb);
        first = false;
        x.sync();
        v.rr = x.sum1(true_residual(x, y, sp, fo, ft, fn, r), RedSlots<S::W>::truth);
        if (!finite(v.rr))
            return kStNonfinite;
        if (!(v.rr > v.rtol2 * v.bb))
            return 0;
        stalled = v.rr > 0.25 * best ? stalled + 1 : 0;
        if (stalled >= 3)
            return v.rr > v.floor2 * v.bb ? kStRedo : 0;
        best = v.rr < best ? v.rr : best;
#pragma unroll
        for (int i = 0; i < S::R; ++i)
            d[i] = 0.0f;
        // FP32 recursion: at most five digits per correction
        const double stop2 = fmax(0.0625 * v.rtol2 * v.bb, 1e-10 * v.rr);
        const int st = pcg(x, y, r, sg, d, stop2, v);
        if (st)
            return st;
    }
}

// One item: all IMEX steps, then the outputs and the misfit.
template <bool kFp64, class X>
__device__ __forceinline__ void solve_item(const SolveArgs &a, int c, const GridDev &gd, X &x)
{
    using S = typename X::Sh;
    constexpr int C = S::C, R = S::R, N = S::N, K = S::K;
    constexpr size_t NN = (size_t)N * N;
    const double th0 = a.theta[4 * c], th1 = a.theta[4 * c + 1], th2 = a.theta[4 * c + 2],
                 th3 = a.theta[4 * c + 3];
    // fields: FP32 problems u, v (advanced in place); FP64 problems u, v of
    // the present and the next level, in turn
#pragma unroll 1
    for (int k = 0; k < K; ++k) {
        double u[C], v[C];
#pragma unroll
        for (int cc = 0; cc < C; ++cc) {
            const size_t gi = x.cell0() + x.row(k) + x.o + cc;
            if constexpr (kFp64) {
                u[cc] = ((const double *)gd.u0)[gi];
                v[cc] = ((const double *)gd.v0)[gi];
            } else {  // stored as [hi | lo]
                u[cc] = (double)((const float *)gd.u0)[gi] + (double)((const float *)gd.u0)[NN + gi];
                v[cc] = (double)((const float *)gd.v0)[gi] + (double)((const float *)gd.v0)[NN + gi];
            }
        }
        store_cols(x.field(0) + x.row(k), x.o, u);
        store_cols(x.field(1) + x.row(k), x.o, v);
        x.put_edge(0, k, u);
        x.put_edge(1, k, v);
    }
    x.sync();  // the rows of the neighbouring strips are in place
    const double inv_dt = uniform(1.0 / a.dt);
    const double decay = gd.decay;
    double rho_m2 = 1.0;
    int st = 0, itu = 0, itv = 0, steps = 0, quiet = 0;  // quiet: bit sp
    int cur = 0;  // FP64: fields of the present level are 2 cur, 2 cur + 1
    float r[R], sg[R], d[R];
#pragma unroll
    for (int i = 0; i < R; ++i)
        d[i] = 0.0f;
    int moved = 0;   // the last system's increment may differ from zero
    int zeroed = 0;  // increment buffers (2 species + buffer) known to hold zeros
    Scalars v;
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
            const int fo = 2 * cur + sp, ft = 2 * cur + (1 - sp);
            double es;
            // (FP32: d is the increment of the other species' last system, and
            // goes to its buffer hb; an increment of zero, of a field that has
            // come to rest, changes nothing but that buffer once.  The slot's
            // traffic bounds such steps: 4096 prior draws of 128^2, 8000 steps,
            // rtol 1e-9: 2.90 s against 3.86 with the stores, at 1e-7 2.66
            // against 3.86.)
            const int hb = sp ? kn : kn ^ 1, zb = 1 << (2 * (1 - sp) + hb);
            const bool advance = !kFp64 && (moved || !(zeroed & zb));
            zeroed = moved ? zeroed & ~zb : zeroed | zb;
            if (sp == 0 && advance)
                residual<0, !kFp64>(x, y, fo, ft, r, sg, v.bb, v.rr, es, d, hb);
            else if (sp == 0)
                residual<0, false>(x, y, fo, ft, r, sg, v.bb, v.rr, es, d, hb);
            else if (advance)
                residual<1, !kFp64>(x, y, fo, ft, r, sg, v.bb, v.rr, es, d, hb);
            else
                residual<1, false>(x, y, fo, ft, r, sg, v.bb, v.rr, es, d, hb);
            int still = 0;
            v.it = 0;
            v.maxit = a.maxit;
            v.floor2 = kFp64 ? uniform(fp64_floor2(y.c * a.dt)) : 0.0;
            v.rtol2 = kFp64 ? uniform(fp64_rtol2(a.rtol2, v.floor2)) : fp32_rtol2(a.rtol2, sp, a.maxit);
            const int npred = (quiet >> sp) & 1 ? 0 : np;
            start(x, y, sp, kn, npred, r, sg, d, es, v, still);
            st = pcg(x, y, r, sg, d, v.rtol2 * v.bb, v, kFp64 && out_of_range<S>(y, v) ? kStRedo : 0);
            if constexpr (kFp64) {
                if (st == 0)
                    st = refine(x, y, sp, fo, ft, 2 * (cur ^ 1) + sp, r, sg, d, v, kn);
            }
            moved = uniform((int)(npred > 0 || v.it > 0));
            quiet = (quiet & ~(1 << sp)) | (still << sp);
            itu += sp == 0 ? v.it : 0;
            itv += sp == 1 ? v.it : 0;
            if (st)
                break;
        }
        if (st) {
            if (!kFp64 && sp == 1) {
                // the step is not taken: u goes back to level n
#pragma unroll 1
                for (int k = 0; k < K; ++k)
#pragma unroll
                    for (int cc = 0; cc < C; ++cc) {
                        const int i = x.row(k) + x.o + cc;
                        x.field(0)[i] -= (double)x.h(0, kn)[i];
                    }
            }
            break;
        }
        steps = n + 1;
        if constexpr (kFp64)
            cur ^= 1;
        if (a.steady_tt > 0.0) {
            double acc = 0.0;
            const unsigned o = opaque(x.o);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                float du[C], dv[C];
                load_cols(x.h(0, kn) + x.row(k), o, du);
                if (kFp64)
                    load_cols(x.h(1, kn) + x.row(k), o, dv);
#pragma unroll
                for (int cc = 0; cc < C; ++cc) {
                    const double a0 = du[cc], a1 = kFp64 ? dv[cc] : d[k * C + cc];
                    acc += a0 * a0 + a1 * a1;
                }
                group_end();
            }
            const double thr = a.steady_tt * (double)N;
            if (x.sum1(acc, RedSlots<S::W>::step) < thr * thr)
                break;
            if (n + 1 == a.n_steps)
                st = kStNotSteady;  // the cap came first
        }
    }
    if (a.n_steps == 0 && a.steady_tt > 0.0)
        st = kStNotSteady;
    const bool pending = !kFp64 && steps > 0 && (st == 0 || st == kStNotSteady);
    const size_t off = (size_t)c * a.out_stride;
    double sum = 0.0;
    const unsigned o1 = opaque(x.o);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        double uu[C], vv[C];
        load_cols(x.field(2 * cur) + x.row(k), o1, uu);
        load_cols(x.field(2 * cur + 1) + x.row(k), o1, vv);
#pragma unroll
        for (int cc = 0; cc < C; ++cc) {
            const size_t gi = x.cell0() + x.row(k) + o1 + cc;
            const double u = uu[cc];
            const double w = vv[cc] + (pending ? (double)d[k * C + cc] : 0.0);  // v's last increment
            if (a.u_out) {
                if constexpr (kFp64)
                    ((double *)a.u_out)[off + gi] = u;
                else
                    ((float *)a.u_out)[off + gi] = (float)u;
            }
            if (a.v_out) {
                if constexpr (kFp64)
                    ((double *)a.v_out)[off + gi] = w;
                else
                    ((float *)a.v_out)[off + gi] = (float)w;
            }
            if (a.phi && gd.y) {
                const double e = gd.y[gi] - u;
                sum = fma(e, e, sum);
            }
        }
        group_end();
    }
    // A group's last exchange, with or without a misfit: any member that gave
    // up a wait before it (and may have written wrong rows) is silent in it, so
    // that the leader gives up too and reports the item failed.
    if (a.phi)
        sum = x.sum1(sum, RedSlots<S::W>::misfit);
    else if (S::G > 1)
        x.sync();
    if (x.failed())
        st = kStGroupTimeout;
    if (a.phi) {
        if (x.leader())
            a.phi[c] = (st != 0 || !gd.y || !finite(sum)) ? __builtin_inf() : sum * gd.inv_2s2;
    }
    if (x.leader()) {
        a.status[c] = st;
        if (kFp64 && st == kStRedo)
            atomicAdd(a.redo_count, 1u);
        if (a.steps_out)
            a.steps_out[c] = steps;
        if (a.iters) {
            a.iters[2 * c] = itu;
            a.iters[2 * c + 1] = itv;
        }
    }
}

// Fields of an item's slot, and the slot's size (they are followed by the
// last two increments of each species).
template <bool kFp64>
constexpr int n_fields()
{
    return kFp64 ? 4 : 2;
}
template <class S>
constexpr size_t slot_bytes(bool fp64)
{
    return (size_t)S::cells * ((fp64 ? 4 : 2) * sizeof(double) + 4 * sizeof(float));
}

// Queue loop of a workgroup over the items of S's grid size (a launch over
// several classes takes one kernel per size, each with a queue of its own).
template <class S, bool kFp64>
__device__ __forceinline__ void serve(const SolveArgs &a, Lds<S> &s, int *s_item)
{
    init_tables<S>(s);
    Ctx<S> x(s, (char *)a.gws + (size_t)blockIdx.x * a.gws_stride, n_fields<kFp64>());
    for (int item = next_item(a.queue, s_item); item < a.n_items;
         item = next_item(a.queue, s_item)) {
        const int c = uniform(a.order ? a.order[item] : item);
        if (!a.need || uniform(a.need[c])) {
            const int gid = item_grid(a, c);
            if (gid >= 0 && uniform(a.grids[gid].n) == S::N)
                solve_item<kFp64>(a, c, a.grids[gid], x);
        }
    }
}

template <class S, bool kFp64, int kWavesPerSimd>
__global__ __launch_bounds__(S::T, kWavesPerSimd) void k_solve_pcg(SolveArgs a)
{
    __shared__ __attribute__((aligned(16))) Lds<S> s;
    serve<S, kFp64>(a, s, &s.item);
}

}  // namespace pcg
}  // namespace rd
