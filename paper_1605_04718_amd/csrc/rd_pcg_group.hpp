// The spectrally preconditioned solve at 256 x 256: a group of four
// workgroups per item.
//
// Member m owns rows 64 m .. 64 m + 63 (eight waves of 8 rows, 4 columns per
// lane) in a slot of its own.  The members exchange, through a per-group area
// of global memory with agent-coherent loads and stores, the partial sums of
// every reduction (numbered words, which are also the group's barrier, as in
// the plain-CG group above), the rows at the strips' edges, and twice per
// application of the preconditioner an FP16 array: each member transforms its
// 64 rows horizontally for all 256 modes, takes over 64 modes for both
// vertical transforms, and gets its rows back for the last one.  The tables
// (128 KB each) come from L2.
//
// What bounds it: five group exchanges per iteration and three per set-up of
// a system (a round trip between workgroups of one XCD is about 1 us): vector
// instructions are active in 0.29 of the cycles of its CUs, and its waves wait
// in 0.63 of theirs.  37 growing items, 60 steps: 6.5 ms (109 us per step);
// plain CG by a group of four 1024-thread workgroups, 120 iterations a step,
// 41.6 ms.  The 511 items of the uneven batch, 60 steps: 16.8 against 122 ms.
// Twelve FP64 items: plain CG streamed
// by one workgroup each took up to a hundred times as long.
#pragma once

namespace rd {
namespace pcg {

using S256 = Shape<256, 8, 8, 4>;

struct GroupLds {
    _Float16 x[S256::M * S256::SN];
    _Float16 y[S256::M * S256::SN];
    float z[S256::M * S256::ZN];
    float lam[S256::N];
    double red[RedSlots<S256::W>::total];
    double gather[S256::G * 8];
    int fail, item;
};

// Workspace of the groups: the item queue, every group's partial sums
// [2][G][8] of two words (zeroed before a launch), the tables Q and Q^T in fragment order,
// then per group the edge rows of the fields [4][G][2][N] f64, of the
// increments [4][G][2][N] f32 and of z [G][2][N] f32, and the exchanged FP16
// arrays [N][N] (modes of all rows; rows of all modes).
struct GroupArea {
    static constexpr size_t N = S256::N, G = S256::G;
    static constexpr size_t partial = 2 * G * 8 * 2 * sizeof(uint64_t);
    static constexpr size_t table = N * N * sizeof(_Float16);
    static constexpr size_t xrows = 4 * G * 2 * N * sizeof(double);
    static constexpr size_t hrows = 4 * G * 2 * N * sizeof(float);
    static constexpr size_t zrows = G * 2 * N * sizeof(float);
    static constexpr size_t bulk = xrows + hrows + zrows + 2 * table;
    static constexpr size_t head(int groups) { return 256 + (size_t)groups * partial; }
    static constexpr size_t bytes(int groups)
    {
        return head(groups) + 2 * table + (size_t)groups * bulk;
    }
};

// C columns of a row, coherently, at this lane's columns.
template <int C, typename T>
__device__ __forceinline__ void put_row(T *row, int col, const T (&v)[C])
{
    static_assert(C * sizeof(T) % 8 == 0, "8-byte pieces");
    u64 t[C * sizeof(T) / 8];
    __builtin_memcpy(t, v, sizeof t);
#pragma unroll
    for (unsigned i = 0; i < C * sizeof(T) / 8; ++i)
        put64((char *)(row + col) + 8 * i, t[i]);
}
template <int C, typename T>
__device__ __forceinline__ void get_row(const T *row, int col, T (&v)[C])
{
    u64 t[C * sizeof(T) / 8];
#pragma unroll
    for (unsigned i = 0; i < C * sizeof(T) / 8; ++i)
        t[i] = get64((const char *)(row + col) + 8 * i);
    __builtin_memcpy(v, t, sizeof t);
}

struct GroupCtx {
    using S = S256;
    using Sh = S256;
    GroupLds &s;
    double *xs;
    float *hs;
    int w;
    unsigned o, os, on;
    int m;                   // member
    unsigned seq;            // exchanges of this launch
    u64 wait_ticks;          // bound of one wait (100 MHz ticks)
    u64 *part;               // partial sums of the group
    unsigned char *area;     // edge rows and exchanged arrays
    const _Float16 *qf, *qt;

    __device__ GroupCtx(GroupLds &lds, const SolveArgs &a, int group, int member, int n_fields)
        : s(lds), m(member), seq(0), wait_ticks(a.coop_wait_ticks)
    {
        unsigned char *ws = (unsigned char *)a.group_ws;
        part = (u64 *)(ws + 256 + (size_t)group * GroupArea::partial);
        unsigned char *tab = ws + GroupArea::head(a.group_cap);
        qf = (const _Float16 *)tab;
        qt = (const _Float16 *)(tab + GroupArea::table);
        area = tab + 2 * GroupArea::table + (size_t)group * GroupArea::bulk;
        xs = (double *)((char *)a.gws + (size_t)blockIdx.x * a.gws_stride);
        hs = (float *)(xs + (size_t)n_fields * S::cells);
        w = wave_index();
        const int col = lane() * S::C;
        o = col;
        os = (w > 0 ? w * S::K - 1 : 0) * S::N + col;
        on = (w < S::W - 1 ? (w + 1) * S::K : S::M - 1) * S::N + col;
    }
    __device__ int strip() const { return w; }
    __device__ int lane() const { return (int)threadIdx.x % 64; }
    __device__ int row(int k) const { return (w * S::K + k) * S::N; }
    __device__ double *field(int k) const { return opaque(xs + (size_t)k * S::cells); }
    __device__ float *h(int sp, int k) const { return opaque(hs + (size_t)(2 * sp + k) * S::cells); }
    __device__ size_t cell0() const { return (size_t)m * S::M * S::N; }
    __device__ bool failed() const { return uniform(s.fail) != 0; }
    __device__ bool leader() const { return threadIdx.x == 0 && m == 0; }

    __device__ double *xrow(int field, int member, int side) const
    {
        return (double *)area + (((size_t)field * S::G + member) * 2 + side) * S::N;
    }
    __device__ float *hrow(int sp, int buf, int member, int side) const
    {
        return (float *)(area + GroupArea::xrows) +
               (((size_t)(2 * sp + buf) * S::G + member) * 2 + side) * S::N;
    }
    __device__ float *zrow(int member, int side) const
    {
        return (float *)(area + GroupArea::xrows + GroupArea::hrows) +
               ((size_t)member * 2 + side) * S::N;
    }
    __device__ _Float16 *spread(int k) const  // the exchanged arrays
    {
        return (_Float16 *)(area + GroupArea::xrows + GroupArea::hrows + GroupArea::zrows +
                            (size_t)k * GroupArea::table);
    }
    __device__ const float *zlds(int r) const { return s.z + r * S::ZN + lane() * S::C; }

    // This thread's coherent stores are complete; the workgroup's after the
    // barrier that the callers place next.
    static __device__ void drain()
    {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
    }
    // Sums over the members of M values that every thread of the member holds,
    // in member order (the same bits in every member).  A value travels as two
    // words, a half of it and the exchange's number each, so that the word is
    // its own arrival flag and the sum loses no bits; with numbers of 32 bits,
    // zeroed before a launch, no stale word can match.  Bounded: a member that
    // waits too long raises fail, and neither waits nor publishes again, so
    // every exchange ends, and the other members take none of its later values
    // for sums: they give up in turn at their next exchange, before the item is
    // reported.
    template <int M>
    __device__ void exchange(double (&v)[M])
    {
        static_assert(M <= 8 && S::G * 2 * M <= kWave, "one lane per word");
        seq += 1;
        u64 *buf = part + (size_t)(seq & 1u) * S::G * 16;
        const int t = threadIdx.x;
        unsigned *got = (unsigned *)s.gather;  // [member][value][half]
        if (t < 2 * M) {
            const unsigned mine = half_of(v, t);
            if (!s.fail)
                put64(buf + lane_off(m * 16 + t), (u64)mine << 32 | seq);
            got[m * 2 * M + t] = mine;
        }
        asm volatile("" ::: "memory");  // the store is issued before any poll
        if (t < S::G * 2 * M && t / (2 * M) != m) {
            const int mm = t / (2 * M), j = t % (2 * M);
            got[t] = await(buf + lane_off(mm * 16 + j), seq, wait_ticks, &s.fail);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < M; ++j) {
            double sum = 0.0;
#pragma unroll
            for (int mm = 0; mm < S::G; ++mm)
                sum += s.gather[mm * M + j];
            v[j] = uniform(sum);
        }
    }
    template <int M>
    __device__ void sum(double (&v)[M], int slot)
    {
        wave_totals<S::W>(v, s.red + slot, w);
        drain();
        __syncthreads();
        slots_sum<S::W>(v, s.red + slot);
        exchange(v);
    }
    __device__ double sum1(double v, int slot)
    {
        double t[1] = {v};
        sum(t, slot);
        return t[0];
    }
    __device__ void sync()
    {
        drain();
        __syncthreads();
        double z[1] = {0.0};
        exchange(z);
    }
    __device__ void halo(int k, double (&lo)[S::C], double (&hi)[S::C]) const
    {
        const int col = lane() * S::C;
        if (w > 0 || m == 0)
            load_cols(field(k), opaque(os), lo);
        else
            get_row(xrow(k, m - 1, 1), col, lo);
        if (w < S::W - 1 || m == S::G - 1)
            load_cols(field(k), opaque(on), hi);
        else
            get_row(xrow(k, m + 1, 0), col, hi);
    }
    __device__ void halo(int sp, int k, float (&lo)[S::C], float (&hi)[S::C]) const
    {
        const int col = lane() * S::C;
        if (w > 0 || m == 0)
            load_cols(h(sp, k), opaque(os), lo);
        else
            get_row(hrow(sp, k, m - 1, 1), col, lo);
        if (w < S::W - 1 || m == S::G - 1)
            load_cols(h(sp, k), opaque(on), hi);
        else
            get_row(hrow(sp, k, m + 1, 0), col, hi);
    }
    __device__ void halo_z(float (&lo)[S::C], float (&hi)[S::C]) const
    {
        const int col = lane() * S::C;
        if (w > 0 || m == 0) {
#pragma unroll
            for (int c = 0; c < S::C; ++c)
                lo[c] = zlds(w > 0 ? w * S::K - 1 : 0)[c];
        } else {
            get_row(zrow(m - 1, 1), col, lo);
        }
        if (w < S::W - 1 || m == S::G - 1) {
#pragma unroll
            for (int c = 0; c < S::C; ++c)
                hi[c] = zlds(w < S::W - 1 ? (w + 1) * S::K : S::M - 1)[c];
        } else {
            get_row(zrow(m + 1, 0), col, hi);
        }
    }
    __device__ void put_edge(int k, int r, const double (&v)[S::C]) const
    {
        const int col = lane() * S::C;
        if (r == 0 && w == 0)
            put_row(xrow(k, m, 0), col, v);
        if (r == S::K - 1 && w == S::W - 1)
            put_row(xrow(k, m, 1), col, v);
    }
    __device__ void put_edge(int sp, int k, int r, const float (&v)[S::C]) const
    {
        const int col = lane() * S::C;
        if (r == 0 && w == 0)
            put_row(hrow(sp, k, m, 0), col, v);
        if (r == S::K - 1 && w == S::W - 1)
            put_row(hrow(sp, k, m, 1), col, v);
    }
    __device__ void put_edge_z(const float (&z)[S::R]) const
    {
        const int col = lane() * S::C;
        float t[S::C];
        if (w == 0) {
#pragma unroll
            for (int c = 0; c < S::C; ++c)
                t[c] = z[c];
            put_row(zrow(m, 0), col, t);
        }
        if (w == S::W - 1) {
#pragma unroll
            for (int c = 0; c < S::C; ++c)
                t[c] = z[(S::K - 1) * S::C + c];
            put_row(zrow(m, 1), col, t);
        }
    }
    __device__ void set_z(const float (&r)[S::R]) const
    {
#pragma unroll
        for (int k = 0; k < S::K; ++k)
#pragma unroll
            for (int c = 0; c < S::C; ++c)
                s.z[(w * S::K + k) * S::ZN + lane() * S::C + c] = r[k * S::C + c];
    }
};

// One transform stage of a wave: the tiles 2 w and 2 w + 1 of the table with
// the four 16-row tiles of the member's 64 rows (LDS), handed to
// f(table tile, row tile, acc); kTableFirst as in product().
template <bool kTableFirst, typename F>
__device__ __forceinline__ void group_product(const _Float16 *m, int w, const _Float16 *rows, F &&f)
{
    using S = S256;
    constexpr int KS = S::KS, SN = S::SN;
    const int lane = lane_here(), lr = lane & 15, lq = lane >> 4;
    const _Float16 *ml = m + (size_t)2 * w * KS * 512 + lane * 8;
    half8 b[2][KS];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            b[u][ks] = *(const half8 *)&ml[(u * KS + ks) * 512];
#pragma unroll 1
    for (int mt = 0; mt < S::M / 16; ++mt) {
        const _Float16 *p = rows + (mt * 16 + lr) * SN + lq * 8;
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const half8 a = *(const half8 *)&p[ks * 32];
#pragma unroll
            for (int u = 0; u < 2; ++u)
                acc[u] = kTableFirst ? mfma(b[u][ks], a, acc[u]) : mfma(a, b[u][ks], acc[u]);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
            f(2 * w + u, mt, acc[u]);
    }
}

// The member's 64 rows of an exchanged array into LDS (256 values each).
__device__ __forceinline__ void gather_rows(const _Float16 *from, _Float16 *to)
{
    using S = S256;
    constexpr int kPieces = S::M * S::N / 4 / S::T;  // 8-byte pieces per thread
    u64 t[kPieces];
    const char *src = (const char *)from;
#pragma unroll
    for (int i = 0; i < kPieces; ++i)
        t[i] = get64(src + (size_t)(i * S::T + threadIdx.x) * 8);
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
        const int e = (i * S::T + threadIdx.x) * 4;
        *(u64 *)&to[e / S::N * S::SN + e % S::N] = t[i];
    }
}

// z = M^-1 r on the group (see apply_precond of one workgroup).
__device__ __forceinline__ void apply_precond(GroupCtx &x, const float (&r)[S256::R],
                                              float (&z)[S256::R], float scale, float cs, float out)
{
    using S = S256;
    constexpr int C = S::C, SN = S::SN, N = S::N, M = S::M;
    GroupLds &s = x.s;
    const int lane = lane_here(), lr = lane & 15, lq = lane >> 4, m0 = x.m * M;
#pragma unroll
    for (int k = 0; k < S::K; ++k) {
        half4 h;
#pragma unroll
        for (int c = 0; c < C; ++c)
            h[c] = (_Float16)(r[k * C + c] * scale);
        *(half4 *)&s.x[(x.w * S::K + k) * SN + lane * C] = h;
    }
    __syncthreads();
    // stage 1: T[j][k], own rows j, all modes k -> spread(0)[k][j]
    {
        _Float16 *t = x.spread(0);
        group_product<false>(x.qf, x.w, s.x, [&](int nt, int mt, f32x4 acc) {
            put64(&t[(size_t)(nt * 16 + lr) * N + m0 + mt * 16 + lq * 4],
                  __builtin_bit_cast(u64, to_half(acc)));
        });
    }
    x.sync();
    // own modes k of all rows
    gather_rows(x.spread(0) + (size_t)m0 * N, s.y);
    __syncthreads();
    // stage 2: U[q][k] / (1 + cs (lam_q + lam_k)) -> x[k][q]
    group_product<true>(x.qf, x.w, s.y, [&](int qt, int kt, f32x4 acc) {
        const float base = fmaf(cs, s.lam[m0 + kt * 16 + lr], 1.0f);
        const f32x4 lam = *(const f32x4 *)&s.lam[qt * 16 + lq * 4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            acc[i] *= __builtin_amdgcn_rcpf(fmaf(cs, lam[i], base));
        *(half4 *)&s.x[(kt * 16 + lr) * SN + qt * 16 + lq * 4] = to_half(acc);
    });
    __syncthreads();
    // stage 3: V[j][k], all rows j -> spread(1)[j][k]
    {
        _Float16 *t = x.spread(1);
        group_product<false>(x.qt, x.w, s.x, [&](int jt, int kt, f32x4 acc) {
            put64(&t[(size_t)(jt * 16 + lr) * N + m0 + kt * 16 + lq * 4],
                  __builtin_bit_cast(u64, to_half(acc)));
        });
    }
    x.sync();
    // own rows j of all modes
    gather_rows(x.spread(1) + (size_t)m0 * N, s.y);
    __syncthreads();
    // stage 4: z[j][i]
    group_product<true>(x.qt, x.w, s.y, [&](int it, int jt, f32x4 acc) {
        acc *= out;
        *(f32x4 *)&s.z[(jt * 16 + lr) * S::ZN + it * 16 + lq * 4] = acc;
    });
    __syncthreads();
#pragma unroll
    for (int k = 0; k < S::K; ++k) {
        const f32x4 t = *(const f32x4 *)&s.z[(x.w * S::K + k) * S::ZN + lane * C];
#pragma unroll
        for (int c = 0; c < C; ++c)
            z[k * C + c] = t[c];
    }
}

// Marks queue items failed, starting with the one in *s_item, until the
// queue (or its 256^2 prefix) is exhausted.
__device__ __forceinline__ void mark_item(const SolveArgs &a, int c, int st)
{
    a.status[c] = st;
    if (a.phi)
        a.phi[c] = __builtin_inf();
    if (a.iters) {
        a.iters[2 * c] = 0;
        a.iters[2 * c + 1] = 0;
    }
    if (a.steps_out)
        a.steps_out[c] = 0;
}

// Groups pull items from a queue of their own (the first word of the
// workspace): member 0 takes the next index and the group exchange hands it
// to the other members.  In a class-ordered batch the 256^2 items form the
// queue's prefix, and a group stops at the first item of another class (or
// with an invalid class, which sorts last).
template <bool kFp64>
__device__ __forceinline__ void group_run(const SolveArgs &a, bool prefix_only, GroupLds &s)
{
    // workgroup ids congruent modulo 8 share an XCD
    const int b = blockIdx.x, lane32 = b % 32;
    const int member = lane32 / 8, group = b / 32 * 8 + lane32 % 8;
    if (threadIdx.x == 0)
        s.fail = 0;
    for (int k = threadIdx.x; k < S256::N; k += S256::T)
        s.lam[k] = 2.0f - 2.0f * cospif((float)k / (float)S256::N);
    __syncthreads();
    GroupCtx x(s, a, group, member, n_fields<kFp64>());
    unsigned *queue = (unsigned *)a.group_ws;
    if (a.coop_stall_ticks && member == 1) {
        // Test hook (host-set): this member arrives late at the group's
        // first exchange, so that the other members' bounded waits give up.
        const u64 t0 = __builtin_amdgcn_s_memrealtime();
        while (__builtin_amdgcn_s_memrealtime() - t0 < a.coop_stall_ticks)
            __builtin_amdgcn_s_sleep(8);
    }
    for (;;) {
        if (member == 0 && threadIdx.x == 0)
            s.item = (int)atomicAdd(queue, 1u);
        __syncthreads();
        // members other than 0 contribute 0: the sum is member 0's index
        double v[1] = {member == 0 ? (double)s.item : 0.0};
        GroupCtx::drain();
        __syncthreads();
        x.exchange(v);
        if (x.failed()) {
            // A member timed out (it cannot happen while every member is
            // resident): the group stops, and member 0 marks the items it
            // still pulls, its last one included, as failed.
            if (member != 0)
                break;
            for (int item = uniform(s.item); item < a.n_items;) {
                const int c = uniform(a.order ? a.order[item] : item);
                const int gid = uniform(a.grid_id ? a.grid_id[c] : 0);
                const bool bad = (unsigned)gid >= (unsigned)a.n_grids;
                if (prefix_only && (bad || uniform(a.grids[gid].n) != S256::N))
                    break;
                if (threadIdx.x == 0 && (!a.need || a.need[c]))
                    mark_item(a, c, bad ? kStBadGrid : kStGroupTimeout);
                __syncthreads();
                if (threadIdx.x == 0)
                    s.item = (int)atomicAdd(queue, 1u);
                __syncthreads();
                item = uniform(s.item);
            }
            break;
        }
        const int item = (int)(v[0] + 0.5);
        if (item >= a.n_items)
            break;
        const int c = uniform(a.order ? a.order[item] : item);
        const int gid = uniform(a.grid_id ? a.grid_id[c] : 0);
        const bool bad = (unsigned)gid >= (unsigned)a.n_grids;
        if (prefix_only && (bad || uniform(a.grids[gid].n) != S256::N))
            break;
        if (a.need && !uniform(a.need[c]))
            continue;
        if (bad) {
            if (x.leader())
                mark_item(a, c, kStBadGrid);
            continue;
        }
        solve_item<kFp64>(a, c, a.grids[gid], x);
    }
    // a member whose wait gave up is counted once per launch (host-visible)
    if (x.failed() && threadIdx.x == 0 && a.coop_timeouts)
        atomicAdd(a.coop_timeouts, 1u);
    __syncthreads();  // every thread has read fail before the LDS is reused
}

// 256^2 items by the first a.coop_wgs workgroups (whole blocks of 32, all
// resident); in a class-ordered batch every workgroup then serves its 128^2
// items.
template <bool kFp64>
__global__ __launch_bounds__(S256::T, 2) void k_solve_group(SolveArgs a, bool mixed)
{
    constexpr size_t kLds =
        sizeof(GroupLds) > sizeof(Lds<S128>) ? sizeof(GroupLds) : sizeof(Lds<S128>);
    __shared__ __attribute__((aligned(16))) unsigned char raw[kLds];
    __shared__ int s_item;
    if ((int)blockIdx.x < a.coop_wgs)
        group_run<kFp64>(a, mixed, *(GroupLds *)raw);
    if (mixed)
        serve<S128, kFp64>(a, *(Lds<S128> *)raw, &s_item);
}

__global__ void k_group_tables(_Float16 *qf, _Float16 *qt)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    int row, col;
    fragment_entry<S256>(t, row, col);
    qf[t] = (_Float16)dct<S256::N>(row, col);
    qt[t] = (_Float16)dct<S256::N>(col, row);
}

}  // namespace pcg
}  // namespace rd
