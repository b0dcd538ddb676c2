// Surrogate MLP of the delayed-acceptance sampler: training and inference
// with BF16 matrix-core (MFMA) GEMMs, FP32 accumulation, FP32 master weights.
//
// Network: x = phi scaled to [-1, 1] on the prior box (4 inputs)
//          -> depth x [Linear(width) + GELU] -> Linear(out_side^2),
// output in per-pixel standardised units.  Weights are [out][in] row-major.
//
// Every product has both operands with the contraction contiguous
// (C = A B^T, A [M][K], B [N][K]): activations, output gradients and weights
// are written in both orders by the kernels that produce them, so that no
// product transposes an operand in LDS (element by element that cost more
// than the matrix instructions).  Each product's epilogue finishes what
// follows it, so an activation is written once and nothing is read again for
// an elementwise pass:
//   forward         bias, GELU; the last layer's the squared error's gradient
//                   (training), the misfit (first stage of the sampler) or
//                   the bias alone
//   input gradient  times GELU'(z)
//   weight gradient Adam; one launch over all layers, which also takes the
//                   bias gradients and layer 0's weight gradient
// A training step is 2 (depth + 1) launches, a screening depth + 2.
//
// Tiles: TM x 64, K in steps of BK, 256 threads = 4 waves of TM/2 x 32 made of
// v_mfma_f32_16x16x32_bf16 blocks.  The next step's tiles are loaded into
// registers while the present one is multiplied.  What bounds a product of
// this size (0.5 GFLOP) is the latency of its steps (two barriers, the LDS
// write and read) and the launch, not the matrix cores: hence small tiles, so
// that every CU has some, and long steps.
//
// Measured: four training steps of 1024 rows through 4 -> 512 x 4 -> 1024 with
// the copy of the weights, 358 us (one launch per operation, 31 a step:
// 1290 us); the misfits of 84 rows, 25.9 us (7 launches: 34.7 us).
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "rd_device.hpp"
#include "rd_internal.hpp"
#include "rd_mlp.hpp"

namespace rd {

typedef __bf16 bf16;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBN = 64, kLdsPad = 8;

__device__ __forceinline__ float gelu_f(float z)
{
    return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
}

__device__ __forceinline__ float gelu_grad_f(float z)
{
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) +
           z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// acc[i][j] of a wave: rows wm TM/2 + 16 i, columns wn 32 + 16 j of the tile
// at (m0, n0); lane l holds row l % 16 and columns 4 (l / 16) .. + 3 of a
// block.  K is a multiple of BK.
template <int TM, int BK>
struct Tile {
    static constexpr int IM = TM / 32;
    bf16 As[TM][BK + kLdsPad];
    bf16 Bs[kBN][BK + kLdsPad];
};

template <int TM, int BK>
__device__ __forceinline__ void tile_product(Tile<TM, BK> &s, const bf16 *A, int lda,
                                             const bf16 *B, int ldb, int m0, int n0, int K,
                                             f32x4 (&acc)[TM / 32][2])
{
    constexpr int IM = TM / 32;
    constexpr int CA = TM * BK / 2048, CB = kBN * BK / 2048;  // 16-byte loads per thread
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 va[CA], vb[CB];
    auto load = [&](int k0) {
#pragma unroll
        for (int c = 0; c < CA; ++c) {
            const int idx = t + 256 * c, row = idx / (BK / 8), kc = (idx % (BK / 8)) * 8;
            va[c] = *(const bf16x8 *)&A[(size_t)(m0 + row) * lda + k0 + kc];
        }
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const int idx = t + 256 * c, row = idx / (BK / 8), kc = (idx % (BK / 8)) * 8;
            vb[c] = *(const bf16x8 *)&B[(size_t)(n0 + row) * ldb + k0 + kc];
        }
    };
    load(0);
    for (int k0 = 0; k0 < K; k0 += BK) {
        __syncthreads();  // the previous step's LDS reads are done
#pragma unroll
        for (int c = 0; c < CA; ++c) {
            const int idx = t + 256 * c, row = idx / (BK / 8), kc = (idx % (BK / 8)) * 8;
            *(bf16x8 *)&s.As[row][kc] = va[c];
        }
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const int idx = t + 256 * c, row = idx / (BK / 8), kc = (idx % (BK / 8)) * 8;
            *(bf16x8 *)&s.Bs[row][kc] = vb[c];
        }
        __syncthreads();
        if (k0 + BK < K)  // next step's tiles, in flight during the products
            load(k0 + BK);
        const int r = lane & 15, kq = (lane >> 4) * 8;
#pragma unroll
        for (int ks = 0; ks < BK; ks += 32) {
            bf16x8 a[IM], b[2];
#pragma unroll
            for (int i = 0; i < IM; ++i)
                a[i] = *(const bf16x8 *)&s.As[wm * (TM / 2) + i * 16 + r][ks + kq];
#pragma unroll
            for (int j = 0; j < 2; ++j)
                b[j] = *(const bf16x8 *)&s.Bs[wn * 32 + j * 16 + r][ks + kq];
#pragma unroll
            for (int i = 0; i < IM; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)  // (B first: a lane's four values are one row's)
                    acc[i][j] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
        }
    }
}

__device__ __forceinline__ bf16x4 to_bf16(f32x4 v)
{
    return bf16x4{(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
}

enum Epi {
    kEpiBias = 0,   // y = v + b
    kEpiGelu,       // h = GELU(v + b)
    kEpiGeluTrain,  // the same, with z kept and h in both orders
    kEpiMse,        // dy = 2 (v + b - t) / (rows cols)
    kEpiMisfit,     // |ybar - (mean + sd (v + b))|^2 of each row
    kEpiGrad,       // dz = v GELU'(z)
    kEpiGrad0       // the same for layer 0, whose BF16 copies nothing reads
};

struct GemmArgs {
    const bf16 *A, *B;   // [M][K], [N][K]
    int M, N, K;
    const float *bias;   // [N]
    float *c32;          // [M][N] y, z or dz (out)
    const float *z;      // [M][N] pre-activation (kEpiGrad, kEpiGrad0)
    bf16 *c16, *c16t;    // [M][N], [N][ldt]
    int ldt;
    int rows;            // rows that are not padding
    const float *target; // [rows][N] (kEpiMse)
    float scale;
    double *sse;         // one per tile, or null (kEpiMse)
    const float *mean, *sd;   // kEpiMisfit
    const double *ybar;
    double *rowpart;     // [N / 64][M]
};

template <int TM, int BK, int EPI>
__global__ __launch_bounds__(256) void k_gemm(GemmArgs g)
{
    constexpr int IM = TM / 32;
    __shared__ __attribute__((aligned(16))) Tile<TM, BK> s;
    __shared__ double red[4];
    __shared__ double rowsum[4][TM / 2];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * kBN;
    f32x4 acc[IM][2];
    tile_product<TM, BK>(s, g.A, g.K, g.B, g.K, m0, n0, g.K, acc);
    double sse = 0.0, rs[IM];
#pragma unroll
    for (int i = 0; i < IM; ++i) {
        const int m = m0 + wm * (TM / 2) + i * 16 + (lane & 15);
        rs[i] = 0.0;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = n0 + wn * 32 + j * 16 + (lane >> 4) * 4;
            const size_t o = (size_t)m * g.N + n;
            f32x4 v = acc[i][j];
            if constexpr (EPI != kEpiGrad && EPI != kEpiGrad0)
                v += *(const f32x4 *)&g.bias[n];
            if constexpr (EPI == kEpiBias) {
                *(f32x4 *)&g.c32[o] = v;
            } else if constexpr (EPI == kEpiGelu || EPI == kEpiGeluTrain) {
                if constexpr (EPI == kEpiGeluTrain)
                    *(f32x4 *)&g.c32[o] = v;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    v[q] = gelu_f(v[q]);
            } else if constexpr (EPI == kEpiMse) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float e = m < g.rows ? v[q] - g.target[o + q] : 0.0f;
                    sse += (double)e * (double)e;
                    v[q] = g.scale * e;
                }
                *(f32x4 *)&g.c32[o] = v;
            } else if constexpr (EPI == kEpiMisfit) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double u = (double)g.mean[n + q] + (double)g.sd[n + q] * (double)v[q];
                    const double e = g.ybar[n + q] - u;
                    rs[i] += e * e;
                }
            } else {
                const f32x4 z = *(const f32x4 *)&g.z[o];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    v[q] *= gelu_grad_f(z[q]);
                *(f32x4 *)&g.c32[o] = v;
            }
            if constexpr (EPI == kEpiGelu || EPI == kEpiGeluTrain || EPI == kEpiMse ||
                          EPI == kEpiGrad) {
                const bf16x4 h = to_bf16(v);
                *(bf16x4 *)&g.c16[o] = h;
                if constexpr (EPI != kEpiGelu) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        g.c16t[(size_t)(n + q) * g.ldt + m] = h[q];
                }
            }
        }
    }
    if constexpr (EPI == kEpiMse) {
        if (g.sse) {
            sse = block_sum<4>(sse, red);
            if (t == 0)
                g.sse[blockIdx.y * gridDim.x + blockIdx.x] = sse;
        }
    }
    if constexpr (EPI == kEpiMisfit) {
        // a row's sum over the tile's 64 columns: four lanes, then two waves
#pragma unroll
        for (int i = 0; i < IM; ++i) {
            double v = rs[i];
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (lane < 16)
                rowsum[wave][i * 16 + lane] = v;
        }
        __syncthreads();
        if (t < TM) {
            const int h = t / (TM / 2), r = t % (TM / 2);
            g.rowpart[(size_t)blockIdx.x * g.M + m0 + t] = rowsum[2 * h][r] + rowsum[2 * h + 1][r];
        }
    }
}

// Misfits from the column tiles' sums, added in their order.
__global__ void k_misfit(int n, int M, int tiles, const double *rowpart, double inv_2s2, double *ll)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n)
        return;
    double v = 0.0;
    for (int b = 0; b < tiles; ++b)
        v += rowpart[(size_t)b * M + r];
    ll[r] = finite(v) ? v * inv_2s2 : __builtin_inf();
}

// Tile of an M x N x K product: 64 rows where that gives every CU two
// workgroups (kTall tiles), 32 below, with the longest step up to 256 that
// divides K (128 for 64 rows: the registers that hold the next step).
// Measured, four training steps of 1024 rows at width 512: 358 us; with steps
// of 128: 378 us, of 512: 369 us; with 64 rows from 256 tiles on: 369 us.
constexpr int kTall = 512;
static int tile_rows(int M, int N)
{
    return (M / 64) * (N / kBN) >= kTall ? 64 : 32;
}

template <int TM, int BK, int EPI>
static void launch(const GemmArgs &g, dim3 grid, dim3 block, hipStream_t s)
{
    hipLaunchKernelGGL((k_gemm<TM, BK, EPI>), grid, block, 0, s, g);
}

template <int EPI>
static hipError_t gemm(const GemmArgs &g, hipStream_t s)
{
    if (g.M % 64 || g.N % kBN || g.K % 64 || g.K <= 0)
        return hipErrorInvalidValue;
    const int tm = tile_rows(g.M, g.N);
    const dim3 grid(g.N / kBN, g.M / tm), block(256);
    if (tm == 64)
        g.K % 128 == 0 ? launch<64, 128, EPI>(g, grid, block, s) : launch<64, 64, EPI>(g, grid, block, s);
    else if (g.K % 256 == 0)
        launch<32, 256, EPI>(g, grid, block, s);
    else if (g.K % 128 == 0)
        launch<32, 128, EPI>(g, grid, block, s);
    else
        launch<32, 64, EPI>(g, grid, block, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// First layer (fan-in 4): x = 2 (phi - lo) / (hi - lo) - 1 (zero in padded
// rows), z = x W^T + b, h = GELU(z).  A block takes 16 rows and 64 columns; a
// thread four rows of one column.  z, x and ht are written in training only.
// (Rows on the grid's x: its y ends at 65535 blocks, a million rows of 16.)
template <bool kTrain>
__global__ __launch_bounds__(256) void k_layer0(int n, int width, const double *phi, SurScale sc,
                                                const float *W, const float *b, float *x0,
                                                float *z, bf16 *h, bf16 *ht, int ldt)
{
    __shared__ float xs[16][4];
    const int t = threadIdx.x, m0 = blockIdx.x * 16, col = blockIdx.y * 64 + (t & 63);
    if (t < 64) {
        const int r = m0 + (t >> 2), c = t & 3;
        const float v =
            r < n ? (float)(2.0 * (phi[4 * (size_t)r + c] - sc.lo[c]) / (sc.hi[c] - sc.lo[c]) - 1.0)
                  : 0.0f;
        xs[t >> 2][c] = v;
        if (kTrain && blockIdx.y == 0)
            x0[4 * (size_t)r + c] = v;
    }
    __syncthreads();
    const f32x4 w = *(const f32x4 *)&W[4 * col];
    const float bias = b[col];
    const int r0 = (t >> 6) * 4;
    bf16x4 hv;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float s = bias;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            s = fmaf(xs[r0 + q][k], w[k], s);
        const size_t o = (size_t)(m0 + r0 + q) * width + col;
        hv[q] = (bf16)gelu_f(s);
        h[o] = hv[q];
        if (kTrain)
            z[o] = s;
    }
    if (kTrain)
        *(bf16x4 *)&ht[(size_t)col * ldt + m0 + r0] = hv;
}

// Mean of the tiles' squared errors.
__global__ void k_loss(int tiles, double inv_count, const double *sse, double *loss)
{
    __shared__ double red[4];
    double s = 0.0;
    for (int r = threadIdx.x; r < tiles; r += blockDim.x)
        s += sse[r];
    s = block_sum<4>(s, red);
    if (threadIdx.x == 0)
        *loss = s * inv_count;
}

// Adam with bias correction.
struct AdamArgs {
    float lr, b1, b2, eps;
    int t;
};

struct Adam {
    float lr, b1, b2, eps, c1, c2;
    __device__ __forceinline__ explicit Adam(const AdamArgs &a)
        : lr(a.lr), b1(a.b1), b2(a.b2), eps(a.eps), c1(1.f - powf(a.b1, (float)a.t)),
          c2(1.f - powf(a.b2, (float)a.t))
    {
    }
    __device__ __forceinline__ float step(float w, float gi, float &m, float &v) const
    {
        // (contractions written out: the same bits in every kernel)
        const float mi = fmaf(1.f - b1, gi, b1 * m);
        const float vi = fmaf((1.f - b2) * gi, gi, b2 * v);
        m = mi;
        v = vi;
        const float mh = mi / c1;
        const float vh = vi / c2;
        return w - lr * mh / (sqrtf(vh) + eps);
    }
};

constexpr int kMaxLayers = 9;  // depth <= 8, and the output layer

struct LayerUpdate {
    int din, dout, tiles;    // tiles: workgroups of its weight gradient (0: layer 0)
    const bf16 *dzt, *ht;    // [dout][ldt], [din][ldt]
    const float *dz32;       // [rows][dout]
    float *W, *gW, *mW, *vW, *b, *gb, *mb, *vb;
    bf16 *W16, *W16t;        // [dout][din], [din][dout]
};

struct UpdateArgs {
    LayerUpdate l[kMaxLayers];
    const float *x;          // [rows][4] network inputs
    int layers, rows, ldt;   // rows: contraction length (padded batch)
    AdamArgs adam;
};

// Weight gradients of layers 1 .. (a workgroup per 32 x 64 tile) with Adam and
// the BF16 copies in the epilogue.  The remaining workgroups take 16 columns
// each of the bias gradients of all layers and of layer 0's weight gradient:
// 16 row groups (every 16th row) add up in row order and their sums in group
// order.  (Column sums of the row tiles would spare the FP32 gradients, but
// Adam divides a gradient by its own size, so that near-zero ones would turn
// another rounding of the sum into another step.)
//
// Bound by the passes over W, m, v (24 bytes a weight, 32 MB with the
// gradient and the copies: 7 us at 4.7 TB/s) and the two passes' latency: 23
// us.  32-row tiles with steps of kUpdateBK = 128; 64-row tiles leave a third
// of the CUs one workgroup (369 us for the four steps above against 358).
constexpr int kUpdateBK = 128;
template <int BK>
__global__ __launch_bounds__(256) void k_update(UpdateArgs u)
{
    constexpr int TM = 32, IM = TM / 32;
    __shared__ __attribute__((aligned(16))) Tile<TM, BK> s;
    __shared__ float cols[5][16][16];
    const Adam adam(u.adam);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    int wg = blockIdx.x;
    for (int l = 1; l < u.layers; ++l) {
        const LayerUpdate &L = u.l[l];
        if (wg >= L.tiles) {
            wg -= L.tiles;
            continue;
        }
        const int nt = L.din / kBN;
        const int m0 = wg / nt * TM, n0 = wg % nt * kBN;
        f32x4 acc[IM][2];
        tile_product<TM, BK>(s, L.dzt, u.ldt, L.ht, u.ldt, m0, n0, u.rows, acc);
#pragma unroll
        for (int i = 0; i < IM; ++i) {
            const int m = m0 + wm * (TM / 2) + i * 16 + (lane & 15);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int n = n0 + wn * 32 + j * 16 + (lane >> 4) * 4;
                const size_t o = (size_t)m * L.din + n;
                f32x4 w = *(const f32x4 *)&L.W[o], mm = *(const f32x4 *)&L.mW[o],
                      vv = *(const f32x4 *)&L.vW[o];
                const f32x4 g = acc[i][j];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float a = mm[q], b = vv[q];
                    w[q] = adam.step(w[q], g[q], a, b);
                    mm[q] = a;
                    vv[q] = b;
                }
                *(f32x4 *)&L.gW[o] = g;
                *(f32x4 *)&L.W[o] = w;
                *(f32x4 *)&L.mW[o] = mm;
                *(f32x4 *)&L.vW[o] = vv;
                const bf16x4 h = to_bf16(w);
                *(bf16x4 *)&L.W16[o] = h;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    L.W16t[(size_t)(n + q) * L.dout + m] = h[q];
            }
        }
        return;
    }
    for (int l = 0; l < u.layers; ++l) {
        const LayerUpdate &L = u.l[l];
        const int blocks = L.dout / 16;
        if (wg >= blocks) {
            wg -= blocks;
            continue;
        }
        const int c = t & 15, grp = t >> 4, n = wg * 16 + c;
        float v[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
        if (l == 0) {
#pragma unroll 4
            for (int r = grp; r < u.rows; r += 16) {
                const float d = L.dz32[(size_t)r * L.dout + n];
                const f32x4 x = *(const f32x4 *)&u.x[(size_t)r * 4];
                v[0] += d;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    v[k + 1] = fmaf(d, x[k], v[k + 1]);
            }
        } else {
#pragma unroll 8
            for (int r = grp; r < u.rows; r += 16)
                v[0] += L.dz32[(size_t)r * L.dout + n];
        }
#pragma unroll
        for (int k = 0; k < 5; ++k)
            cols[k][grp][c] = v[k];
        __syncthreads();
        if (grp < (l == 0 ? 5 : 1)) {  // group k finishes sum k
            float g = 0.f;
            for (int q = 0; q < 16; ++q)
                g += cols[grp][q][c];
            if (grp == 0) {
                L.gb[n] = g;
                L.b[n] = adam.step(L.b[n], g, L.mb[n], L.vb[n]);
            } else {
                const int o = 4 * n + grp - 1;
                L.gW[o] = g;
                L.W[o] = adam.step(L.W[o], g, L.mW[o], L.vW[o]);
            }
        }
        return;
    }
}

// BF16 copies of W [dout][din] in both orders.
__global__ void k_to_bf16(int dout, int din, const float *p, bf16 *p16, bf16 *p16t)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < dout * din) {
        const bf16 h = (bf16)p[i];
        p16[i] = h;
        p16t[(size_t)(i % din) * dout + i / din] = h;
    }
}

// Two arrays in one launch.
__global__ void k_copy2(const float *a, float *oa, int na, const float *b, float *ob, int nb)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < na)
        oa[i] = a[i];
    else if (i - na < nb)
        ob[i - na] = b[i - na];
}

// Uniform(-bound, bound) initialisation from the counter-based generator
// (key = (tensor id, seed), counter = element index).
__global__ void k_init_uniform(int count, float *p, float bound, uint32_t seed, uint32_t tensor)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count)
        return;
    const U32x4 w = philox10(U32x4{(uint32_t)i, 0u, 0u, 0u}, tensor, seed);
    const double u = unit_open(w.x, w.y);
    p[i] = (float)((2.0 * u - 1.0) * bound);
}

// Block means: u [n][N][N] -> out [n][S][S], blocks of (N/S)^2 cells.
template <typename Real>
__global__ void k_downsample(int n, int N, int S, const Real *u, float *out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * S * S)
        return;
    const int c = i / (S * S), J = (i / S) % S, I = i % S, f = N / S;
    double s = 0.0;
    for (int jj = 0; jj < f; ++jj)
        for (int ii = 0; ii < f; ++ii)
            s += (double)u[(size_t)c * N * N + (size_t)(J * f + jj) * N + I * f + ii];
    out[i] = (float)(s / (double)(f * f));
}

__global__ void k_destandardise(int n, int cols, const float *y, const float *mean, const float *sd,
                                float *out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n * cols)
        out[i] = mean[i % cols] + sd[i % cols] * y[i];
}

__global__ void k_ybar(int N, int S, const double *y, double *ybar)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S * S)
        return;
    const int J = i / S, I = i % S, f = N / S;
    double s = 0.0;
    for (int jj = 0; jj < f; ++jj)
        for (int ii = 0; ii < f; ++ii)
            s += y[(size_t)(J * f + jj) * N + I * f + ii];
    ybar[i] = s / (double)(f * f);
}

static inline dim3 blocks_for(size_t n, int t = 256)
{
    return dim3((unsigned)((n + t - 1) / t));
}

// ---------------------------------------------------------------------------
// Host side.

struct Surrogate {
    SurrogateDesc d{};
    int L = 0;               // linear layers = depth + 1
    int out = 0;             // out_side^2
    int bpad = 0;            // row capacity (multiple of 64)
    std::vector<int> din, dout;
    std::vector<float *> W, b, gW, gb, mW, vW, mb, vb;
    std::vector<bf16 *> W16, W16t;  // [dout][din], [din][dout]
    std::vector<float *> Z;    // pre-activations [bpad][dout] (hidden layers)
    std::vector<bf16 *> H, Ht; // activations [bpad][dout], [dout][bpad]
    std::vector<bf16 *> dz, dzt;  // output gradients, likewise (layers 1 ..)
    std::vector<float *> dz32;    // [bpad][dout]
    float *x0 = nullptr;       // [bpad][4]
    float *Y = nullptr;        // [bpad][out]
    double *sse = nullptr;     // squared error per tile
    double *rowpart = nullptr; // [out / 64][bpad] misfit per column tile
    float *mean = nullptr, *sd = nullptr;
    double *ybar = nullptr;
    double inv_2s2 = 0.0;
    bool scaled = false;
    int t = 0;
    std::vector<void *> allocs;
};

static void *salloc(Surrogate *s, size_t bytes, bool *ok)
{
    void *p = nullptr;
    if (hipMalloc(&p, bytes ? bytes : 16) != hipSuccess) {
        *ok = false;
        return nullptr;
    }
    s->allocs.push_back(p);
    return p;
}

int32_t surrogate_new(Surrogate **out, const SurrogateDesc &d, uint32_t seed)
{
    *out = nullptr;
    Surrogate *s = new Surrogate();
    s->d = d;
    s->L = d.depth + 1;
    s->out = d.out_side * d.out_side;
    s->bpad = ((d.max_batch + 63) / 64) * 64;
    bool ok = true;
    const size_t tiles = s->bpad / 32;  // most row tiles of a product
    for (int l = 0; l < s->L; ++l) {
        const int fi = l == 0 ? 4 : d.width;
        const int fo = l == s->L - 1 ? s->out : d.width;
        s->din.push_back(fi);
        s->dout.push_back(fo);
        const size_t nw = (size_t)fi * fo;
        s->W.push_back((float *)salloc(s, nw * 4, &ok));
        s->b.push_back((float *)salloc(s, fo * 4, &ok));
        s->gW.push_back((float *)salloc(s, nw * 4, &ok));
        s->gb.push_back((float *)salloc(s, fo * 4, &ok));
        s->mW.push_back((float *)salloc(s, nw * 4, &ok));
        s->vW.push_back((float *)salloc(s, nw * 4, &ok));
        s->mb.push_back((float *)salloc(s, fo * 4, &ok));
        s->vb.push_back((float *)salloc(s, fo * 4, &ok));
        s->W16.push_back((bf16 *)salloc(s, nw * 2, &ok));
        s->W16t.push_back((bf16 *)salloc(s, nw * 2, &ok));
        const bool hidden = l < s->L - 1;
        const size_t act = (size_t)s->bpad * fo;
        s->Z.push_back((float *)salloc(s, hidden ? act * 4 : 0, &ok));
        s->H.push_back((bf16 *)salloc(s, hidden ? act * 2 : 0, &ok));
        s->Ht.push_back((bf16 *)salloc(s, hidden ? act * 2 : 0, &ok));
        s->dz.push_back((bf16 *)salloc(s, l > 0 ? act * 2 : 0, &ok));
        s->dzt.push_back((bf16 *)salloc(s, l > 0 ? act * 2 : 0, &ok));
        s->dz32.push_back((float *)salloc(s, act * 4, &ok));
    }
    s->x0 = (float *)salloc(s, (size_t)s->bpad * 4 * 4, &ok);
    s->Y = (float *)salloc(s, (size_t)s->bpad * s->out * 4, &ok);
    s->sse = (double *)salloc(s, tiles * (s->out / kBN) * 8, &ok);
    s->rowpart = (double *)salloc(s, (size_t)s->bpad * (s->out / kBN) * 8, &ok);
    s->mean = (float *)salloc(s, s->out * 4, &ok);
    s->sd = (float *)salloc(s, s->out * 4, &ok);
    s->ybar = (double *)salloc(s, s->out * 8, &ok);
    if (!ok) {
        surrogate_destroy(s);
        return -3;
    }
    for (int l = 0; l < s->L; ++l) {
        const int nw = s->din[l] * s->dout[l];
        const float bound = 1.0f / sqrtf((float)s->din[l]);
        hipLaunchKernelGGL(k_init_uniform, blocks_for(nw), dim3(256), 0, nullptr, nw, s->W[l], bound,
                           seed, (uint32_t)(2 * l));
        hipLaunchKernelGGL(k_init_uniform, blocks_for(s->dout[l]), dim3(256), 0, nullptr, s->dout[l],
                           s->b[l], bound, seed, (uint32_t)(2 * l + 1));
        hipLaunchKernelGGL(k_to_bf16, blocks_for(nw), dim3(256), 0, nullptr, s->dout[l], s->din[l],
                           s->W[l], s->W16[l], s->W16t[l]);
        if (hipMemset(s->mW[l], 0, (size_t)nw * 4) != hipSuccess ||
            hipMemset(s->vW[l], 0, (size_t)nw * 4) != hipSuccess ||
            hipMemset(s->mb[l], 0, (size_t)s->dout[l] * 4) != hipSuccess ||
            hipMemset(s->vb[l], 0, (size_t)s->dout[l] * 4) != hipSuccess)
            ok = false;
    }
    if (!ok || hipDeviceSynchronize() != hipSuccess) {
        surrogate_destroy(s);
        return -2;
    }
    *out = s;
    return 0;
}

void surrogate_destroy(Surrogate *s)
{
    if (!s)
        return;
    hipDeviceSynchronize();
    for (void *p : s->allocs)
        hipFree(p);
    delete s;
}

bool surrogate_ready(const Surrogate *s) { return s && s->scaled; }
int surrogate_max_batch(const Surrogate *s) { return s ? s->bpad : 0; }
int surrogate_layers(const Surrogate *s) { return s ? s->L : 0; }

hipError_t surrogate_downsample(Surrogate *s, int n, const void *u, float *out, hipStream_t st)
{
    if (n <= 0)
        return hipSuccess;
    const size_t cnt = (size_t)n * s->out;
    if (s->d.precision == 0)
        hipLaunchKernelGGL(k_downsample<float>, blocks_for(cnt), dim3(256), 0, st, n, s->d.n,
                           s->d.out_side, (const float *)u, out);
    else
        hipLaunchKernelGGL(k_downsample<double>, blocks_for(cnt), dim3(256), 0, st, n, s->d.n,
                           s->d.out_side, (const double *)u, out);
    return hipGetLastError();
}

// Box of the sampling coordinates that the network's inputs are mapped to
// [-1, 1] over (the prior box by default).
void surrogate_input_box(Surrogate *s, const double lo[4], const double hi[4])
{
    for (int i = 0; i < 4; ++i) {
        s->d.lo[i] = lo[i];
        s->d.hi[i] = hi[i];
    }
}

hipError_t surrogate_scaling(Surrogate *s, const float *mean, const float *sd, double sigma1,
                             hipStream_t st)
{
    hipError_t e;
    if ((e = hipMemcpyAsync(s->mean, mean, s->out * 4, hipMemcpyDeviceToDevice, st)) != hipSuccess ||
        (e = hipMemcpyAsync(s->sd, sd, s->out * 4, hipMemcpyDeviceToDevice, st)) != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_ybar, blocks_for(s->out), dim3(256), 0, st, s->d.n, s->d.out_side, s->d.y,
                       s->ybar);
    s->inv_2s2 = 0.5 / (sigma1 * sigma1);
    s->scaled = true;
    return hipGetLastError();
}

// Forward pass of `rows` rows (padded to a multiple of 64) up to the last
// layer, whose product the caller finishes with `tail`.
template <bool kTrain, typename F>
static hipError_t forward(Surrogate *s, int rows, const double *phi, hipStream_t st, F &&tail)
{
    const int mp = ((rows + 63) / 64) * 64;
    SurScale sc;
    for (int i = 0; i < 4; ++i) {
        sc.lo[i] = s->d.lo[i];
        sc.hi[i] = s->d.hi[i];
    }
    hipLaunchKernelGGL(k_layer0<kTrain>, dim3(mp / 16, s->dout[0] / 64), dim3(256), 0, st, rows,
                       s->dout[0], phi, sc, s->W[0], s->b[0], s->x0, s->Z[0], s->H[0], s->Ht[0],
                       s->bpad);
    hipError_t e = hipGetLastError();
    for (int l = 1; l < s->L && e == hipSuccess; ++l) {
        GemmArgs g{};
        g.A = s->H[l - 1];
        g.B = s->W16[l];
        g.M = mp;
        g.N = s->dout[l];
        g.K = s->din[l];
        g.bias = s->b[l];
        g.rows = rows;
        if (l < s->L - 1) {
            g.c32 = s->Z[l];
            g.c16 = s->H[l];
            g.c16t = s->Ht[l];
            g.ldt = s->bpad;
            e = kTrain ? gemm<kEpiGeluTrain>(g, st) : gemm<kEpiGelu>(g, st);
        } else {
            e = tail(g);
        }
    }
    return e;
}

static hipError_t forward_y(Surrogate *s, int rows, const double *phi, hipStream_t st)
{
    return forward<false>(s, rows, phi, st, [&](GemmArgs &g) {
        g.c32 = s->Y;
        return gemm<kEpiBias>(g, st);
    });
}

hipError_t surrogate_train(Surrogate *s, int batch, const double *phi, const float *target,
                           double lr, double *loss, hipStream_t st)
{
    const int mp = ((batch + 63) / 64) * 64;
    const int top = s->L - 1;
    hipError_t e = forward<true>(s, batch, phi, st, [&](GemmArgs &g) {
        g.c16 = s->dz[top];
        g.c16t = s->dzt[top];
        g.ldt = s->bpad;
        g.c32 = s->dz32[top];
        g.target = target;
        g.scale = 2.0f / ((float)batch * (float)s->out);
        g.sse = loss ? s->sse : nullptr;
        return gemm<kEpiMse>(g, st);
    });
    if (e != hipSuccess)
        return e;
    if (loss)
        hipLaunchKernelGGL(k_loss, dim3(1), dim3(256), 0, st,
                           mp / tile_rows(mp, s->out) * (s->out / kBN),
                           1.0 / ((double)batch * (double)s->out), s->sse, loss);
    UpdateArgs u{};
    u.layers = s->L;
    u.rows = mp;
    u.x = s->x0;
    u.ldt = s->bpad;
    for (int l = top; l >= 1; --l) {
        // dz_{l-1} = (dz_l W_l) .* GELU'(z_{l-1})
        GemmArgs g{};
        g.A = s->dz[l];
        g.B = s->W16t[l];
        g.M = mp;
        g.N = s->din[l];
        g.K = s->dout[l];
        g.z = s->Z[l - 1];
        g.c32 = s->dz32[l - 1];
        g.rows = batch;
        if (l > 1) {
            g.c16 = s->dz[l - 1];
            g.c16t = s->dzt[l - 1];
            g.ldt = s->bpad;
            e = gemm<kEpiGrad>(g, st);
        } else {
            e = gemm<kEpiGrad0>(g, st);
        }
        if (e != hipSuccess)
            return e;
    }
    s->t += 1;
    u.adam = AdamArgs{(float)lr, 0.9f, 0.999f, 1e-8f, s->t};
    int wgs = 0;
    for (int l = 0; l < s->L; ++l) {
        LayerUpdate &L = u.l[l];
        L.din = s->din[l];
        L.dout = s->dout[l];
        L.tiles = l == 0 ? 0 : (L.dout / 32) * (L.din / kBN);
        if (l > 0) {
            L.dzt = s->dzt[l];
            L.ht = s->Ht[l - 1];
        }
        L.dz32 = s->dz32[l];
        L.W = s->W[l];
        L.gW = s->gW[l];
        L.mW = s->mW[l];
        L.vW = s->vW[l];
        L.b = s->b[l];
        L.gb = s->gb[l];
        L.mb = s->mb[l];
        L.vb = s->vb[l];
        L.W16 = s->W16[l];
        L.W16t = s->W16t[l];
        wgs += L.tiles + L.dout / 16;
    }
    if (mp % kUpdateBK == 0)
        hipLaunchKernelGGL(k_update<kUpdateBK>, dim3(wgs), dim3(256), 0, st, u);
    else
        hipLaunchKernelGGL(k_update<64>, dim3(wgs), dim3(256), 0, st, u);
    return hipGetLastError();
}

hipError_t surrogate_predict(Surrogate *s, int n, const double *phi, float *out, int raw,
                             hipStream_t st)
{
    if (n <= 0)
        return hipSuccess;
    hipError_t e = forward_y(s, n, phi, st);
    if (e != hipSuccess)
        return e;
    if (raw)
        return hipMemcpyAsync(out, s->Y, (size_t)n * s->out * 4, hipMemcpyDeviceToDevice, st);
    hipLaunchKernelGGL(k_destandardise, blocks_for((size_t)n * s->out), dim3(256), 0, st, n, s->out,
                       s->Y, s->mean, s->sd, out);
    return hipGetLastError();
}

int32_t surrogate_enqueue_loglik(Surrogate *s, int n, const double *phi, double *ll, hipStream_t st)
{
    if (n <= 0)
        return 0;
    if (!s->scaled)
        return -1;
    const hipError_t e = forward<false>(s, n, phi, st, [&](GemmArgs &g) {
        g.mean = s->mean;
        g.sd = s->sd;
        g.ybar = s->ybar;
        g.rowpart = s->rowpart;
        return gemm<kEpiMisfit>(g, st);
    });
    if (e != hipSuccess)
        return -2;
    hipLaunchKernelGGL(k_misfit, blocks_for(n, 64), dim3(64), 0, st, n, ((n + 63) / 64) * 64,
                       s->out / kBN, s->rowpart, s->inv_2s2, ll);
    return hipGetLastError() == hipSuccess ? 0 : -2;
}

hipError_t surrogate_copy_params(Surrogate *s, int layer, float *w, float *b, int dir,
                                 hipStream_t st)
{
    const int nw = s->din[layer] * s->dout[layer], nb = s->dout[layer];
    auto copy = [&](const float *fw, float *tw, const float *fb, float *tb) {
        hipLaunchKernelGGL(k_copy2, blocks_for((size_t)nw + nb), dim3(256), 0, st, fw, tw, nw, fb,
                           tb, nb);
        return hipGetLastError();
    };
    if (dir == 2)
        return copy(s->gW[layer], w, s->gb[layer], b);
    if (dir == 0)
        return copy(s->W[layer], w, s->b[layer], b);
    const hipError_t e = copy(w, s->W[layer], b, s->b[layer]);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_to_bf16, blocks_for(nw), dim3(256), 0, st, s->dout[layer], s->din[layer],
                       s->W[layer], s->W16[layer], s->W16t[layer]);
    return hipGetLastError();
}

}  // namespace rd
