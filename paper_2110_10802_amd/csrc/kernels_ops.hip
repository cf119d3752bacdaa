// Mish, layer normalisation and softmax: HBM-bound operators, one pass over their tensors.
//
// Row-wise operators (layer normalisation, softmax): a wavefront owns a row.  The row lives in
// registers (NV float4 per lane, coalesced 1 KB per load instruction), so every statistic is a
// register pass plus a DPP wavefront reduction and the row is read from HBM exactly once (the
// paper's warp tiling with warp-level reductions, section "Softmax"; what depends on a
// reduction is recomputed from registers instead of being written out).  Rows longer than 2048
// take a workgroup per row, rows of one to three columns a thread.  The weight gradients of layer normalisation
// are accumulated per lane over the rows a wavefront walks (a lane owns the same columns in
// every row), combined over the four wavefronts of a workgroup in LDS, written once per
// workgroup and added in a fixed order by a second stage: no atomics.
//
// Mish: forward y = x*t with t = tanh(softplus(x)) = n/(n+2), n = e^x*(e^x+2); backward
// recomputes t and sigmoid(x) from x alone, 1 - t^2 = w*(2-w) with w = 2/(n+2) (no
// cancellation).  16 bytes per lane, grid-stride.
#include "../../include/dnnops.h"
#include "mbconv_dev.h"
#include "mbconv_launch.h"

#include <algorithm>
#include <mutex>

namespace mbk {
namespace {

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}

// ---- Mish ---------------------------------------------------------------------------------
__device__ __forceinline__ float mish_t(float x, float &w)
{
    // t = tanh(log(1+e^x)) = n/(n+2), w = 1 - t = 2/(n+2); beyond x = 20 the difference from 1
    // is below fp32 resolution and e^x*(e^x+2) would overflow
    const float e = __expf(fminf(x, 20.0f));
    const float n = e * (e + 2.0f);
    w = 2.0f * __builtin_amdgcn_rcpf(n + 2.0f);
    return 1.0f - w;
}
__device__ __forceinline__ float mish_val(float x)
{
    float w;
    return x * mish_t(x, w);
}
__device__ __forceinline__ float mish_grad(float x)
{
    float w;
    const float t = mish_t(x, w);
    const float s = sigmoidf_fast(x);
    return fmaf(x * s, w * (2.0f - w), t);
}

// Four 16-byte runs per thread and round, all loads of a round issued before the first use (a
// load-use-store loop would pay one memory round trip per run).
template <bool BWD>
__global__ __launch_bounds__(256) void mish_kernel(const float *__restrict__ x, const float *dy,
                                                   float *out, size_t n)
{
    constexpr int U = 4;
    const size_t n4 = n / 4;
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t i0 = (size_t)blockIdx.x * 256 + threadIdx.x; i0 < n4; i0 += U * stride) {
        float4 xv[U], g[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t i = min(i0 + u * stride, n4 - 1); // clamped: always a valid run
            xv[u] = reinterpret_cast<const float4 *>(x)[i];
            if (BWD)
                g[u] = reinterpret_cast<const float4 *>(dy)[i];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float4 r;
            if (BWD)
                r = make_float4(g[u].x * mish_grad(xv[u].x), g[u].y * mish_grad(xv[u].y),
                                g[u].z * mish_grad(xv[u].z), g[u].w * mish_grad(xv[u].w));
            else
                r = make_float4(mish_val(xv[u].x), mish_val(xv[u].y), mish_val(xv[u].z), mish_val(xv[u].w));
            if (i0 + u * stride < n4)
                reinterpret_cast<float4 *>(out)[i0 + u * stride] = r;
        }
    }
    if (blockIdx.x == 0) { // at most three trailing elements
        const size_t i = 4 * n4 + threadIdx.x;
        if (i < n)
            out[i] = BWD ? dy[i] * mish_grad(x[i]) : mish_val(x[i]);
    }
}

// ---- rows in registers ------------------------------------------------------------------------
// TPR threads own a row (a DPP row of 16 lanes up to 128 columns, a wavefront up to 2048, else the whole
// workgroup): thread t, vector j covers columns 4*(t + TPR*j) .. +3, cols >= 4, cols <= 4*TPR*NV.  Rows
// whose length is no multiple of four start at any 4-byte boundary (the 16-byte accesses of this chip
// may) and end in a partial vector: it is moved back to the row's last four columns, `own` tells the
// columns that no other thread covers, and both threads write the same values to the others.  Softmax
// of 48768 x 381, forward and backward: 64.9 us (5.7 TB/s); with a workgroup per row, the row in LDS and
// 4-byte accesses 108.0.  4000 x 8192: 112 us against 270.  The 16 lanes: 65536 x 45 10.9 us against 21.6
// with a wavefront per row.  RAG: cols % 4 != 0 (the masks cost 4096 x 1024 five per cent forward).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
template <int NV, int TPR, bool RAG>
struct RowRegs {
    float v[NV][4];
    // (row_nv takes the smallest form that holds the row: the first half of the vectors never reach its end)
    static __device__ __forceinline__ int start(int cols, int t, int j)
    {
        const int c = 4 * (t + TPR * j);
        return j < NV / 2 ? c : min(c, cols - 4);
    }
    static __device__ __forceinline__ bool own(int cols, int t, int j, int k)
    {
        const int c = 4 * (t + TPR * j);
        return j < NV / 2 || (c < cols && (!RAG || min(c, cols - 4) + k >= c));
    }
    __device__ __forceinline__ void load(const float *row, int cols, int t)
    {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const f32x4u x = *reinterpret_cast<const f32x4u *>(row + start(cols, t, j));
#pragma unroll
            for (int k = 0; k < 4; ++k)
                v[j][k] = x[k];
        }
    }
    __device__ __forceinline__ void store(float *row, int cols, int t) const
    {
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (j < NV / 2 || 4 * (t + TPR * j) < cols)
                *reinterpret_cast<f32x4u *>(row + start(cols, t, j)) = (f32x4u){v[j][0], v[j][1], v[j][2], v[j][3]};
    }
};

__device__ __forceinline__ float row16_max(float v)
{
#define MBK_STEP(ctrl)                                                                            \
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, 0xf, 0xf, false)));
    MBK_STEP(0x128) // row_ror:8
    MBK_STEP(0x124)
    MBK_STEP(0x122)
    MBK_STEP(0x121)
#undef MBK_STEP
    return v;
}

// Sum (or maximum) over the TPR threads of a row, the same bits in all of them.
template <int TPR>
__device__ __forceinline__ float row_reduce(float v, float *red, bool is_max)
{
    if (TPR == 16)
        return is_max ? row16_max(v) : row16_sum(v);
    v = is_max ? wave_max(v) : wave_sum(v);
    if (TPR == kWave)
        return v;
    __syncthreads(); // red may still be read from the previous reduction
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = red[0];
#pragma unroll
    for (int i = 1; i < 4; ++i)
        r = is_max ? fmaxf(r, red[i]) : r + red[i];
    return r;
}

template <int NV, int TPR, bool RAG>
__global__ __launch_bounds__(256) void layernorm_fwd_kernel(const float *__restrict__ x,
                                                            const float *__restrict__ gamma,
                                                            const float *__restrict__ beta, float eps,
                                                            int rows, int cols, float *y, float *mean,
                                                            float *rstd)
{
    __shared__ float red[4];
    const int t = threadIdx.x % TPR;
    const int first = blockIdx.x * (256 / TPR) + threadIdx.x / TPR, step = gridDim.x * (256 / TPR);
    RowRegs<NV, TPR, RAG> g, b;
    g.load(gamma, cols, t);
    b.load(beta, cols, t);
    const float inv = 1.0f / (float)cols;
    for (int r = first; r < rows; r += step) {
        RowRegs<NV, TPR, RAG> a;
        a.load(x + (size_t)r * cols, cols, t);
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                s += a.own(cols, t, j, k) ? a.v[j][k] : 0.f;
        const float mu = row_reduce<TPR>(s, red, false) * inv;
        float s2 = 0.f;
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float d = a.own(cols, t, j, k) ? a.v[j][k] - mu : 0.f;
                s2 = fmaf(d, d, s2);
            }
        const float rs = 1.0f / sqrtf(row_reduce<TPR>(s2, red, false) * inv + eps);
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                a.v[j][k] = fmaf(g.v[j][k], (a.v[j][k] - mu) * rs, b.v[j][k]);
        a.store(y + (size_t)r * cols, cols, t);
        if (t == 0) {
            mean[r] = mu;
            rstd[r] = rs;
        }
    }
}

// Rows of up to 1024 (4096): the next row is requested before this one is reduced.  With 16 rows per
// workgroup there are few wavefronts, and their loads have to overlap the reductions (4096 x 1024:
// 10.5 us; 11.5 without).  Longer rows have no registers for it.
template <int NV, int TPR, bool RAG>
__global__ __launch_bounds__(256) void layernorm_bwd_kernel(const float *__restrict__ x,
                                                            const float *__restrict__ dy,
                                                            const float *__restrict__ gamma,
                                                            const float *__restrict__ mean,
                                                            const float *__restrict__ rstd, int rows,
                                                            int cols, float *dx, float *pgamma,
                                                            float *pbeta)
{
    __shared__ float red[4];
    const int t = threadIdx.x % TPR;
    const int first = blockIdx.x * (256 / TPR) + threadIdx.x / TPR, step = gridDim.x * (256 / TPR);
    RowRegs<NV, TPR, RAG> g, ag, ab, na, nd;
    g.load(gamma, cols, t);
#pragma unroll
    for (int j = 0; j < NV; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k)
            ag.v[j][k] = ab.v[j][k] = 0.f;
    const float inv = 1.0f / (float)cols;
    constexpr bool AHEAD = NV <= 4;
    const auto fetch = [&](int r) __attribute__((always_inline)) {
        na.load(x + (size_t)r * cols, cols, t);
        nd.load(dy + (size_t)r * cols, cols, t);
    };
    if (AHEAD && first < rows)
        fetch(first);
    for (int r = first; r < rows; r += step) {
        RowRegs<NV, TPR, RAG> a, d;
        if (AHEAD) {
            a = na;
            d = nd;
        } else {
            a.load(x + (size_t)r * cols, cols, t);
            d.load(dy + (size_t)r * cols, cols, t);
            __builtin_amdgcn_sched_barrier(0);
        }
        const float mu = mean[r], rs = rstd[r];
        if (AHEAD)
            fetch(min(r + step, rows - 1)); // (past the end the last row again, never used)
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float xh = (a.v[j][k] - mu) * rs;
                const float gg = d.v[j][k] * g.v[j][k];
                ag.v[j][k] = fmaf(d.v[j][k], xh, ag.v[j][k]);
                ab.v[j][k] += d.v[j][k];
                a.v[j][k] = xh;
                d.v[j][k] = gg;
                // (the sums are selected, not the terms: a masked term could still be 0 * infinity)
                s1 = a.own(cols, t, j, k) ? s1 + gg : s1;
                s2 = a.own(cols, t, j, k) ? fmaf(gg, xh, s2) : s2;
            }
        const float m1 = row_reduce<TPR>(s1, red, false) * inv, m2 = row_reduce<TPR>(s2, red, false) * inv;
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                d.v[j][k] = rs * (d.v[j][k] - m1 - a.v[j][k] * m2);
        d.store(dx + (size_t)r * cols, cols, t);
    }
    // one partial row per workgroup: the thread groups of different rows are added in a fixed order
    // through LDS (a workgroup per row: every column has one thread)
    if (TPR == 256) {
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (ag.own(cols, t, j, k)) {
                    const int c = ag.start(cols, t, j) + k;
                    pgamma[(size_t)blockIdx.x * cols + c] = ag.v[j][k];
                    pbeta[(size_t)blockIdx.x * cols + c] = ab.v[j][k];
                }
        return;
    }
    constexpr int G = 256 / TPR, GC = TPR == 256 ? 1 : 4 * TPR * NV;
    __shared__ float part[2][G][GC];
    const int grp = threadIdx.x / TPR;
#pragma unroll
    for (int j = 0; j < NV; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (ag.own(cols, t, j, k)) {
                const int c = (ag.start(cols, t, j) + k) % GC;
                part[0][grp][c] = ag.v[j][k];
                part[1][grp][c] = ab.v[j][k];
            }
    __syncthreads();
    const auto total = [&](int w, int c) {
        float s = 0.f;
#pragma unroll
        for (int u = 0; u < G; u += 4)
            s += (part[w][u][c % GC] + part[w][(u + 1) % G][c % GC]) + (part[w][(u + 2) % G][c % GC] + part[w][(u + 3) % G][c % GC]);
        return s;
    };
    if (TPR == 16) { // at most 128 columns
        if ((int)threadIdx.x < 2 * cols) {
            const int w = (int)threadIdx.x >= cols, c = threadIdx.x - w * cols;
            (w ? pbeta : pgamma)[(size_t)blockIdx.x * cols + c] = total(w, c);
        }
        return;
    }
    for (int c = threadIdx.x; c < cols; c += 256) {
        pgamma[(size_t)blockIdx.x * cols + c] = total(0, c);
        pbeta[(size_t)blockIdx.x * cols + c] = total(1, c);
    }
}

template <int NV, int TPR, bool RAG, bool BWD>
__global__ __launch_bounds__(256) void softmax_kernel(const float *__restrict__ in0, const float *in1, float *out,
                                                      int rows, int cols)
{
    __shared__ float red[4];
    const int t = threadIdx.x % TPR;
    const int first = blockIdx.x * (256 / TPR) + threadIdx.x / TPR, step = gridDim.x * (256 / TPR);
    for (int r = first; r < rows; r += step) {
        RowRegs<NV, TPR, RAG> a;
        a.load(in0 + (size_t)r * cols, cols, t);
        if (!BWD) {
            float m = -INFINITY;
#pragma unroll
            for (int j = 0; j < NV; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k) // (columns read twice, or past the end: another thread's as well)
                    m = fmaxf(m, a.v[j][k]);
            m = row_reduce<TPR>(m, red, true);
            float s = 0.f;
#pragma unroll
            for (int j = 0; j < NV; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    a.v[j][k] = __expf(a.v[j][k] - m);
                    s += a.own(cols, t, j, k) ? a.v[j][k] : 0.f;
                }
            const float is = 1.0f / row_reduce<TPR>(s, red, false);
#pragma unroll
            for (int j = 0; j < NV; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    a.v[j][k] *= is;
        } else {
            RowRegs<NV, TPR, RAG> d;
            d.load(in1 + (size_t)r * cols, cols, t); // dy (in0 is y)
            float s = 0.f;
#pragma unroll
            for (int j = 0; j < NV; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    s = a.own(cols, t, j, k) ? fmaf(d.v[j][k], a.v[j][k], s) : s; // (not 0 * dy: dy may be infinite)
            s = row_reduce<TPR>(s, red, false);
#pragma unroll
            for (int j = 0; j < NV; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    a.v[j][k] *= d.v[j][k] - s;
        }
        a.store(out + (size_t)r * cols, cols, t);
    }
}

// ---- rows of one to three columns: a thread per row ------------------------------------------------
// mode 0: layer-norm forward, 1: layer-norm backward (dx only; the column sums are taken by
// ln_colsum_kernel), 2: softmax forward, 3: softmax backward.
template <int MODE>
__global__ __launch_bounds__(256) void row_short_kernel(const float *__restrict__ in0, const float *in1,
                                                        const float *__restrict__ gamma,
                                                        const float *__restrict__ beta, float eps,
                                                        int rows, int cols, float *out, float *mean,
                                                        float *rstd)
{
    const float inv = 1.0f / (float)cols;
    for (int r = blockIdx.x * 256 + threadIdx.x; r < rows; r += gridDim.x * 256) {
        const size_t o = (size_t)r * cols;
        float a[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 0.f};
        for (int c = 0; c < cols; ++c) {
            a[c] = in0[o + c];
            if (MODE == 1 || MODE == 3)
                d[c] = in1[o + c];
        }
        if (MODE == 0) {
            const float mu = (a[0] + a[1] + a[2]) * inv;
            float s2 = 0.f;
            for (int c = 0; c < cols; ++c)
                s2 = fmaf(a[c] - mu, a[c] - mu, s2);
            const float rs = 1.0f / sqrtf(s2 * inv + eps);
            for (int c = 0; c < cols; ++c)
                out[o + c] = fmaf(gamma[c], (a[c] - mu) * rs, beta[c]);
            mean[r] = mu;
            rstd[r] = rs;
        } else if (MODE == 1) { // in0 = x, in1 = dy
            const float mu = mean[r], rs = rstd[r];
            float s1 = 0.f, s2 = 0.f;
            for (int c = 0; c < cols; ++c) {
                const float gg = d[c] * gamma[c];
                s1 += gg;
                s2 = fmaf(gg, (a[c] - mu) * rs, s2);
            }
            for (int c = 0; c < cols; ++c)
                out[o + c] = rs * (d[c] * gamma[c] - s1 * inv - (a[c] - mu) * rs * (s2 * inv));
        } else if (MODE == 2) {
            float m = -INFINITY, s = 0.f;
            for (int c = 0; c < cols; ++c)
                m = fmaxf(m, a[c]);
            for (int c = 0; c < cols; ++c) {
                a[c] = __expf(a[c] - m);
                s += a[c];
            }
            const float is = 1.0f / s;
            for (int c = 0; c < cols; ++c)
                out[o + c] = a[c] * is;
        } else { // in0 = y, in1 = dy
            const float s = fmaf(a[0], d[0], fmaf(a[1], d[1], a[2] * d[2]));
            for (int c = 0; c < cols; ++c)
                out[o + c] = a[c] * (d[c] - s);
        }
    }
}

// Column sums for the layer-norm backward of such rows: workgroup (column block of 64, row slice)
// writes partial[slice][cols] for dgamma and dbeta; rows are added in ascending order.
__global__ __launch_bounds__(256) void ln_colsum_kernel(const float *__restrict__ x,
                                                        const float *__restrict__ dy,
                                                        const float *__restrict__ mean,
                                                        const float *__restrict__ rstd, int rows,
                                                        int cols, int rowsPerSlice, float *pgamma,
                                                        float *pbeta)
{
    __shared__ float red[2][4][64];
    const int c = blockIdx.x * 64 + (threadIdx.x & 63), q = threadIdx.x >> 6;
    const int r0 = blockIdx.y * rowsPerSlice, r1 = min(r0 + rowsPerSlice, rows);
    float sg = 0.f, sb = 0.f;
    if (c < cols)
        for (int r = r0 + q; r < r1; r += 4) {
            const float d = dy[(size_t)r * cols + c];
            sg = fmaf(d, (x[(size_t)r * cols + c] - mean[r]) * rstd[r], sg);
            sb += d;
        }
    red[0][q][threadIdx.x & 63] = sg;
    red[1][q][threadIdx.x & 63] = sb;
    __syncthreads();
    if (q == 0 && c < cols) {
        const int l = threadIdx.x;
        pgamma[(size_t)blockIdx.y * cols + c] = (red[0][0][l] + red[0][1][l]) + (red[0][2][l] + red[0][3][l]);
        pbeta[(size_t)blockIdx.y * cols + c] = (red[1][0][l] + red[1][1][l]) + (red[1][2][l] + red[1][3][l]);
    }
}

// ---- host side ----------------------------------------------------------------------------------
bool bad_align(const void *p) { return ((uintptr_t)p & 15u) != 0; }

// form of the row kernels: 1, 2, 4, 8: that many vectors per thread with a wavefront per row (129 to
// 2048 columns); -1, -2: one and two with 16 lanes per row; 16, 32: four and eight with a workgroup per
// row; 0: rows of less than four columns
int row_nv(int cols)
{
    if (cols < 4)
        return 0;
    if (cols <= 128)
        return cols <= 64 ? -1 : -2;
    if (cols > 2048)
        return cols <= 4096 ? 16 : 32;
    return cols <= 256 ? 1 : cols <= 512 ? 2 : cols <= 1024 ? 4 : 8;
}
int row_grid(int rows, int nv) // a workgroup's rows (16, four, or one) in flight, at most 2048 workgroups
{
    const int g = nv >= 16 ? rows : nv < 0 ? (rows + 15) / 16 : (rows + 3) / 4;
    return g < 1 ? 1 : (g > 2048 ? 2048 : g);
}
int row_grid_bwd(int rows) // sixteen rows per workgroup, at most 512 partial rows
{
    const int g = (rows + 15) / 16;
    return g < 1 ? 1 : (g > 512 ? 512 : g);
}
int short_grid(int rows) { return std::min((rows + 255) / 256, 4096); }
int ln_slices(int rows) // row slices of the column sums of rows of less than four columns
{
    const int s = (rows + 63) / 64;
    return s > 256 ? 256 : (s < 1 ? 1 : s);
}
// Partial rows of the layer-norm weight gradients (one per workgroup of the backward kernel).  Rows
// longer than 2048: a workgroup per row up to 256, and no more than the 8 MiB of the static scratch
// hold wherever one per 64 rows fits into them (the shapes the entry point without scratch takes).
int ln_parts(int rows, int cols)
{
    const int nv = row_nv(cols);
    if (!nv)
        return ln_slices(rows);
    if (nv < 16)
        return row_grid_bwd(rows);
    const int fits = (1 << 20) / cols;
    return ln_slices(rows) > fits ? ln_slices(rows) : std::min(rows, std::min(fits, 256));
}

} // namespace
} // namespace mbk

using namespace mbk;

// ---- scratch for callers that cannot allocate --------------------------------------------------
// dnnops_layernorm_backward_noalloc keeps the partial sums of the two weight gradients in this
// array instead of a caller's workspace.  One copy exists on every GPU the library runs on, from
// the time the code object is loaded until the process ends.  In host code the array's name is
// only a handle for hipGetSymbolAddress: the device address is looked up once per device, with
// that device current, and kept in g_ln_scratch_ptr; kernels and the second stage receive that
// address as an ordinary pointer argument.
#define DNNOPS_STATIC_SCRATCH_BYTES (8u << 20)
static __device__ __align__(256) unsigned char ln_static_scratch[DNNOPS_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_ln_scratch_mutex;
void *g_ln_scratch_ptr[kMaxDevices] = {};

// Device address of this GPU's copy of ln_static_scratch (nullptr on failure).
void *ln_static_scratch_ptr()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
        return nullptr;
    std::lock_guard<std::mutex> lock(g_ln_scratch_mutex);
    if (!g_ln_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(ln_static_scratch)) != hipSuccess || !ptr)
            return nullptr;
        g_ln_scratch_ptr[dev] = ptr;
    }
    return g_ln_scratch_ptr[dev];
}
} // namespace

extern "C" {

dnnops_status dnnops_mish_forward(const float *x, float *y, size_t n, void *hip_stream)
{
    if (!x || !y || n == 0)
        return DNNOPS_EINVAL;
    if (bad_align(x) || bad_align(y))
        return DNNOPS_EALIGN;
    const size_t wg = (n / 4 + 1023) / 1024; // four runs per thread
    const unsigned grid = (unsigned)(wg < 1 ? 1 : (wg > 65536 ? 65536 : wg));
    hipLaunchKernelGGL(mish_kernel<false>, dim3(grid), dim3(256), 0, (hipStream_t)hip_stream, x,
                       (const float *)nullptr, y, n);
    return hipGetLastError() == hipSuccess ? DNNOPS_OK : DNNOPS_EHIP;
}

dnnops_status dnnops_mish_backward(const float *x, const float *dy, float *dx, size_t n,
                                   void *hip_stream)
{
    if (!x || !dy || !dx || n == 0)
        return DNNOPS_EINVAL;
    if (bad_align(x) || bad_align(dy) || bad_align(dx))
        return DNNOPS_EALIGN;
    const size_t wg = (n / 4 + 1023) / 1024;
    const unsigned grid = (unsigned)(wg < 1 ? 1 : (wg > 65536 ? 65536 : wg));
    hipLaunchKernelGGL(mish_kernel<true>, dim3(grid), dim3(256), 0, (hipStream_t)hip_stream, x, dy,
                       dx, n);
    return hipGetLastError() == hipSuccess ? DNNOPS_OK : DNNOPS_EHIP;
}

#define DNNOPS_FORM(n, v, tpr, ...)                                                               \
    case n: {                                                                                     \
        constexpr int NV = v, TPR = tpr;                                                          \
        if (cols % 4 != 0) {                                                                      \
            constexpr bool RAG = true;                                                            \
            __VA_ARGS__;                                                                          \
        } else {                                                                                  \
            constexpr bool RAG = false;                                                           \
            __VA_ARGS__;                                                                          \
        }                                                                                         \
    } break;
#define DNNOPS_NV_SWITCH(nv, ...)                                                                 \
    switch (nv) {                                                                                 \
        DNNOPS_FORM(-1, 1, 16, __VA_ARGS__)                                                       \
        DNNOPS_FORM(-2, 2, 16, __VA_ARGS__)                                                       \
        DNNOPS_FORM(1, 1, 64, __VA_ARGS__)                                                        \
        DNNOPS_FORM(2, 2, 64, __VA_ARGS__)                                                        \
        DNNOPS_FORM(4, 4, 64, __VA_ARGS__)                                                        \
        DNNOPS_FORM(8, 8, 64, __VA_ARGS__)                                                        \
        DNNOPS_FORM(16, 4, 256, __VA_ARGS__)                                                      \
        DNNOPS_FORM(32, 8, 256, __VA_ARGS__)                                                      \
    }

dnnops_status dnnops_layernorm_forward(const float *x, const float *gamma, const float *beta,
                                       float eps, int32_t rows, int32_t cols, float *y, float *mean,
                                       float *rstd, void *hip_stream)
{
    if (!x || !gamma || !beta || !y || !mean || !rstd || rows < 1 || cols < 1 || !(eps >= 0.f))
        return DNNOPS_EINVAL;
    if (cols > DNNOPS_MAX_COLS)
        return DNNOPS_EUNSUPPORTED;
    if (bad_align(x) || bad_align(gamma) || bad_align(beta) || bad_align(y))
        return DNNOPS_EALIGN;
    hipStream_t st = (hipStream_t)hip_stream;
    const int nv = row_nv(cols);
    if (nv) {
        DNNOPS_NV_SWITCH(nv, hipLaunchKernelGGL((layernorm_fwd_kernel<NV, TPR, RAG>), dim3(row_grid(rows, nv)), dim3(256),
                                                0, st, x, gamma, beta, eps, rows, cols, y, mean, rstd));
    } else {
        hipLaunchKernelGGL((row_short_kernel<0>), dim3(short_grid(rows)), dim3(256), 0, st, x, (const float *)nullptr, gamma, beta, eps, rows,
                           cols, y, mean, rstd);
    }
    return hipGetLastError() == hipSuccess ? DNNOPS_OK : DNNOPS_EHIP;
}

size_t dnnops_layernorm_backward_scratch_bytes(int32_t rows, int32_t cols)
{
    if (rows < 1 || cols < 1 || cols > DNNOPS_MAX_COLS)
        return 0;
    const size_t parts = (size_t)ln_parts(rows, cols);
    return 2 * parts * (size_t)cols * sizeof(float);
}

static dnnops_status layernorm_backward_check(const float *x, const float *dy, const float *gamma,
                                              const float *mean, const float *rstd, int32_t rows,
                                              int32_t cols, float *dx, float *dgamma, float *dbeta)
{
    if (!x || !dy || !gamma || !mean || !rstd || !dx || !dgamma || !dbeta || rows < 1 || cols < 1)
        return DNNOPS_EINVAL;
    if (cols > DNNOPS_MAX_COLS)
        return DNNOPS_EUNSUPPORTED;
    if (bad_align(x) || bad_align(dy) || bad_align(gamma) || bad_align(dx))
        return DNNOPS_EALIGN;
    return DNNOPS_OK;
}

// Both entry points: dx and the per-workgroup partial sums of dgamma, dbeta into `scratch`, then
// their fixed-order sum.  Every partial the second stage reads is written by the first.
static dnnops_status layernorm_backward_launch(const float *x, const float *dy, const float *gamma,
                                               const float *mean, const float *rstd, int32_t rows,
                                               int32_t cols, float *dx, float *dgamma, float *dbeta,
                                               void *scratch, hipStream_t st)
{
    const int nv = row_nv(cols);
    const int parts = ln_parts(rows, cols);
    float *pg = (float *)scratch;
    if (nv) {
        float *pb = pg + (size_t)parts * cols;
        DNNOPS_NV_SWITCH(nv, hipLaunchKernelGGL((layernorm_bwd_kernel<NV, TPR, RAG>), dim3(parts), dim3(256),
                                                0, st, x, dy, gamma, mean, rstd, rows, cols, dx, pg, pb));
    } else {
        float *pb = pg + (size_t)parts * cols;
        hipLaunchKernelGGL((row_short_kernel<1>), dim3(short_grid(rows)), dim3(256), 0, st, x, dy, gamma, (const float *)nullptr, 0.f,
                           rows, cols, dx, const_cast<float *>(mean), const_cast<float *>(rstd));
        const int per = (rows + parts - 1) / parts;
        hipLaunchKernelGGL(ln_colsum_kernel, dim3((cols + 63) / 64, parts), dim3(256), 0, st, x, dy,
                           mean, rstd, rows, cols, per, pg, pb);
    }
    if (hipGetLastError() != hipSuccess)
        return DNNOPS_EHIP;
    float *pb = pg + (size_t)parts * cols;
    if (launch_reduce_splits2({pg, parts, (size_t)cols, dgamma}, {pb, parts, (size_t)cols, dbeta}, st) !=
        hipSuccess)
        return DNNOPS_EHIP;
    return DNNOPS_OK;
}

dnnops_status dnnops_layernorm_backward(const float *x, const float *dy, const float *gamma,
                                        const float *mean, const float *rstd, int32_t rows,
                                        int32_t cols, float *dx, float *dgamma, float *dbeta,
                                        void *scratch, void *hip_stream)
{
    if (!scratch)
        return DNNOPS_EINVAL;
    const dnnops_status s = layernorm_backward_check(x, dy, gamma, mean, rstd, rows, cols, dx, dgamma, dbeta);
    if (s != DNNOPS_OK)
        return s;
    if (bad_align(scratch))
        return DNNOPS_EALIGN;
    return layernorm_backward_launch(x, dy, gamma, mean, rstd, rows, cols, dx, dgamma, dbeta, scratch,
                                     (hipStream_t)hip_stream);
}

size_t dnnops_layernorm_backward_noalloc_max_scratch_bytes(void) { return DNNOPS_STATIC_SCRATCH_BYTES; }

dnnops_status dnnops_layernorm_backward_noalloc(const float *x, const float *dy, const float *gamma,
                                                const float *mean, const float *rstd, int32_t rows,
                                                int32_t cols, float *dx, float *dgamma,
                                                float *dbeta, void *hip_stream)
{
    const dnnops_status s = layernorm_backward_check(x, dy, gamma, mean, rstd, rows, cols, dx, dgamma, dbeta);
    if (s != DNNOPS_OK)
        return s;
    // host-side size check ahead of any HIP call
    if (dnnops_layernorm_backward_scratch_bytes(rows, cols) > DNNOPS_STATIC_SCRATCH_BYTES)
        return DNNOPS_ESCRATCH;
    void *scratch = ln_static_scratch_ptr();
    if (!scratch)
        return DNNOPS_EHIP;
    return layernorm_backward_launch(x, dy, gamma, mean, rstd, rows, cols, dx, dgamma, dbeta, scratch,
                                     (hipStream_t)hip_stream);
}

static dnnops_status softmax_launch(bool bwd, const float *in0, const float *in1, float *out,
                                    int32_t rows, int32_t cols, void *hip_stream)
{
    if (!in0 || (bwd && !in1) || !out || rows < 1 || cols < 1)
        return DNNOPS_EINVAL;
    if (cols > DNNOPS_MAX_COLS)
        return DNNOPS_EUNSUPPORTED;
    if (bad_align(in0) || bad_align(in1) || bad_align(out))
        return DNNOPS_EALIGN;
    hipStream_t st = (hipStream_t)hip_stream;
    const int nv = row_nv(cols);
    if (nv) {
        if (bwd) {
            DNNOPS_NV_SWITCH(nv, hipLaunchKernelGGL((softmax_kernel<NV, TPR, RAG, true>), dim3(row_grid(rows, nv)),
                                                    dim3(256), 0, st, in0, in1, out, rows, cols));
        } else {
            DNNOPS_NV_SWITCH(nv, hipLaunchKernelGGL((softmax_kernel<NV, TPR, RAG, false>), dim3(row_grid(rows, nv)),
                                                    dim3(256), 0, st, in0, in1, out, rows, cols));
        }
    } else if (bwd) {
        hipLaunchKernelGGL((row_short_kernel<3>), dim3(short_grid(rows)), dim3(256), 0, st, in0, in1, (const float *)nullptr,
                           (const float *)nullptr, 0.f, rows, cols, out, (float *)nullptr,
                           (float *)nullptr);
    } else {
        hipLaunchKernelGGL((row_short_kernel<2>), dim3(short_grid(rows)), dim3(256), 0, st, in0, in1, (const float *)nullptr,
                           (const float *)nullptr, 0.f, rows, cols, out, (float *)nullptr,
                           (float *)nullptr);
    }
    return hipGetLastError() == hipSuccess ? DNNOPS_OK : DNNOPS_EHIP;
}

dnnops_status dnnops_softmax_forward(const float *x, float *y, int32_t rows, int32_t cols,
                                     void *hip_stream)
{
    return softmax_launch(false, x, nullptr, y, rows, cols, hip_stream);
}

dnnops_status dnnops_softmax_backward(const float *y, const float *dy, float *dx, int32_t rows,
                                      int32_t cols, void *hip_stream)
{
    return softmax_launch(true, y, dy, dx, rows, cols, hip_stream);
}

} // extern "C"
