// Small kernels: batch-norm statistics finalisation (forward and backward), the
// squeeze-and-excitation fully connected layers and their gradients, and the fixed-order
// second stage of the split reductions.  All of them touch O(N*C) values.
#include <algorithm>
#include "mbconv_x3.h"
#include "mbconv_bnfin.h"

namespace mbk {

// One wavefront per channel.  Partials are fp32 sums over at most a plane or a GEMM tile;
// they are combined in fp64 so that var = E[x^2]-E[x]^2 loses nothing in this stage.
// BN formula and running statistics: section "Statistical Normalization".
// PREP: the workgroups past the channels' write the weight images of convolutions later in the
// sequence (a launch of their own cost 4 to 5 us; this one's few workgroups leave the chip empty).
template <bool PREP>
__global__ __launch_bounds__(256) void bn_finalize_kernel(int C, int NP, double m,
                                                          const float *__restrict__ psum,
                                                          const float *__restrict__ psq,
                                                          const float *__restrict__ gamma,
                                                          const float *__restrict__ beta, float eps,
                                                          float momentum, float *run_mean,
                                                          float *run_var, float *bn, float *ones,
                                                          size_t ones_count, X3PrepArgs prep)
{
    if (PREP && (int)blockIdx.x >= (C + 3) / 4) {
        x3_prep_tile(prep, blockIdx.x - (C + 3) / 4, threadIdx.x);
        return;
    }
    // a block without squeeze-and-excitation has its gate buffer set to one here, by the launch
    // that precedes the gate's first reader anyway
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < ones_count; i += (size_t)((C + 3) / 4) * 256)
        ones[i] = 1.0f;
    const int c = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (c >= C)
        return;
    // everything the last step needs is requested up front, and the partials are read four
    // strides at a time, so the kernel costs a few memory round trips whatever NP is
    const float gm = gamma[c], bt = beta[c];
    // (a null running-stat pointer reads gamma instead: no branch in front of the loads)
    const float rm = (run_mean ? run_mean : gamma)[c], rv = (run_var ? run_var : gamma)[c];
    const float *ps = psum + (size_t)c * NP, *pq = psq + (size_t)c * NP;
    double s = 0.0, s2 = 0.0;
    int i0 = lane;
    // (many partials: sixteen strides at a time, in the same order.  conv_xk leaves one per 32 pixels: the
    // 30752 of 1024 31x31 images took 78 us with four strides, 26 now)
    for (; i0 + 15 * kWave < NP; i0 += 16 * kWave) {
        float a0[16], a1[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            a0[u] = ps[i0 + kWave * u];
            a1[u] = pq[i0 + kWave * u];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            s += (double)a0[u];
            s2 += (double)a1[u];
        }
    }
    for (; i0 < NP; i0 += 4 * kWave) {
        float a0[4], a1[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = min(i0 + kWave * u, NP - 1); // unconditional loads, masked below
            a0[u] = ps[i];
            a1[u] = pq[i];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (i0 + kWave * u < NP) {
                s += (double)a0[u];
                s2 += (double)a1[u];
            }
        }
    }
    s = wave_sum_d(s);
    s2 = wave_sum_d(s2);
    if (lane == 0) {
        // Divisions and a square root, although they are chains of a dozen fp64 instructions each: with a rounded 1/m a constant
        // channel's variance is not zero but its square times 2^-53, which a small eps does not cover.
        const double mean = s / m;
        double var = s2 / m - mean * mean;
        if (var < 0.0)
            var = 0.0;
        const double rstd = 1.0 / sqrt(var + (double)eps);
        const double scale = (double)gm * rstd;
        bn[c] = (float)scale;
        bn[C + c] = (float)((double)bt - mean * scale);
        bn[2 * C + c] = (float)mean;
        bn[3 * C + c] = (float)rstd;
        if (run_mean)
            run_mean[c] = (float)((1.0 - (double)momentum) * (double)rm + (double)momentum * mean);
        if (run_var) {
            const double unbiased = m > 1.0 ? var * m / (m - 1.0) : var;
            run_var[c] = (float)((1.0 - (double)momentum) * (double)rv + (double)momentum * unbiased);
        }
    }
}

hipError_t launch_bn_finalize(int C, int NP, double m, const float *psum, const float *psq,
                              const float *gamma, const float *beta, float eps, float momentum,
                              float *run_mean, float *run_var, float *bn, hipStream_t st,
                              float *ones, size_t ones_count, const X3PrepArgs *prep)
{
    const unsigned own = (unsigned)((C + 3) / 4);
    if (prep && prep->tiles)
        hipLaunchKernelGGL(bn_finalize_kernel<true>, dim3(own + prep->tiles), dim3(256), 0, st, C, NP, m, psum, psq,
                           gamma, beta, eps, momentum, run_mean, run_var, bn, ones, ones ? ones_count : 0, *prep);
    else
        hipLaunchKernelGGL(bn_finalize_kernel<false>, dim3(own), dim3(256), 0, st, C, NP, m, psum, psq, gamma, beta,
                           eps, momentum, run_mean, run_var, bn, ones, ones ? ones_count : 0, X3PrepArgs());
    return hipGetLastError();
}

__device__ __forceinline__ void bn_bwd_coef(int C, int c, double inv_m, double dgamma, double dbeta,
                                            float gamma, const float *bn, float *coef)
{
    bn_bwd_coef_vals(C, c, inv_m, dgamma, dbeta, gamma, bn[2 * C + c], bn[3 * C + c], coef);
}

__device__ __forceinline__ void bn_bwd_finalize_body(int block, int C, int NP, double inv_m,
                                                     const float *__restrict__ psb,
                                                     const float *__restrict__ psr,
                                                     const float *__restrict__ gamma,
                                                     const float *__restrict__ bn, float *dgamma,
                                                     float *dbeta, float *coef)
{
    const int c = block * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (c >= C)
        return;
    const float gm = gamma[c], mean = bn[2 * C + c], rstd = bn[3 * C + c]; // requested up front
    const float *pb = psb + (size_t)c * NP, *pr = psr + (size_t)c * NP;
    double sb = 0.0, sr = 0.0;
    for (int i0 = lane; i0 < NP; i0 += 4 * kWave) {
        float a0[4], a1[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = min(i0 + kWave * u, NP - 1); // unconditional loads, masked below
            a0[u] = pb[i];
            a1[u] = pr[i];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (i0 + kWave * u < NP) {
                sb += (double)a0[u];
                sr += (double)a1[u];
            }
        }
    }
    sb = wave_sum_d(sb);
    sr = wave_sum_d(sr);
    if (lane == 0) {
        if (dbeta)
            dbeta[c] = (float)sb;
        if (dgamma)
            dgamma[c] = (float)sr;
        bn_bwd_coef_vals(C, c, inv_m, sr, sb, gm, mean, rstd, coef);
    }
}

__global__ __launch_bounds__(256) void bn_bwd_finalize_kernel(int C, int NP, double inv_m,
                                                              const float *__restrict__ psb,
                                                              const float *__restrict__ psr,
                                                              const float *__restrict__ gamma,
                                                              const float *__restrict__ bn,
                                                              float *dgamma, float *dbeta,
                                                              float *coef)
{
    bn_bwd_finalize_body(blockIdx.x, C, NP, inv_m, psb, psr, gamma, bn, dgamma, dbeta, coef);
}

// Block without squeeze-and-excitation: one wavefront per channel adds the plane sums of the
// batch in a fixed order (lane l takes images l, l+64, ...; fp64 butterfly), writes BN2's
// parameter gradients and backward coefficients, and zeroes the channel's column of dzs.
__global__ __launch_bounds__(256) void bn2_bwd_nose_kernel(int N, int C, double inv_m,
                                                           const float *__restrict__ A1,
                                                           const float *__restrict__ A2,
                                                           const float *__restrict__ gamma,
                                                           const float *__restrict__ bn,
                                                           float *dgamma, float *dbeta, float *coef,
                                                           float *dzs)
{
    const int c = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (c >= C)
        return;
    double sb = 0.0, sr = 0.0;
    for (int n = lane; n < N; n += kWave) {
        sb += (double)A1[(size_t)n * C + c];
        sr += (double)A2[(size_t)n * C + c];
        dzs[(size_t)n * C + c] = 0.f;
    }
    sb = wave_sum_d(sb);
    sr = wave_sum_d(sr);
    if (lane == 0) {
        dbeta[c] = (float)sb;
        dgamma[c] = (float)sr;
        bn_bwd_coef(C, c, inv_m, sr, sb, gamma[c], bn, coef);
    }
}

hipError_t launch_bn2_bwd_nose(int N, int C, double m, const float *A1, const float *A2,
                               const float *gamma, const float *bn, float *dgamma, float *dbeta,
                               float *coef, float *dzs, hipStream_t st)
{
    hipLaunchKernelGGL(bn2_bwd_nose_kernel, dim3((C + 3) / 4), dim3(256), 0, st, N, C, 1.0 / m, A1, A2,
                       gamma, bn, dgamma, dbeta, coef, dzs);
    return hipGetLastError();
}

hipError_t launch_bn_bwd_finalize(int C, int NP, double m, const float *psb, const float *psr,
                                  const float *gamma, const float *bn, float *dgamma,
                                  float *dbeta, float *coef, hipStream_t st)
{
    hipLaunchKernelGGL(bn_bwd_finalize_kernel, dim3((C + 3) / 4), dim3(256), 0, st, C, NP, 1.0 / m, psb,
                       psr, gamma, bn, dgamma, dbeta, coef);
    return hipGetLastError();
}

// ---- squeeze-and-excitation --------------------------------------------------------------------
// One workgroup per image.  q = W1 z + b1 (a wavefront per output, lanes stride over C),
// r = swish(q), g = sigmoid(W2 r + b2) (a thread per channel).

// (PARTS: z is a sum of several arrays)
template <bool PARTS>
__global__ __launch_bounds__(256) void se_fwd_kernel(int C, int Cse, const float *__restrict__ z,
                                                     int nz, const float *__restrict__ w1,
                                                     const float *__restrict__ b1,
                                                     const float *__restrict__ w2,
                                                     const float *__restrict__ b2, float *q,
                                                     float *g)
{
    extern __shared__ float lds[];
    float *zs = lds, *rs = lds + C;
    const int n = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int c = tid; c < C; c += 256) {
        float v = z[(size_t)n * C + c];
#pragma unroll 4
        for (int s = 1; PARTS && s < nz; ++s)
            v += z[((size_t)s * gridDim.x + n) * C + c];
        zs[c] = v;
    }
    __syncthreads();
    for (int j = wave; j < Cse; j += 4) {
        float acc = 0.f;
        for (int c = lane; c < C; c += kWave)
            acc = fmaf(w1[(size_t)j * C + c], zs[c], acc);
        acc = wave_sum(acc);
        if (lane == 0) {
            const float qv = acc + b1[j];
            q[(size_t)n * Cse + j] = qv;
            rs[j] = swishf(qv);
        }
    }
    __syncthreads();
    for (int c = tid; c < C; c += 256) {
        float acc = b2[c];
        for (int j = 0; j < Cse; ++j)
            acc = fmaf(w2[(size_t)c * Cse + j], rs[j], acc);
        g[(size_t)n * C + c] = sigmoidf_fast(acc);
    }
}

// The same for 128 to 2048 channels and 4 to 64 squeezed ones: a workgroup of 1024 threads per (image,
// channel slice).  What bounds it is the chain of memory round trips (about a microsecond each), so a
// wavefront owns at most four rows of W1 and every load of the kernel - z, the wavefront's rows of W1
// (16*CI bytes per lane and row), the thread's part of its channel's row of W2 - is requested before
// the first one is used.  Every workgroup of an image recomputes the whole of q, which keeps the
// kernel free of a grid-wide dependency.  (One image: 480 -> 20 channels 4.1 us, 1152 -> 48 6.3; with
// 256 threads and 16 rows of W1 at a time 6.6 and 11.  Batch 64: 4.7 and 8.1 against 4.7 and 12.3.
// The same form of the backward kernel measured no faster, 6.8 and 11.4 against 6.8 and 11, and is not
// used.)
// Rows whose length is no multiple of four are read in pieces of four that are clamped to the row's
// end; the elements a piece shares with the one before it are masked, in both factors: either may be
// infinite.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
template <int CI, int JR, bool PARTS>
__global__ __launch_bounds__(1024) void se_fwd_wide_kernel(int C, int Cse, int slice,
                                                           const float *__restrict__ z, int nz,
                                                           const float *__restrict__ w1,
                                                           const float *__restrict__ b1,
                                                           const float *__restrict__ w2,
                                                           const float *__restrict__ b2, float *q,
                                                           float *g)
{
    constexpr int RU = JR * CI <= 15 ? JR : 10 / CI > 1 ? 10 / CI : 1; // rows of W1 in flight (128 registers)
    constexpr int FULL = CI == 5 || CI == 8 ? CI - 2 : CI - 1; // pieces of a row that end before C in every lane
    __shared__ float rs[64];
    const int n = blockIdx.x, sl = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    f32x4u zv[CI], wv[RU][CI], w2v[JR];
    const auto fetch_w1 = [&](int u) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < CI; ++i)
            wv[u % RU][i] = *reinterpret_cast<const f32x4u *>(w1 + (size_t)min(wave + 16 * u, Cse - 1) * C +
                                                              min(4 * (lane + 64 * i), C - 4));
    };
#pragma unroll
    for (int i = 0; i < CI; ++i)
        zv[i] = *reinterpret_cast<const f32x4u *>(z + (size_t)n * C + min(4 * (lane + 64 * i), C - 4));
#pragma unroll
    for (int u = 0; u < RU; ++u)
        fetch_w1(u);
    // W2: four threads per channel, thread t%4 takes the pieces t%4, t%4 + 4, ...
    const int part = tid & 3, cend = min(C, (sl + 1) * slice);
    int c = sl * slice + (tid >> 2);
    const auto fetch_w2 = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < JR; ++v)
            w2v[v] = *reinterpret_cast<const f32x4u *>(w2 + (size_t)min(ch, C - 1) * Cse +
                                                       min(4 * (part + 4 * v), Cse - 4));
    };
    fetch_w2(c);
#pragma unroll 1
    for (int s = 1; PARTS && s < nz; ++s)
#pragma unroll
        for (int i = 0; i < CI; ++i)
            zv[i] += *reinterpret_cast<const f32x4u *>(z + ((size_t)s * gridDim.x + n) * C + min(4 * (lane + 64 * i), C - 4));
    __builtin_amdgcn_sched_barrier(0);
    const auto own = [&](int i, int e) { return min(4 * (lane + 64 * i), C - 4) + e >= 4 * (lane + 64 * i); };
#pragma unroll
    for (int i = FULL; i < CI; ++i) // (a piece past the end, or the part of one that another lane has)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            zv[i][e] = own(i, e) ? zv[i][e] : 0.f;
#pragma unroll
    for (int u = 0; u < JR; ++u) {
        const int j = wave + 16 * u;
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < CI; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc = fmaf(i < FULL || own(i, e) ? wv[u % RU][i][e] : 0.f, zv[i][e], acc);
        if (u + RU < JR)
            fetch_w1(u + RU);
        acc = wave_sum(acc);
        if (lane == 0) {
            const float qv = acc + b1[min(j, Cse - 1)];
            if (sl == 0 && j < Cse)
                q[(size_t)n * Cse + j] = qv;
            rs[j] = j < Cse ? swishf(qv) : 0.f;
        }
        if (RU < JR)
            __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    for (; c < cend; c += 256) { // (once, unless the slice is the whole of a wide block)
        float acc = 0.f;
#pragma unroll
        for (int v = 0; v < JR; ++v) {
            const int want = 4 * (part + 4 * v), at = min(want, Cse - 4);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc = fmaf(at + e >= want ? w2v[v][e] : 0.f, at + e >= want ? rs[at + e] : 0.f, acc);
        }
        if (c + 256 < sl * slice + slice) // (uniform over the workgroup but for the last round)
            fetch_w2(c + 256);
        acc += __shfl_xor(acc, 1, kWave);
        acc += __shfl_xor(acc, 2, kWave);
        if (part == 0)
            g[(size_t)n * C + c] = sigmoidf_fast(acc + b2[c]);
    }
}

hipError_t launch_se_fwd(int N, int C, int Cse, const float *z, int nz, const float *w1, const float *b1,
                         const float *w2, const float *b2, float *q, float *g, hipStream_t st)
{
    // (128 channels and more: 240 -> 10, batch 64, 7.8 -> 4.8 us; 96 -> 4, two images, no faster)
    if (C >= 128 && C <= 2048 && Cse >= 4 && Cse <= 64) {
        // channel slices per image: as many as leave one workgroup per compute unit, since every one of
        // them computes the whole of q (1152 -> 48: 64 images, four slices 9.0 us, five 12.8; 128, two
        // 10.0, five 17.1; 512, one 20.5, five 49.5)
        const int G = std::max(1, std::min(8, std::min(256 / N, (C + 63) / 64)));
        const int slice = (C + G - 1) / G, ci = (C + 255) / 256, jr = (Cse + 15) / 16;
#define MBK_CASE(CI_, JR_)                                                                        \
    if (ci <= CI_ && jr == JR_) {                                                                 \
        if (nz > 1)                                                                               \
            hipLaunchKernelGGL((se_fwd_wide_kernel<CI_, JR_, true>), dim3(N, G), dim3(1024), 0, st, C, Cse, \
                               slice, z, nz, w1, b1, w2, b2, q, g);                               \
        else                                                                                      \
            hipLaunchKernelGGL((se_fwd_wide_kernel<CI_, JR_, false>), dim3(N, G), dim3(1024), 0, st, C, Cse, \
                               slice, z, nz, w1, b1, w2, b2, q, g);                               \
        return hipGetLastError();                                                                 \
    }
#define MBK_CI(CI_) MBK_CASE(CI_, 1) MBK_CASE(CI_, 2) MBK_CASE(CI_, 3) MBK_CASE(CI_, 4)
        MBK_CI(1)
        MBK_CI(2)
        MBK_CI(3)
        MBK_CI(5)
        MBK_CI(6)
        MBK_CI(8)
#undef MBK_CI
#undef MBK_CASE
    }
    const size_t lds = sizeof(float) * (C + Cse);
    if (nz > 1)
        hipLaunchKernelGGL((se_fwd_kernel<true>), dim3(N), dim3(256), lds, st, C, Cse, z, nz, w1, b1, w2, b2, q, g);
    else
        hipLaunchKernelGGL((se_fwd_kernel<false>), dim3(N), dim3(256), lds, st, C, Cse, z, nz, w1, b1, w2, b2, q, g);
    return hipGetLastError();
}

// Backward, per image: dt = dg*g*(1-g); dq = (W2^T dt)*swish'(q); dzs = (W1^T dq)/HW.
__global__ __launch_bounds__(256) void se_bwd_image_kernel(SeBwdArgs a)
{
    extern __shared__ float lds[];
    float *dts = lds, *dqs = lds + a.C;
    const int n = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int C = a.C, Cse = a.Cse;
    for (int c = tid; c < C; c += 256) {
        const float gv = a.g[(size_t)n * C + c];
        const float v = a.dg[(size_t)n * C + c] * gv * (1.f - gv);
        dts[c] = v;
        a.dt[(size_t)n * C + c] = v;
    }
    __syncthreads();
    for (int j = wave; j < Cse; j += 4) {
        float acc = 0.f;
        for (int c = lane; c < C; c += kWave)
            acc = fmaf(a.w2[(size_t)c * Cse + j], dts[c], acc);
        acc = wave_sum(acc);
        if (lane == 0) {
            float val, grad;
            swish_both(a.q[(size_t)n * Cse + j], val, grad);
            const float v = acc * grad;
            dqs[j] = v;
            a.dq[(size_t)n * Cse + j] = v;
        }
    }
    __syncthreads();
    const float inv = 1.f / (float)a.HW;
    for (int c = tid; c < C; c += 256) {
        float acc = 0.f;
        for (int j = 0; j < Cse; ++j)
            acc = fmaf(a.w1[(size_t)j * C + c], dqs[j], acc);
        a.dzs[(size_t)n * C + c] = acc * inv;
    }
}

// Sums over the batch.  Each output element is owned by 32 consecutive lanes: lane l adds
// the images l, l+32, ... and the 32 partial sums are combined by a fixed butterfly, so the
// result does not depend on scheduling.  Output elements in order:
//   [0, C*Cse)            dW2[c,j] = sum_n dt[n,c]*swish(q[n,j])
//   [C*Cse, 2*C*Cse)      dW1[j,c] = sum_n dq[n,j]*z[n,c]
//   next C                db2[c], and BN2's dbeta/dgamma/coef from the plane sums:
//                         dbeta2 = sum_n g*A1 + dzs*s3,  dgamma2 = sum_n g*A2 + dzs*s4
//   next Cse              db1[j]
__device__ __forceinline__ double half_wave_sum_d(double v)
{
#pragma unroll
    for (int o = 16; o > 0; o >>= 1)
        v += __shfl_xor(v, o, kWave);
    return v;
}

__global__ __launch_bounds__(256) void se_bwd_batch_kernel(SeBwdArgs a)
{
    const int C = a.C, Cse = a.Cse, N = a.N;
    const int ln = threadIdx.x & 31;
    int i = blockIdx.x * 8 + (threadIdx.x >> 5);
    if (i < C * Cse) {
        const int c = i / Cse, j = i - c * Cse;
        float acc = 0.f;
        for (int n = ln; n < N; n += 32)
            acc = fmaf(a.dt[(size_t)n * C + c], swishf(a.q[(size_t)n * Cse + j]), acc);
        acc = half_wave_sum(acc);
        if (ln == 0)
            a.dw2[i] = acc;
        return;
    }
    i -= C * Cse;
    if (i < C * Cse) {
        const int j = i / C, c = i - j * C;
        float acc = 0.f;
        for (int n = ln; n < N; n += 32)
            acc = fmaf(a.dq[(size_t)n * Cse + j], a.z[(size_t)n * C + c], acc);
        acc = half_wave_sum(acc);
        if (ln == 0)
            a.dw1[i] = acc;
        return;
    }
    i -= C * Cse;
    if (i < C) {
        const int c = i;
        float sb = 0.f;
        double dbeta = 0.0, dgamma = 0.0;
        for (int n = ln; n < N; n += 32) {
            const size_t o = (size_t)n * C + c;
            sb += a.dt[o];
            dbeta += (double)a.g[o] * a.A1[o] + (double)a.dzs[o] * a.s3[o];
            dgamma += (double)a.g[o] * a.A2[o] + (double)a.dzs[o] * a.s4[o];
        }
        sb = half_wave_sum(sb);
        dbeta = half_wave_sum_d(dbeta);
        dgamma = half_wave_sum_d(dgamma);
        if (ln == 0) {
            a.db2[c] = sb;
            a.dbeta2[c] = (float)dbeta;
            a.dgamma2[c] = (float)dgamma;
            bn_bwd_coef(C, c, a.inv_m, dgamma, dbeta, a.gamma2[c], a.bn2, a.coef2);
        }
        return;
    }
    i -= C;
    if (i < Cse) {
        float sb = 0.f;
        for (int n = ln; n < N; n += 32)
            sb += a.dq[(size_t)n * Cse + i];
        sb = half_wave_sum(sb);
        if (ln == 0)
            a.db1[i] = sb;
    }
}

// The two steps for 4 to 64 squeezed channels.  Both are a chain of memory round trips and nothing else, so
// every load of a kernel (of a round, for large batches and channel counts) is requested before the first
// is used, no product is computed twice, and what does not depend on each other has workgroups of its own.
//
// Step 1: a workgroup per image and sixteen squeezed channels.  dt = dg*g*(1-g) for all channels (the first
// slice stores it), dq = (W2^T dt)*swish'(q): four threads read 64 bytes of a row of W2, 64 rows at a
// time.  (1152 channels, 48 squeezed, 64 images, step 1 and 2: 11.8 + 8.1 us with the whole of W2 in every one of
// eight slices of channels and the dzs of a slice behind it; now 5.0 + 5.1, little above an
// empty launch.  672, 28, 128 images: 7.5 + 13.1 then, 4.8 + 5.7 now.)
__global__ __launch_bounds__(256) void se_bwd_dq_kernel(SeBwdArgs a)
{
    constexpr int U = 12; // rows in flight
    __shared__ float red[4][16];
    const int C = a.C, Cse = a.Cse, n = blockIdx.x, j0 = 16 * blockIdx.y;
    const int tid = threadIdx.x, part = tid & 3, row = tid >> 2;
    // (a piece that would end past the row is moved back; what it shares with the piece before it counts there)
    const int want = j0 + 4 * part, at = min(want, Cse - 4);
    const float *dg = a.dg + (size_t)n * C, *gt = a.g + (size_t)n * C;
    const float qv = a.q[(size_t)n * Cse + min(j0 + (tid & 15), Cse - 1)];
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int c0 = row; c0 < C; c0 += 64 * U) {
        f32x4u w[U];
        float dv[U], gv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = min(c0 + 64 * u, C - 1);
            dv[u] = dg[c];
            gv[u] = gt[c];
            w[u] = *reinterpret_cast<const f32x4u *>(a.w2 + (size_t)c * Cse + at);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + 64 * u;
            if (c < C) {
                const float dt = dv[u] * gv[u] * (1.f - gv[u]);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[e] = fmaf(w[u][e], dt, acc[e]);
                if (j0 == 0 && part == 0)
                    a.dt[(size_t)n * C + c] = dt;
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int o = 4; o < 64; o <<= 1)
            acc[e] += __shfl_xor(acc[e], o, kWave);
        // element e of the piece is squeezed channel at + e
        const int j = at + e - j0;
        if ((tid & 63) < 4 && at + e >= want && j < 16)
            red[tid >> 6][j] = acc[e];
    }
    __syncthreads();
    if (tid < 16 && j0 + tid < Cse) {
        float val, grad;
        swish_both(qv, val, grad);
        a.dq[(size_t)n * Cse + j0 + tid] = ((red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid])) * grad;
    }
}

// Step 2.  The first `chan` workgroups own sixteen channels: dzs = (W1^T dq)/HW for every image, and the batch
// sums of the channel: db2 = sum dt, BN2's dbeta = sum g*A1 + dzs*s3, dgamma = sum g*A2 + dzs*s4 and coefficients.
// The next `fc` have a tile of sixteen channels by sixteen squeezed ones per wavefront, of both weight
// gradients: dW2[c][j] = sum_n dt[n][c]*swish(q[n][j]), dW1[j][c] = sum_n dq[n][j]*z[n][c], fp32 MFMA on four
// images at a time, operands straight from memory.  The last adds db1[j] = sum_n dq[n][j].
__global__ __launch_bounds__(256) void se_bwd_sums_kernel(SeBwdArgs a, int chan, int fc)
{
    constexpr int TN = 64; // images a round
    __shared__ __attribute__((aligned(16))) float dqL[TN][64], w1L[64][16];
    __shared__ float sbL[16][16];
    __shared__ double dbL[16][16], dgL[16][16];
    const int C = a.C, Cse = a.Cse, N = a.N;
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < chan) {
        const int cl = tid & 15, nl = tid >> 4, c = 16 * blockIdx.x + cl, cc = min(c, C - 1);
        const int J4 = (Cse + 3) / 4;
        const float inv = 1.f / (float)a.HW;
        float wv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) // W1's column, squeezed channel nl + 16u
            wv[u] = and_mask(a.w1[(size_t)min(nl + 16 * u, Cse - 1) * C + cc], nl + 16 * u < Cse ? 0xffffffffu : 0u);
        const float gm = a.gamma2[cc], mean = a.bn2[2 * C + cc], rstd = a.bn2[3 * C + cc];
        float sb = 0.f;
        double dbeta = 0.0, dgamma = 0.0;
        for (int n0 = 0; n0 < N; n0 += TN) {
            // the round's dq, [image][squeezed channel], and the channel's own values of four images a thread
            float dv[TN * 64 / 256], dt[4], g[4], A1[4], A2[4], s3[4], s4[4];
#pragma unroll
            for (int u = 0; u < TN * 64 / 256; ++u) {
                const int nn = (tid >> 6) + 4 * u, j = tid & 63;
                dv[u] = a.dq[(size_t)min(n0 + nn, N - 1) * Cse + min(j, Cse - 1)];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const size_t o = (size_t)min(n0 + nl + 16 * u, N - 1) * C + cc;
                dt[u] = a.dt[o];
                g[u] = a.g[o];
                A1[u] = a.A1[o];
                A2[u] = a.A2[o];
                s3[u] = a.s3[o];
                s4[u] = a.s4[o];
            }
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < TN * 64 / 256; ++u)
                dqL[(tid >> 6) + 4 * u][tid & 63] = and_mask(dv[u], (tid & 63) < Cse ? 0xffffffffu : 0u);
            if (n0 == 0) {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    w1L[nl + 16 * u][cl] = wv[u];
            }
            __syncthreads();
            float dz[4] = {0.f, 0.f, 0.f, 0.f};
            for (int j4 = 0; j4 < J4; ++j4) { // (past the last squeezed channel both factors are zero: dq may be infinite)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float4 d4 = *reinterpret_cast<const float4 *>(&dqL[nl + 16 * u][4 * j4]);
                    dz[u] = fmaf(w1L[4 * j4][cl], d4.x, dz[u]);
                    dz[u] = fmaf(w1L[4 * j4 + 1][cl], d4.y, dz[u]);
                    dz[u] = fmaf(w1L[4 * j4 + 2][cl], d4.z, dz[u]);
                    dz[u] = fmaf(w1L[4 * j4 + 3][cl], d4.w, dz[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int n = n0 + nl + 16 * u;
                if (n < N && c < C) {
                    const float d = dz[u] * inv;
                    a.dzs[(size_t)n * C + c] = d;
                    sb += dt[u];
                    dbeta += (double)g[u] * A1[u] + (double)d * s3[u];
                    dgamma += (double)g[u] * A2[u] + (double)d * s4[u];
                }
            }
        }
        sbL[nl][cl] = sb;
        dbL[nl][cl] = dbeta;
        dgL[nl][cl] = dgamma;
        __syncthreads();
        if (nl == 0 && c < C) {
            sb = 0.f;
            dbeta = dgamma = 0.0;
            for (int u = 0; u < 16; ++u) {
                sb += sbL[u][cl];
                dbeta += dbL[u][cl];
                dgamma += dgL[u][cl];
            }
            a.db2[c] = sb;
            a.dbeta2[c] = (float)dbeta;
            a.dgamma2[c] = (float)dgamma;
            bn_bwd_coef_vals(C, c, a.inv_m, dgamma, dbeta, gm, mean, rstd, a.coef2);
        }
        return;
    }
    if ((int)blockIdx.x < chan + fc) {
        const int lane = tid & 63, r = lane & 15, g = lane >> 4, JT = (Cse + 15) / 16;
        const int tile = 4 * ((int)blockIdx.x - chan) + __builtin_amdgcn_readfirstlane(tid >> 6);
        const int c0 = 16 * (tile / JT), j0 = 16 * (tile % JT);
        if (c0 >= C)
            return;
        const int c = min(c0 + r, C - 1), j = min(j0 + r, Cse - 1);
        f32x4 acc2 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc2;
        for (int n0 = 0; n0 < N; n0 += 32) {
            float dt[8], z[8], q[8], dq[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const size_t n = (size_t)min(n0 + 4 * u + g, N - 1);
                dt[u] = a.dt[n * C + c];
                z[u] = a.z[n * C + c];
                q[u] = a.q[n * Cse + j];
                dq[u] = a.dq[n * Cse + j];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool ok = n0 + 4 * u + g < N;
                acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(ok ? dt[u] : 0.f, ok ? swishf(q[u]) : 0.f, acc2, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ok ? dq[u] : 0.f, ok ? z[u] : 0.f, acc1, 0, 0, 0);
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (c0 + 4 * g + v < C && j0 + r < Cse)
                a.dw2[(size_t)(c0 + 4 * g + v) * Cse + j0 + r] = acc2[v];
            if (j0 + 4 * g + v < Cse && c0 + r < C)
                a.dw1[(size_t)(j0 + 4 * g + v) * C + c0 + r] = acc1[v];
        }
        return;
    }
    // db1: four thread groups take every fourth image (sixteen loads in flight each), combined in a fixed order
    const int j = tid & 63, part = tid >> 6;
    float s = 0.f;
    if (j < Cse) {
#pragma unroll 16
        for (int n = part; n < N; n += 4)
            s += a.dq[(size_t)n * Cse + j];
    }
    dqL[part][j] = s;
    __syncthreads();
    if (tid < Cse)
        a.db1[tid] = (dqL[0][tid] + dqL[1][tid]) + (dqL[2][tid] + dqL[3][tid]);
}

// Few channels of few images: the plain kernels' shorter chain; backward of a block, plain / here, 96
// channels, 2 images 38.0 / 39.1 us, 32 images 44.7 / 45.0; 144, 8 images 37.7 / 38.0, 32 images 158 / 157; 240, 2
// images 46.5 / 45.8; the step alone, 16 channels, 2048 images 56.6 / 60.3, 32 channels 63.0 / 61.6.
bool se_bwd_tiled(int N, int C, int Cse)
{
    return Cse >= 4 && Cse <= 64 && (C >= 160 || (C >= 32 && (long long)N * C >= 4096));
}

hipError_t launch_se_bwd(const SeBwdArgs &a, hipStream_t st)
{
    if (se_bwd_tiled(a.N, a.C, a.Cse)) {
        hipLaunchKernelGGL(se_bwd_dq_kernel, dim3(a.N, (a.Cse + 15) / 16), dim3(256), 0, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        const int chan = (a.C + 15) / 16, fc = (chan * ((a.Cse + 15) / 16) + 3) / 4;
        hipLaunchKernelGGL(se_bwd_sums_kernel, dim3(chan + fc + 1), dim3(256), 0, st, a, chan, fc);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(se_bwd_image_kernel, dim3(a.N), dim3(256), sizeof(float) * (a.C + a.Cse), st,
                       a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    const int total = 2 * a.C * a.Cse + a.C + a.Cse;
    hipLaunchKernelGGL(se_bwd_batch_kernel, dim3((total + 7) / 8), dim3(256), 0, st, a);
    return hipGetLastError();
}

// out[c*inner+i] = sum_n in[(c*N+n)*inner+i].  Eight lanes share an output: lane s adds
// the images s, s+8, ... and the eight partial sums are combined by a fixed butterfly.
__device__ __forceinline__ void reduce_planes_body(int block, const float *__restrict__ in, int C,
                                                   int N, int inner, float *__restrict__ out)
{
    const int gid = block * 256 + threadIdx.x;
    const int i = gid >> 3, sub = gid & 7;
    float s = 0.f;
    if (i < C * inner) {
        const int c = i / inner, t = i - c * inner;
        const float *src = in + (size_t)c * N * inner + t;
        float s0 = 0.f, s1 = 0.f;
        int n = sub;
        for (; n + 8 < N; n += 16) {
            s0 += src[(size_t)n * inner];
            s1 += src[(size_t)(n + 8) * inner];
        }
        if (n < N)
            s0 += src[(size_t)n * inner];
        s = s0 + s1;
    }
    s += __shfl_xor(s, 4, kWave);
    s += __shfl_xor(s, 2, kWave);
    s += __shfl_xor(s, 1, kWave);
    if (sub == 0 && i < C * inner)
        out[i] = s;
}

__global__ __launch_bounds__(256) void reduce_planes_kernel(const float *__restrict__ in, int C,
                                                            int N, int inner,
                                                            float *__restrict__ out)
{
    reduce_planes_body(blockIdx.x, in, C, N, inner, out);
}

// The two second stages that follow the fused depthwise backward, in one launch: the first nb1
// workgroups add the filter-gradient partials, the others finalise BN1's backward.
__global__ __launch_bounds__(256) void dw_bwd_finalize_kernel(int nb1, const float *__restrict__ pdw,
                                                              int C, int NP, int inner,
                                                              float *__restrict__ dw, double inv_m,
                                                              const float *__restrict__ psb,
                                                              const float *__restrict__ psr,
                                                              const float *__restrict__ gamma,
                                                              const float *__restrict__ bn,
                                                              float *dgamma, float *dbeta,
                                                              float *coef)
{
    if ((int)blockIdx.x < nb1)
        reduce_planes_body(blockIdx.x, pdw, C, NP, inner, dw);
    else
        bn_bwd_finalize_body(blockIdx.x - nb1, C, NP, inv_m, psb, psr, gamma, bn, dgamma, dbeta, coef);
}

hipError_t launch_dw_bwd_finalize(const float *pdw, int C, int NP, int inner, float *dw, double m,
                                  const float *psb, const float *psr, const float *gamma,
                                  const float *bn, float *dgamma, float *dbeta, float *coef,
                                  hipStream_t st)
{
    const long long total = (long long)C * inner * 8;
    const int nb1 = (int)((total + 255) / 256), nb2 = (C + 3) / 4;
    hipLaunchKernelGGL(dw_bwd_finalize_kernel, dim3((unsigned)(nb1 + nb2)), dim3(256), 0, st, nb1, pdw,
                       C, NP, inner, dw, 1.0 / m, psb, psr, gamma, bn, dgamma, dbeta, coef);
    return hipGetLastError();
}

hipError_t launch_reduce_planes(const float *in, int C, int N, int inner, float *out,
                                hipStream_t st)
{
    const long long total = (long long)C * inner * 8;
    hipLaunchKernelGGL(reduce_planes_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                       in, C, N, inner, out);
    return hipGetLastError();
}

} // namespace mbk
