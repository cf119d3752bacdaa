// Both gradients of a narrow -> wide 1x1 convolution, a wavefront per pixel chunk, with the convolution's
// output computed again instead of read (fp32 storage, at most 16 narrow channels).
//
// The expansion conv's backward: dx = W^T de (+ dout) and dW = de x^T from one pass over
// de = c0*dy1 + c1*e + c2 (BN1's backward on the way in).  e and dy1 are the two widest tensors of the
// block, and what bounds a kernel that reads both is memory: 16 -> 96 channels on 803 k pixels are 719 MB,
// 160 us in this form, 170 with a workgroup per chunk.  But e = W x, and x is here for the weight gradient
// anyway, so a chunk's e costs matrix-core time only (section "Guided Optimization Case Study:
// EfficientNet": recompute instead of load): 411 MB, 99 us.
//   - A wavefront owns chunks of 32 pixels (chunk = W*workgroup + wavefront, stride W*grid); nothing crosses
//     wavefronts inside the loop, so there is no barrier in it.
//   - Lane (r, g) = (lane % 16, lane / 16) holds pixels 2r and 2r+1, eight bytes per load, sixteen lanes to a
//     128-byte line.  Of x it loads channels 4g .. 4g+3, which are the B operand of e on fp32 MFMA; A = W, in LDS.
//     e has to be as good as the fp32 value that the forward pass stored: an error that all pixels share, of a rounded
//     weight or of an accumulator that truncates, meets a mean of x in the weight gradient and does not average out.
//     (On bf16 MFMA, in three planes, from c2 up: relative error of dW against 64 bits, channels of mean 5, 16 -> 96,
//     300 k pixels, 1.3e-5; with the stored e 2.4e-6; as here 6.0e-7.)
//   - The result has the lane's two pixels of channels 4g .. 4g+3, and that is how dy1 is loaded, so
//     de = c0*dy1 + (c1*e + c2) is two fma per element.
//   - Data gradient: these registers, split, are its B operand (the contraction's order is free: W^T lies in
//     LDS to match); its small products in accumulators of their own (re_mma; dx 1.3e-7 in one, now 7.1e-8).
//   - Weight gradient: a contraction over pixels, so de and x go through LDS once, [channel][pixel], the
//     lane's two pixels of a channel as one 32-bit store per plane; large and small products in accumulators of their own
//     (5.1e-7 together, 1.1e-7 now, for centred channels).
//   - dy1 is requested three steps of 32 channels ahead (two from 97 channels on, one from 129: registers), across
//     the end of a chunk.
// The wavefronts' weight-gradient tiles are added in wavefront order at the end, the workgroups' by
// reduce_splits: fixed order, no atomics.
// With 17 to 32 narrow channels the accumulators of two tiles leave no registers to run ahead: 24 -> 144 on
// 100 k pixels 52 us (41 with the gradients on fp32 MFMA), bwd1x1_lt 38; those stay there.
#include <algorithm>
#include "mbconv_x3.h"

namespace mbk {

struct Bwd1x1ReArgs {
    int Cn, Cw, HW, W;
    uint32_t Q;
    int numChunks;
    FastDiv divHW;
    const float *x, *dy;       // [N][Cn][HW], [N][Cw][HW]
    const float *c0, *c1, *c2; // [Cw]: de = c0*dy + c1*(w x) + c2
    const float *w;            // [Cw][Cn]
    float *dx;                 // [N][Cn][HW]
    const float *res;          // optional, added to dx
    float *partial;            // [grid][Cw][Cn]
};

__device__ __forceinline__ void re_lds_fence()
{
    // a wavefront's LDS operations execute in order: only the compiler has to be held
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// the halves of two words that belong to the first / second pixel
__device__ __forceinline__ uint32_t re_lo(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t re_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// acc + low += a*b over three planes, for two B operands taking turns.  The small products apart: an MFMA cuts off what of
// its addend lies below its products' last place, the same way in every pixel.  (In one accumulator, small terms first, the
// mean over pixels of dx's error is 7.5e-9 of dx, 16 -> 96 channels, and 1.1e-8 where a step is summed before it is added;
// on fp32 MFMA 7.7e-9; as here 5e-10.  Sums of dx over the pixels that should vanish, the gradient of a bias behind a
// normalisation, are made of it.)
__device__ __forceinline__ void re_mma(const bf16x8 (&a)[3], const bf16x8 (&b0)[3], const bf16x8 (&b1)[3],
                                       f32x4 &acc0, f32x4 &acc1, f32x4 &low0, f32x4 &low1)
{
#define MBK_MMA(i, j, p, q)                                                                       \
    p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b0[j], p, 0, 0, 0);                         \
    q = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b1[j], q, 0, 0, 0);
    MBK_MMA(2, 0, low0, low1)
    MBK_MMA(0, 2, low0, low1)
    MBK_MMA(1, 1, low0, low1)
    MBK_MMA(1, 0, low0, low1)
    MBK_MMA(0, 1, low0, low1)
    MBK_MMA(0, 0, acc0, acc1)
#undef MBK_MMA
}

constexpr int kReHalf = 40;  // halfwords per row of a plane in LDS: 32 pixels + 8 (16-byte reads of 16
                             // consecutive rows fall on distinct banks)

// LDS of a workgroup: the tables, then a step of de, or x, in planes per wavefront
template <int NT>
struct ReLds {
    static constexpr int KS = (NT + 1) / 2;       // steps of 32 wide channels
    static constexpr int kWave = 3 * 32 * kReHalf * 2;
    static constexpr int kExp = NT * 1024;        // W
    static constexpr int kBack = KS * 3 * 1024;   // W^T in planes
    static constexpr int kCoef = 3 * 32 * KS * 4; // c0, c1, c2
    static constexpr int kTile = 16 * NT * 16 * 4; // a weight-gradient tile
    static constexpr size_t bytes(int W)
    {
        const size_t run = (size_t)kExp + kBack + kCoef + (size_t)W * kWave, end = (size_t)4 * kTile;
        return run > end ? run : end;
    }
};

// NT: 16-channel tiles of the wide side
template <int NT>
__global__ __launch_bounds__(512, 2) void bwd1x1_re_kernel(Bwd1x1ReArgs a)
{
    typedef ReLds<NT> L;
    constexpr int KS = L::KS, DEPTH = NT > 8 ? 1 : NT > 6 ? 2 : KS < 3 ? KS : 3;
    extern __shared__ __attribute__((aligned(16))) char ldsb[];
    const int tid = threadIdx.x, lane = tid & 63, W = a.W;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int Cn = a.Cn, Cw = a.Cw, HW = a.HW;
    f32x4 *const We = reinterpret_cast<f32x4 *>(ldsb);
    uint16_t *const Wt = reinterpret_cast<uint16_t *>(ldsb + L::kExp);
    float *const C0 = reinterpret_cast<float *>(ldsb + L::kExp + L::kBack), *const C1 = C0 + 32 * KS, *const C2 = C1 + 32 * KS;
    uint16_t *const Lh = reinterpret_cast<uint16_t *>(ldsb + L::kExp + L::kBack + L::kCoef + wv * L::kWave);

    // ---- loads: 32-bit element offsets (the host checks the tensors' sizes), uniform bases ----
    const uint32_t vimg = (uint32_t)Cw * (uint32_t)HW, uimg = (uint32_t)Cn * (uint32_t)HW;
    // the lane's two pixels of chunk c: one image, HW being even
    const auto locate = [&](int c, uint32_t &vb, uint32_t &ub, uint32_t &okm) __attribute__((always_inline)) {
        const uint32_t q = (uint32_t)c * 32u + 2u * (uint32_t)r;
        okm = q < a.Q ? 0xffffffffu : 0u;
        const uint32_t qs = q < a.Q ? q : 0u;
        const uint32_t n = fdiv(qs, a.divHW), pix = qs - n * (uint32_t)HW;
        vb = n * vimg + pix;
        ub = n * uimg + pix;
    };
    f32x2 vy[KS][8], xv[4];
    const uint32_t rows4 = (uint32_t)(4 * g) * (uint32_t)HW;
    // rows 16t + 4g .. +3 of tile t; the last tiles' rows are clamped to the last group of four
    // (Cw % 4 == 0; what lies past the end meets zero coefficients)
    const auto fetch_step = [&](int s, uint32_t vb) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int tile = 2 * s + t;
            if (tile >= NT)
                continue;
            // (uniform base, one vector register of offset)
            const uint32_t o = vb + (tile < NT - 2 ? rows4 : (uint32_t)min(16 * tile + 4 * g, Cw - 4) * (uint32_t)HW);
            const float *p = a.dy + (tile < NT - 2 ? (size_t)(16 * tile) * HW : 0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                vy[s][4 * t + i] = *reinterpret_cast<const f32x2 *>(p + (size_t)i * HW + o);
        }
    };
    // channels 4g .. 4g+3 of x, those past the last read it (their weights are zero)
    const auto fetch_x = [&](uint32_t ub) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            xv[j] = *reinterpret_cast<const f32x2 *>(a.x + (ub + __umul24((uint32_t)min(4 * g + j, Cn - 1), (uint32_t)HW)));
    };
    const int cStep = W * (int)gridDim.x;
    int ch = W * (int)blockIdx.x + wv;
    uint32_t vb, ub, okm;
    // (a wavefront without a chunk loads chunk 0 and never uses it)
    locate(ch < a.numChunks ? ch : 0, vb, ub, okm);
    fetch_x(ub);
#pragma unroll
    for (int s = 0; s < DEPTH; ++s)
        fetch_step(s, vb);
    __builtin_amdgcn_sched_barrier(0);

    // ---- tables, in the lane order of the operands (a thread's loads all requested before the first is
    // used: a loop of load and store pays a memory round trip per entry) ----
    const int nthr = 64 * W;
    {
        constexpr int B = 3; // entries: [tile][lane] of four weights, then [step][lane] of eight
        for (int e0 = tid; e0 < (NT + KS) * 64; e0 += B * nthr) {
            float v[B][8];
            const int cf = min(e0, Cw - 1);
            const float k0 = a.c0[cf], k1 = a.c1[cf], k2 = a.c2[cf];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int e = e0 + u * nthr, b = e >> 6, er = e & 15, eg = (e >> 4) & 3;
                // W: row = wide channel 16b + r, contraction = narrow channel 4g + t
                // W^T: row = narrow channel, contraction = wide channels 4g + t and 16 + 4g + t - 4
                const bool fwd = b < NT; // uniform over the wavefront
                const int row = fwd ? 16 * b + er : 32 * (b - NT) + 4 * eg;
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int c = fwd ? row : row + (t < 4 ? t : 12 + t), k = fwd ? 4 * eg + t : er;
                    v[u][t] = and_mask(a.w[min(c, Cw - 1) * Cn + min(k, Cn - 1)], c < Cw && k < Cn ? 0xffffffffu : 0u);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (e0 < 32 * KS) {
                const uint32_t m = e0 < Cw ? 0xffffffffu : 0u;
                C0[e0] = and_mask(k0, m);
                C1[e0] = and_mask(k1, m);
                C2[e0] = and_mask(k2, m);
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int e = e0 + u * nthr, b = e >> 6;
                if (e >= (NT + KS) * 64)
                    break;
                if (b < NT) {
                    We[e] = (f32x4){v[u][0], v[u][1], v[u][2], v[u][3]};
                    continue;
                }
                uint32_t p[4][3];
                bf16x8 o[3];
                x3_split8(v[u], p, o);
                uint16_t *dst = Wt + (size_t)(b - NT) * 3 * 512 + (e & 63) * 8;
#pragma unroll
                for (int pl = 0; pl < 3; ++pl)
                    *reinterpret_cast<bf16x8 *>(dst + pl * 512) = o[pl];
            }
        }
    }
    __syncthreads();

    // (the small products in accumulators of their own: the MFMA truncates a small addend to a large accumulator)
    f32x4 acc[NT], low[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
        acc[i] = low[i] = (f32x4){0.f, 0.f, 0.f, 0.f};

    for (; ch < a.numChunks; ch += cStep) {
        // the next chunk (the last one re-reads itself: loads stay unconditional)
        const int nx = ch + cStep < a.numChunks ? ch + cStep : ch;
        uint32_t nvb, nub, nokm;
        locate(nx, nvb, nub, nokm);

        // x: B operand of e (column = pixel, contraction = channel), and through LDS of the weight gradient
        // (column = narrow channel, contraction = pixel)
        f32x2 xc[4];
        bf16x8 bx[3];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            xc[j] = xv[j];
            uint32_t w[3];
            x3_split2(xv[j][0], xv[j][1], w);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
                *reinterpret_cast<uint32_t *>(Lh + (pl * 32 + 4 * g + j) * kReHalf + 2 * r) = w[pl];
        }
        fetch_x(nub);
        re_lds_fence();
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
            bx[pl] = *reinterpret_cast<const bf16x8 *>(Lh + (pl * 32 + r) * kReHalf + 8 * g);
        re_lds_fence(); // these reads before the first step's stores
        __builtin_amdgcn_sched_barrier(0);

        f32x4 accd0 = {0.f, 0.f, 0.f, 0.f}, accd1 = accd0, lowd0 = accd0, lowd1 = accd0;
        f32x2 rs[4];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            float d[2][8];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int tile = 2 * s + t;
                if (tile >= NT) { // (the contraction's second half of an odd number of tiles)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        d[0][4 * t + i] = d[1][4 * t + i] = 0.f;
                    continue;
                }
                const f32x4 aw = We[64 * tile + lane];
                const f32x4 k0 = *reinterpret_cast<const f32x4 *>(C0 + 16 * tile + 4 * g);
                const f32x4 k1 = *reinterpret_cast<const f32x4 *>(C1 + 16 * tile + 4 * g);
                const f32x4 k2 = *reinterpret_cast<const f32x4 *>(C2 + 16 * tile + 4 * g);
                f32x4 e0 = {0.f, 0.f, 0.f, 0.f}, e1 = e0;
#pragma unroll
                for (int j = 0; j < 4; ++j) { // contraction 4g + j of every g
                    e0 = __builtin_amdgcn_mfma_f32_16x16x4f32(aw[j], xc[j][0], e0, 0, 0, 0);
                    e1 = __builtin_amdgcn_mfma_f32_16x16x4f32(aw[j], xc[j][1], e1, 0, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    d[0][4 * t + i] = and_mask(fmaf(k0[i], vy[s][4 * t + i][0], fmaf(k1[i], e0[i], k2[i])), okm);
                    d[1][4 * t + i] = and_mask(fmaf(k0[i], vy[s][4 * t + i][1], fmaf(k1[i], e1[i], k2[i])), okm);
                }
            }
            if (s + DEPTH < KS)
                fetch_step(s + DEPTH, vb);
            else
                fetch_step(s + DEPTH - KS, nvb);
            if (s == KS - 1 && a.res) { // (uniform)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    rs[v] = *reinterpret_cast<const f32x2 *>(
                        a.res + (ub + __umul24((uint32_t)min(4 * g + v, Cn - 1), (uint32_t)HW)));
            }
            {
                uint32_t w[8][3];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    x3_split2(d[0][q], d[1][q], w[q]);
                    if (2 * s + q / 4 < NT) {
#pragma unroll
                        for (int pl = 0; pl < 3; ++pl)
                            *reinterpret_cast<uint32_t *>(Lh + (pl * 32 + 16 * (q >> 2) + 4 * g + (q & 3)) * kReHalf + 2 * r) =
                                w[q][pl];
                    }
                }
                bf16x8 b0[3], b1[3], aw[3];
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) {
                    u32x4 lo, hi;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        lo[t] = re_lo(w[2 * t][pl], w[2 * t + 1][pl]);
                        hi[t] = re_hi(w[2 * t][pl], w[2 * t + 1][pl]);
                    }
                    b0[pl] = __builtin_bit_cast(bf16x8, lo);
                    b1[pl] = __builtin_bit_cast(bf16x8, hi);
                    aw[pl] = *reinterpret_cast<const bf16x8 *>(Wt + (size_t)(s * 3 + pl) * 512 + lane * 8);
                }
                re_mma(aw, b0, b1, accd0, accd1, lowd0, lowd1);
            }
            re_lds_fence();
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int tile = 2 * s + t;
                if (tile >= NT)
                    continue;
                bf16x8 av[3];
#pragma unroll
                for (int pl = 0; pl < 3; ++pl)
                    av[pl] = *reinterpret_cast<const bf16x8 *>(Lh + (pl * 32 + 16 * t + r) * kReHalf + 8 * g);
#define MBK_MMA(i, j) low[tile] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bx[j], low[tile], 0, 0, 0);
                MBK_MMA(2, 0)
                MBK_MMA(0, 2)
                MBK_MMA(1, 1)
                MBK_MMA(1, 0)
                MBK_MMA(0, 1)
#undef MBK_MMA
                acc[tile] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[0], bx[0], acc[tile], 0, 0, 0);
            }
            re_lds_fence(); // these reads before the next step's stores
            __builtin_amdgcn_sched_barrier(0); // (left alone, the scheduler has all steps' operands in flight and spills)
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 4 * g + v;
            f32x2 o = {accd0[v] + lowd0[v], accd1[v] + lowd1[v]};
            if (a.res)
                o += rs[v];
            if (okm && row < Cn)
                *reinterpret_cast<f32x2 *>(a.dx + (ub + __umul24((uint32_t)row, (uint32_t)HW))) = o;
        }
        vb = nvb;
        ub = nub;
        okm = nokm;
    }

#pragma unroll
    for (int i = 0; i < NT; ++i)
        acc[i] += low[i];
    // ---- the wavefronts' weight-gradient tiles, in wavefront order: [wide][narrow] ----
    constexpr int TILE = L::kTile / 4;
    float *const Lt = reinterpret_cast<float *>(ldsb);
    __syncthreads();
    if (W == 8) { // the upper four are added into the lower four
        if (wv >= 4) {
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    Lt[(wv - 4) * TILE + (16 * i + 4 * g + v) * 16 + r] = acc[i][v];
        }
        __syncthreads();
        if (wv < 4) {
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    acc[i][v] += Lt[wv * TILE + (16 * i + 4 * g + v) * 16 + r];
        }
        __syncthreads();
    }
    if (wv < 4) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                Lt[wv * TILE + (16 * i + 4 * g + v) * 16 + r] = acc[i][v];
    }
    __syncthreads();
    float *dst = a.partial + (size_t)blockIdx.x * Cw * Cn;
    for (int el = tid; el < TILE; el += nthr) {
        const int c = el >> 4, j = el & 15;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            sum += Lt[w * TILE + el];
        if (c < Cw && j < Cn)
            dst[(size_t)c * Cn + j] = sum;
    }
}

// The shapes of this file: pixel pairs, groups of four wide channels, and enough chunks that the tables pay (both
// steps of the gradients, bwd1x1_lt / here, us: 16 -> 32 channels, 16 chunks 14.4 / 13.7, 392 16.1 / 14.3, 4214 36.9 / 21.9; 16 ->
// 64, 196 chunks 15.4 / 16.2, 392 17.0 / 16.3; 16 -> 96, 392 chunks 18.0 / 18.4, 544 20.6 / 18.6, 12544 102 / 64; 16 -> 144,
// 544 chunks 22.3 / 22.4; the kernels alone, 4232 chunks, 16 -> 144 44.7 / 33.5, 16 -> 192 61.5 / 39.3).
bool bwd1x1_re_supported(int N, int Cw, int Cn, int HW)
{
    const long long Q = (long long)N * HW, chunks = (Q + 31) / 32;
    return Cn <= 16 && Cn < Cw && Cw <= 192 && Cw % 4 == 0 && HW % 2 == 0 && chunks >= (Cw <= 32 ? 1 : Cw <= 64 ? 256 : 512) &&
           Q * Cw < (1ll << 30); // 32-bit byte offsets in the kernel
}

// At most `splits` workgroups; partial: [*used][Cw][Cn].
hipError_t launch_bwd1x1_re(int N, int Cw, int Cn, int HW, const Operand &de, const void *xin, const void *w, void *dx,
                            const void *res, float *partial, int splits, int *used, hipStream_t st)
{
    if (!bwd1x1_re_supported(N, Cw, Cn, HW) || de.pro != PRO_BNBWD || splits < 1)
        return hipErrorInvalidValue;
    Bwd1x1ReArgs a;
    a.Cn = Cn;
    a.Cw = Cw;
    a.HW = HW;
    a.Q = (uint32_t)((long long)N * HW);
    a.numChunks = (int)((a.Q + 31u) / 32u);
    a.divHW = make_div((uint32_t)HW);
    a.x = (const float *)xin;
    a.dy = (const float *)de.p0;
    a.c0 = de.c0;
    a.c1 = de.c1;
    a.c2 = de.c2;
    a.w = (const float *)w;
    a.dx = (float *)dx;
    a.res = (const float *)res;
    a.partial = partial;
    // a workgroup of eight wavefronts per compute unit; four wavefronts where that leaves units empty
    a.W = a.numChunks >= 8 * 256 ? 8 : 4;
    const int grid = std::min(splits, std::min(256 * 8 / a.W, (a.numChunks + a.W - 1) / a.W));
    *used = grid;
    const int nt = (Cw + 15) / 16;
#define MBK_CASE(NT_)                                                                             \
    if (nt <= NT_) {                                                                              \
        auto kern = bwd1x1_re_kernel<NT_>;                                                        \
        const size_t lds = ReLds<NT_>::bytes(a.W);                                                \
        const hipError_t e_ = hipFuncSetAttribute(                                                \
            (const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);            \
        if (e_ != hipSuccess)                                                                     \
            return e_;                                                                            \
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3((unsigned)(64 * a.W)), lds, st, a);   \
        return hipGetLastError();                                                                 \
    }
    MBK_CASE(2)
    MBK_CASE(3)
    MBK_CASE(4)
    MBK_CASE(6)
    MBK_CASE(8)
    MBK_CASE(10)
    MBK_CASE(12)
#undef MBK_CASE
    return hipErrorInvalidValue;
}

} // namespace mbk
