// 1x1 convolutions of the wide blocks with a long contraction (the projection conv, the data
// gradients, and what conv_xw does not take) on the bf16 matrix cores, without a barrier or an LDS
// store in the contraction.
//
//   out[n][m][q] = sum_k W[m][k] * op(B)[n][k][q]
//
// A workgroup owns 32 pixels and a slab of 16*RT output rows; its wavefronts split the CONTRACTION:
// wavefront w takes the 32-deep steps w, w + W, ... of it for the whole output tile and the partial
// tiles meet once, in LDS, in wavefront order.  What bounds these launches is the prologue and the
// operand split (about 20 vector instructions per activation element) on the one hand and the length
// of a workgroup's dependent chain on the other.  A kernel of 64 x 64 tiles with two barriers per 32
// values of k repeats the first for every 64 rows and serialises stage, barrier, multiply, barrier
// (measured, fp32, batch 64: 1152 -> 192 channels on 7x7 30 us and another 5 for the sum over its
// splits, its gradient 31, 80 <- 480 on 14x14 26, 112 <- 672 33); here
//   - an activation element is loaded, sent through its prologue and split once per slab of up to 128
//     rows: lane (r, g) = (lane % 16, lane / 16) loads the values k = 8g .. 8g+7 of a step for its two
//     pixels (2r and 2r+1 of the chunk when the plane size is even: eight-byte loads; r and 16+r
//     otherwise), and these registers ARE the B operands of v_mfma_f32_16x16x32_bf16;
//   - the weights come from the weight image in lane order straight into registers, 16 bytes per lane
//     and plane, requested ahead of the prologue they overlap with;
//   - the steps of a contraction run on W wavefronts at once, so a launch of few pixels (one image, the
//     7x7 stages) still has a short chain, with no second launch for the partial sums.
// The same shapes: 19, 23, 15 and 22 us.  Half of that is fixed (launch, first loads, adding up and
// storing the tile: 10 us with one step per wavefront), the rest the vector instructions of the
// prologue and the weights' way from L2 in about equal parts; issuing the prologue of the next step
// between the MFMAs, or loading two steps ahead, measured no faster, and sharing the prepared operand
// of all wavefronts through LDS (each then owning rows instead of steps) slower: 26 us for 112 <- 672,
// where eight wavefronts read every operand from LDS.
// Prologue coefficients wait in LDS, {c0, c1} or {c0, c1, c2} per k and the gate per image and k.
//
// Storage fp32: three bf16 planes per operand, six MFMAs per product block (kernels_x3.hip).  Storage
// bf16 (aligned shapes): the weights as they are, the activations rounded to bf16 once after their
// fp32 prologue, one MFMA, fp32 accumulation, as in kernels_bf.hip.
#include <algorithm>
#include <type_traits>
#include "mbconv_x3.h"

namespace mbk {

struct XkArgs {
    int M, K, HW;
    uint32_t Q;
    int numChunks;    // chunks of 32 pixels
    int chunksPerDie; // consecutive chunks whose workgroups share a die (and its L2)
    FastDiv divHW;
    const uint16_t *img; // weight image in lane order
    int CH;              // its 32-deep steps
    int lastTile;        // its last 16-row tile
    const void *w;       // the weights themselves, A(m, k) = w[m*sm + k*sk] (xk_plain only)
    int sm, sk;
    const void *p0, *p1;
    const float *c0, *c1, *c2, *gate;
    void *out;
    const void *res;
    float *psum, *psq; // EPI_STATS: [M][numChunks]; EPI_AFFINE: the rows' scale and shift (read)
    int slabs, W, epi;
};

constexpr int kXkPitch = 36; // floats per row of a partial tile in LDS (32 pixels + 4)

// the two pixels of a lane, one contraction row
template <typename T, bool PAIR>
struct XkRaw {
    float v[2];
    __device__ __forceinline__ void load(const T *p, uint32_t o0, uint32_t o1)
    {
        if (PAIR) {
            const f32x2 t = *reinterpret_cast<const f32x2 *>(p + o0);
            v[0] = t[0];
            v[1] = t[1];
        } else {
            v[0] = p[o0];
            v[1] = p[o1];
        }
    }
    __device__ __forceinline__ float get(int i) const { return v[i]; }
};
template <>
struct XkRaw<bf16_t, true> { // (bf16 is served on planes that are multiples of four)
    uint32_t v;
    __device__ __forceinline__ void load(const bf16_t *p, uint32_t o0, uint32_t)
    {
        v = *reinterpret_cast<const uint32_t *>(p + o0);
    }
    __device__ __forceinline__ float get(int i) const
    {
        return __uint_as_float(i ? v & 0xffff0000u : v << 16);
    }
};

__device__ __forceinline__ void xk_operand(const float (&v)[8], bf16x8 (&o)[3])
{
    uint32_t p[4][3];
    x3_split8(v, p, o);
}
__device__ __forceinline__ void xk_operand(const float (&v)[8], bf16x8 (&o)[1])
{
    u32x4 q;
#pragma unroll
    for (int t = 0; t < 4; ++t)
        q[t] = bf16_pack2(v[2 * t], v[2 * t + 1]);
    o[0] = __builtin_bit_cast(bf16x8, q);
}

// acc0 += a*b0, acc1 += a*b1: the two pixel tiles take turns, so that consecutive MFMAs do not
// depend on each other.  fp32: the products of the upper planes and the five small ones have
// accumulators of their own, added once at the end.  The instruction cuts what it adds off below the
// largest addend's last bits, towards minus infinity, so small terms added to a large accumulator come
// out too small by 1.4e-8 of the result on average, a bias that the sums over whole planes behind these
// convolutions (batch statistics, BN's and the gate's gradients) collect: measured over 256-deep random
// products, mean error -1.4e-8 and rms 2.3e-7 of the result in one accumulator, -1e-10 and 9e-8 in two;
// fp32 MFMA 1e-10 and 2.9e-7.
__device__ __forceinline__ void xk_mma(const bf16x8 (&a)[3], const bf16x8 (&b0)[3], const bf16x8 (&b1)[3],
                                       f32x4 (&acc0)[2], f32x4 (&acc1)[2])
{
#define MBK_MMA(i, j, t)                                                                          \
    acc0[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b0[j], acc0[t], 0, 0, 0);             \
    acc1[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b1[j], acc1[t], 0, 0, 0);
    MBK_MMA(2, 0, 1)
    MBK_MMA(0, 2, 1)
    MBK_MMA(1, 1, 1)
    MBK_MMA(1, 0, 1)
    MBK_MMA(0, 1, 1)
    MBK_MMA(0, 0, 0)
#undef MBK_MMA
}
__device__ __forceinline__ void xk_mma(const bf16x8 (&a)[1], const bf16x8 (&b0)[1], const bf16x8 (&b1)[1],
                                       f32x4 (&acc0)[1], f32x4 (&acc1)[1])
{
    acc0[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b0[0], acc0[0], 0, 0, 0);
    acc1[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b1[0], acc1[0], 0, 0, 0);
}

// sum over eight consecutive lanes (DPP: quads, then the mirrored half row)
__device__ __forceinline__ float sum8(float v)
{
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xb1, 0xf, 0xf, false));  // quad_perm 1,0,3,2
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4e, 0xf, 0xf, false));  // quad_perm 2,3,0,1
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xf, 0xf, false)); // row_half_mirror
    return v;
}

// One output as a plain fp32 sum.  An operand that is infinite, or rounds to an infinite bf16, has NaN
// in its lower planes (x - inf), and so has a finite weight's zero padding times an infinite last row:
// what should be an infinity, or finite behind ReLU6, would come out as NaN.  The epilogue calls this for
// the outputs that are NaN; a NaN operand gives it the same NaN at once.  (The check costs nothing that
// can be measured: 4667 and 4671 us for a training step of the benchmark's 16 blocks.)
template <typename T, int PRO>
__device__ __forceinline__ float xk_plain(const XkArgs &a, int m, uint32_t n, uint32_t pix)
{
    float s = 0.f;
#pragma unroll 1
    for (int k = 0; k < a.K && s == s; ++k) {
        const size_t row = (size_t)n * a.K + k, i = row * a.HW + pix;
        const float v0 = ld<T>((const T *)a.p0, i);
        float b = v0;
        if (PRO == PRO_BNBWD)
            b = x3_apply<PRO>(v0, ld<T>((const T *)a.p1, i), a.c0[k], a.c1[k], a.c2[k]);
        else if (PRO == PRO_BNSWISH_GATE)
            b = x3_apply<PRO>(v0, 0.f, a.c0[k], a.c1[k], a.gate[row]);
        s = fmaf(ld<T>((const T *)a.w, (size_t)m * a.sm + (size_t)k * a.sk), as_stored<T>(b), s);
    }
    return s;
}

// RT: row tiles of the workgroup's slab; PAIR: the plane size is even
template <typename T, int RT, bool PAIR, int PRO>
__global__ __launch_bounds__(512, 2) void conv_xk_kernel(XkArgs a)
{
    constexpr int NP = PRO == PRO_BNBWD ? 2 : 1;
    constexpr int NPL = sizeof(T) == 4 ? 3 : 1; // bf16 planes per operand
    constexpr int TILE = 16 * RT * kXkPitch; // floats of a partial tile
    extern __shared__ __attribute__((aligned(16))) float ldsf[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int M = a.M, K = a.K, HW = a.HW, W = a.W;
    // die = workgroup mod 8: all slabs of a run of consecutive chunks on one die, so that the cache
    // lines neighbouring chunks share, and the operand the slabs share, come out of one L2
    const int die = blockIdx.x & 7, bi = blockIdx.x >> 3;
    const int slab = bi % a.slabs, chunk = die * a.chunksPerDie + bi / a.slabs;
    if (chunk >= a.numChunks) // uniform over the workgroup
        return;
    const T *p0 = (const T *)a.p0, *p1 = (const T *)a.p1;

    // the lane's two pixels (past the end: pixel 0 of the chunk; such columns are never stored)
    const uint32_t q0 = (uint32_t)chunk * 32u;
    uint32_t bo[2], im[2];
    const uint32_t n0 = fdiv(q0, a.divHW);
#pragma unroll
    for (int pt = 0; pt < (PAIR ? 1 : 2); ++pt) {
        const uint32_t q = q0 + (PAIR ? 2u * (uint32_t)r : 16u * pt + (uint32_t)r);
        const uint32_t qs = q < a.Q ? q : q0;
        const uint32_t n = fdiv(qs, a.divHW);
        bo[pt] = n * (uint32_t)K * (uint32_t)HW + (qs - n * (uint32_t)HW);
        im[pt] = n - n0;
    }
    if (PAIR) {
        bo[1] = bo[0];
        im[1] = im[0];
    }
    const uint32_t lastRow = (uint32_t)(K - 1) * (uint32_t)HW;
    XkRaw<T, PAIR> raw[NP][8];
    // contraction rows 32s + 8g .. +7, those past the end read the last one (its weights are zero)
    const auto fetch = [&](int s) __attribute__((always_inline)) {
        const uint32_t row = (uint32_t)(32 * s + 8 * g) * (uint32_t)HW;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const uint32_t o = min(row + (uint32_t)t * (uint32_t)HW, lastRow);
            raw[0][t].load(p0, bo[0] + o, bo[1] + o);
            if (NP == 2)
                raw[NP - 1][t].load(p1, bo[0] + o, bo[1] + o);
        }
    };
    const int steps = a.CH;
    if (wv < steps)
        fetch(wv);

    // prologue coefficients: BN backward {c0, c1, c2, -}[k]; BN + activation {c0, c1}[k] and the gate
    // of every image the chunk touches, [image][k]; zero past K
    const int KP = 32 * a.CH;
    f32x4 *Cb = reinterpret_cast<f32x4 *>(ldsf);
    f32x2 *Cs = reinterpret_cast<f32x2 *>(ldsf);
    float *Gt = ldsf + 2 * KP;
    // (all loads of a thread's share requested before the first is used: a loop of load and store pays a
    // memory round trip per iteration, 1152 -> 320 channels on 7x7 27.7 us, now 26.2; 672 -> 112 on 14x14 20.7,
    // now 20.1.  Where a thread has one entry at most, none is requested for the others: 300 -> 56 channels on two 12x12
    // planes, the block's evaluation 17.1 us with five, 16.8 with one)
    const int nthr = 64 * W;
    const auto coefficients = [&](auto cu) __attribute__((always_inline)) {
        constexpr int CU = decltype(cu)::value;
        if constexpr (PRO == PRO_BNBWD) {
            for (int kb = tid; kb < KP; kb += CU * nthr) {
                float v0[CU], v1[CU], v2[CU];
#pragma unroll
                for (int u = 0; u < CU; ++u) {
                    const int kk = min(kb + u * nthr, K - 1);
                    v0[u] = a.c0[kk];
                    v1[u] = a.c1[kk];
                    v2[u] = a.c2[kk];
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < CU; ++u) {
                    const int k = kb + u * nthr;
                    const uint32_t m = k < K ? 0xffffffffu : 0u;
                    if (k < KP)
                        Cb[k] = (f32x4){and_mask(v0[u], m), and_mask(v1[u], m), and_mask(v2[u], m), 0.f};
                }
            }
        } else if constexpr (PRO == PRO_BNSWISH_GATE) {
            const uint32_t nl = fdiv(min(q0 + 31u, a.Q - 1u), a.divHW) - n0;
            const float *gt0 = a.gate + (size_t)n0 * K, *gt1 = a.gate + (size_t)(n0 + min(nl, 1u)) * K;
            for (int kb = tid; kb < KP; kb += CU * nthr) {
                float v0[CU], v1[CU], g0[CU], g1[CU];
#pragma unroll
                for (int u = 0; u < CU; ++u) {
                    const int kk = min(kb + u * nthr, K - 1);
                    v0[u] = a.c0[kk];
                    v1[u] = a.c1[kk];
                    g0[u] = gt0[kk];
                    g1[u] = gt1[kk];
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < CU; ++u) {
                    const int k = kb + u * nthr;
                    const uint32_t m = k < K ? 0xffffffffu : 0u;
                    if (k < KP) {
                        Cs[k] = (f32x2){and_mask(v0[u], m), and_mask(v1[u], m)};
                        Gt[k] = and_mask(g0[u], m);
                        if (nl)
                            Gt[KP + k] = and_mask(g1[u], m);
                    }
                }
            }
            for (uint32_t i = 2; i <= nl; ++i) // (planes of less than 31 pixels)
                for (int k = tid; k < KP; k += nthr)
                    Gt[i * KP + k] = and_mask(a.gate[(size_t)(n0 + i) * K + min(k, K - 1)], k < K ? 0xffffffffu : 0u);
        }
    };
    if (KP <= nthr) // uniform
        coefficients(std::integral_constant<int, 1>());
    else
        coefficients(std::integral_constant<int, 5>());
    if (PRO != PRO_NONE)
        __syncthreads();

    constexpr int NT = NPL == 3 ? 2 : 1; // accumulators per output (xk_mma)
    f32x4 acc[RT][2][NT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t)
            acc[i][0][t] = acc[i][1][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const uint16_t *wtile[RT]; // the slab's row tiles (those past the image read its last one)
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        const int rt = min(slab * RT + i, a.lastTile);
        wtile[i] = a.img + ((size_t)(rt >> 2) * a.CH * 4 + (rt & 3)) * (NPL * 512);
    }
    // a step's weights are requested as soon as the previous step's have been multiplied
    // (a ring of NA row tiles where all of them would not fit into the registers; RP: its positions per
    // step, of which those past RT are empty)
    constexpr int NA = NPL == 3 && RT >= 7 ? 4 : NPL == 3 && RT == 6 ? 3 : RT, RP = (RT + NA - 1) / NA * NA;
    bf16x8 av[NA][NPL];
    const auto fetch_w = [&](int i, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int pl = 0; pl < NPL; ++pl)
            av[i % NA][pl] = *reinterpret_cast<const bf16x8 *>(wtile[i] + (size_t)s * (4 * NPL * 512) + pl * 512 + lane * 8);
    };
    // step s's activations, already loaded: through the normalisation (`consume`: the loads' registers
    // are free afterwards), then through activation and gate into MFMA operands
    const auto consume = [&](int s, float (&d0)[8], float (&d1)[8]) __attribute__((always_inline)) {
        const int k0 = 32 * s + 8 * g;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const float x0 = raw[0][t].get(0), x1 = raw[0][t].get(1);
            if (PRO == PRO_BNBWD) {
                const f32x4 k = Cb[k0 + t];
                d0[t] = fmaf(k[0], x0, fmaf(k[1], raw[NP - 1][t].get(0), k[2]));
                d1[t] = fmaf(k[0], x1, fmaf(k[1], raw[NP - 1][t].get(1), k[2]));
            } else if (PRO == PRO_BNSWISH_GATE) {
                const f32x2 k = Cs[k0 + t];
                d0[t] = fmaf(x0, k[0], k[1]);
                d1[t] = fmaf(x1, k[0], k[1]);
            } else {
                d0[t] = x0;
                d1[t] = x1;
            }
        }
    };
    const auto operands = [&](int s, float (&d0)[8], float (&d1)[8], bf16x8 (&b0)[NPL],
                              bf16x8 (&b1)[NPL]) __attribute__((always_inline)) {
        if (PRO == PRO_BNSWISH_GATE) {
            const int k0 = 32 * s + 8 * g;
            const float *ga = Gt + im[0] * KP + k0, *gb = Gt + im[1] * KP + k0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 g0 = *reinterpret_cast<const f32x4 *>(ga + 4 * h);
                const f32x4 g1 = PAIR ? g0 : *reinterpret_cast<const f32x4 *>(gb + 4 * h);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    d0[4 * h + j] = actf(d0[4 * h + j]) * g0[j];
                    d1[4 * h + j] = actf(d1[4 * h + j]) * g1[j];
                }
            }
        }
        xk_operand(d0, b0);
        xk_operand(d1, b1);
    };
    // (Loads in one order in and ahead of the loop, fenced, so that the wait counts stay exact: a
    // step's activations, then its weights, each as soon as the registers are free.)
    if (wv < steps) {
#pragma unroll
        for (int i = 0; i < NA; ++i)
            fetch_w(i, wv);
    }
    for (int s = wv; s < steps; s += W) {
        const int ns = min(s + W, steps - 1); // (the last step again: loads stay unconditional)
        bf16x8 b0[NPL], b1[NPL];
        float d0[8], d1[8];
        consume(s, d0, d1);
        __builtin_amdgcn_sched_barrier(0);
        fetch(ns);
        operands(s, d0, d1, b0, b1);
#pragma unroll
        for (int i = 0; i < RP; ++i) {
            if (i < RT)
                xk_mma(av[i % NA], b0, b1, acc[i][0], acc[i][1]);
            if (i + NA < RT)
                fetch_w(i + NA, s);
            else if (i + NA >= RP)
                fetch_w(i + NA - RP, ns);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // ---- the wavefronts' partial tiles, [row][pixel] ----
    if (NT == 2) {
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            acc[i][0][0] += acc[i][0][NT - 1];
            acc[i][1][0] += acc[i][1][NT - 1];
        }
    }
    const auto park = [&](float *dst) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float *d = dst + (16 * i + 4 * g + v) * kXkPitch;
                if (PAIR) {
                    *reinterpret_cast<f32x2 *>(d + 2 * r) = (f32x2){acc[i][0][0][v], acc[i][1][0][v]};
                } else {
                    d[r] = acc[i][0][0][v];
                    d[16 + r] = acc[i][1][0][v];
                }
            }
    };
    __syncthreads(); // the coefficients have been read: the tiles lie over them
    int tiles = W;
    if (W == 8) { // eight tiles would be too much LDS: the upper four are added into the lower four
        if (wv >= 4)
            park(ldsf + (wv - 4) * TILE);
        __syncthreads();
        if (wv < 4) {
            const float *src = ldsf + wv * TILE;
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float *d = src + (16 * i + 4 * g + v) * kXkPitch;
                    acc[i][0][0][v] += d[PAIR ? 2 * r : r];
                    acc[i][1][0][v] += d[PAIR ? 2 * r + 1 : 16 + r];
                }
        }
        __syncthreads();
        tiles = 4;
    }
    if (wv < tiles)
        park(ldsf + wv * TILE);
    __syncthreads();

    // ---- epilogue: eight lanes to a row, four pixels each ----
    const int c = tid & 7;
    const uint32_t q = q0 + 4u * c;
    const bool v4 = (HW & 3) == 0;
    uint32_t n[4], pix[4];
    {
        const uint32_t qs = min(q, a.Q - 1u);
        n[0] = fdiv(qs, a.divHW);
        pix[0] = qs - n[0] * (uint32_t)HW;
#pragma unroll
        for (int j = 1; j < 4; ++j) {
            const bool wrap = pix[j - 1] + 1u == (uint32_t)HW;
            n[j] = n[j - 1] + (wrap ? 1u : 0u);
            pix[j] = wrap ? 0u : pix[j - 1] + 1u;
        }
    }
    T *out = (T *)a.out;
    const T *res = (const T *)a.res;
    const bool withRes = (a.epi == EPI_RES || a.epi == EPI_AFFINE) && res != nullptr;
    for (int row = tid >> 3; row < 16 * RT; row += 8 * W) {
        const int m = slab * (16 * RT) + row, mc = min(m, M - 1);
        f32x4 s = *reinterpret_cast<const f32x4 *>(ldsf + row * kXkPitch + 4 * c);
        for (int w = 1; w < tiles; ++w)
            s += *reinterpret_cast<const f32x4 *>(ldsf + w * TILE + row * kXkPitch + 4 * c);
        const float any = (s[0] + s[1]) + (s[2] + s[3]);
        if (any != any && m < M) { // (not unrolled: one copy of the loop inside)
#pragma unroll 1
            for (uint32_t j = 0; j < 4 && q + j < a.Q; ++j) {
                const float had = j == 0 ? s[0] : j == 1 ? s[1] : j == 2 ? s[2] : s[3];
                if (had == had)
                    continue;
                const uint32_t nj = fdiv(q + j, a.divHW);
                const float f = xk_plain<T, PRO>(a, m, nj, q + j - nj * (uint32_t)HW);
                s[0] = j == 0 ? f : s[0];
                s[1] = j == 1 ? f : s[1];
                s[2] = j == 2 ? f : s[2];
                s[3] = j == 3 ? f : s[3];
            }
        }
        if (a.epi == EPI_AFFINE) {
            const float sc = a.psum[mc], sh = a.psq[mc];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                s[j] = fmaf(s[j], sc, sh);
        }
        float t1 = 0.f, t2 = 0.f;
        if (v4) { // four pixels of one image, aligned to four
            const size_t o = ((size_t)n[0] * M + mc) * HW + pix[0];
            if (q < a.Q && m < M) {
                if (withRes) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        s[j] += ld<T>(res, o + j);
                }
                if constexpr (sizeof(T) == 4) {
                    *reinterpret_cast<f32x4 *>((float *)out + o) = s;
                } else {
                    *reinterpret_cast<uint2 *>(out + o) = make_uint2(bf16_pack2(s[0], s[1]), bf16_pack2(s[2], s[3]));
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float sv = as_stored<T>(s[j]);
                    t1 += sv;
                    t2 = fmaf(sv, sv, t2);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (q + j < a.Q && m < M) {
                    const size_t o = ((size_t)n[j] * M + m) * HW + pix[j];
                    float v = s[j];
                    if (withRes)
                        v += ld<T>(res, o);
                    st<T>(out, o, v);
                    const float sv = as_stored<T>(v);
                    t1 += sv;
                    t2 = fmaf(sv, sv, t2);
                }
            }
        }
        if (a.epi == EPI_STATS) {
            t1 = sum8(t1);
            t2 = sum8(t2);
            if (c == 0 && m < M) {
                a.psum[(size_t)m * a.numChunks + chunk] = t1;
                a.psq[(size_t)m * a.numChunks + chunk] = t2;
            }
        }
    }
}

struct XkPlan {
    int chunks, slabs, rt, W;
    size_t lds;
};

// Shapes and split.  bf16 storage: the shapes whose convolutions take bf16 operands (as
// bf_conv_plan), in the roles with fewer rows than contraction indices, up to a size (below); 112 -> 672
// stays with conv_bf, 31 us either way, and so does the expansion conv, whose operand has no prologue.
static bool xk_plan(bool bf16, int N, int M, int K, int HW, int pro, XkPlan *p)
{
    const long long Q = (long long)N * HW;
    if (K < 32 || M < 8)
        return false;
    if (bf16 && (pro == PRO_NONE || M > K || K % 8 != 0 || M % 8 != 0 || HW % 4 != 0))
        return false;
    if (Q * K >= (1ll << 32) || Q * M >= (1ll << 32)) // 32-bit element offsets in the kernel
        return false;
    const int tiles = (M + 15) / 16, ch = (K + 31) / 32;
    p->chunks = (int)((Q + 31) / 32);
    // Row tiles per slab, up to eight: rounds of workgroups over 256 compute units times a workgroup's
    // time (a prologue worth about four row tiles, then the tiles), plus the re-reading of the operand
    // by every slab where it is large.  Measured, fp32, batch 64, 7x7: 1152 -> 192 channels with six
    // tiles per slab 18.4 us, four 24, three 23; 1152 -> 320 with seven 31, five 27, four 34; 14x14,
    // 672 -> 112 with seven 21, four 26; one image of it with seven 11.8, two 7.8.
    p->rt = 0;
    double best = 0.;
    for (int rt = 8; rt >= 2; --rt) {
        const int slabs = (tiles + rt - 1) / rt;
        if (rt > 2 && (tiles + slabs - 1) / slabs < rt)
            continue; // as many slabs as with fewer tiles each
        const double rounds = (double)(((long long)p->chunks * slabs + 255) / 256);
        const double cost = rounds * (4 + rt) + slabs * std::min(3., p->chunks / 32.);
        if (!p->rt || cost < best) {
            best = cost;
            p->rt = rt;
            p->slabs = slabs;
        }
    }
    // Wavefronts that split the contraction: more where a launch leaves the chip empty (a shorter
    // chain), fewer where there are workgroups enough (less to add up).  Same shapes: 1152 -> 192 (196
    // workgroups) with eight 18.4 us, four 20.6, two 31; 672 -> 112 (392) with four 21, two 33, eight
    // 26; 192 -> 1152 (882) with two 21.7, four 24.
    const long long wgs = (long long)p->chunks * p->slabs;
    // (up to three steps, which two wavefronts share unevenly or hardly at all: one, once there are four
    // workgroups per compute unit; 64 <- 96, 28x28, 512 images 86 us with two, 68 with one, 32 images 11.7
    // and 12.9)
    p->W = wgs <= 256 ? 8 : wgs <= 512 ? 4 : ch <= 3 && wgs > 1024 ? 1 : 2;
    while (p->W > ch)
        p->W /= 2;
    // bf16: up to a number of 16 x 32 output tiles, beyond which conv_bf's 64-pixel tiles are the better
    // ones, and not for contractions of one to three steps in the forward role (64 <- 96, 12x12, 512
    // images, evaluation of a block 46.5 us there, 48.5 here).  conv_bf / here, 14x14: projection conv
    // 112 <- 672, 128 images (5488 tiles) 25.8 / 22.8, 256 images 39.8 / 43.2; 320 <- 1152, 64 images (8232)
    // 46.8 / 50.2; data gradient 112 <- 672, 128 images 33.8 / 26.3, 512 images (21952) 107.5 / 113.7,
    // 20x20, 128 images (11200) 57.5 / 62.7.
    if (bf16 && (wgs * p->rt > (pro == PRO_BNSWISH_GATE ? 6400 : 10000) || (pro == PRO_BNSWISH_GATE && ch < 4)))
        return false;
    const int nimg = 31 / HW + 2; // images a chunk can touch
    const size_t coef = pro == PRO_BNBWD ? (size_t)16 * 32 * ch
                        : pro == PRO_BNSWISH_GATE ? (size_t)(2 + nimg) * 4 * 32 * ch
                                                  : 0;
    const size_t tile = (size_t)std::min(p->W, 4) * 16 * p->rt * kXkPitch * sizeof(float);
    p->lds = std::max(coef, tile);
    return p->lds <= 96 * 1024;
}

bool xk_conv_plan(bool bf16, int N, int M, int K, int HW, int pro, int *chunks)
{
    XkPlan p;
    if (!xk_plan(bf16, N, M, K, HW, pro, &p))
        return false;
    *chunks = p.chunks;
    return true;
}

template <typename T>
static hipError_t xk_launch(const XkArgs &a, const XkPlan &p, int pro, hipStream_t st)
{
    const bool pair = a.HW % 2 == 0;
    const dim3 grid((unsigned)(8 * a.chunksPerDie * a.slabs));
// (bf16: the forms that xk_plan lets through)
#define MBK_CASE(RT_, PAIR_, PRO_)                                                                \
    if constexpr (sizeof(T) == 4 || (PAIR_ && PRO_ != PRO_NONE)) {                                \
        if (p.rt == RT_ && pair == PAIR_ && pro == PRO_) {                                        \
            auto kern = conv_xk_kernel<T, RT_, PAIR_, PRO_>;                                      \
            const hipError_t e_ = hipFuncSetAttribute(                                            \
                (const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds);      \
            if (e_ != hipSuccess)                                                                 \
                return e_;                                                                        \
            hipLaunchKernelGGL(kern, grid, dim3((unsigned)(64 * p.W)), p.lds, st, a);             \
            return hipGetLastError();                                                             \
        }                                                                                         \
    }
#define MBK_RT(RT_)                                                                               \
    MBK_CASE(RT_, true, PRO_BNSWISH_GATE)                                                         \
    MBK_CASE(RT_, false, PRO_BNSWISH_GATE)                                                        \
    MBK_CASE(RT_, true, PRO_BNBWD)                                                                \
    MBK_CASE(RT_, false, PRO_BNBWD)                                                               \
    MBK_CASE(RT_, true, PRO_NONE)                                                                 \
    MBK_CASE(RT_, false, PRO_NONE)
    MBK_RT(2)
    MBK_RT(3)
    MBK_RT(4)
    MBK_RT(5)
    MBK_RT(6)
    MBK_RT(7)
    MBK_RT(8)
#undef MBK_RT
#undef MBK_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_xk_conv1x1(bool bf16, int N, int M, int K, int HW, const void *w, int sAm, int sAk,
                             const void *wimg, const Operand &B, void *out, int epi, const void *res, float *psum, float *psq, hipStream_t st)
{
    XkPlan p;
    if (!wimg || !xk_plan(bf16, N, M, K, HW, B.pro, &p))
        return hipErrorInvalidValue;
    XkArgs a;
    a.M = M;
    a.K = K;
    a.HW = HW;
    a.Q = (uint32_t)((long long)N * HW);
    a.numChunks = p.chunks;
    a.chunksPerDie = (p.chunks + 7) / 8;
    a.divHW = make_div((uint32_t)HW);
    a.img = (const uint16_t *)wimg;
    a.CH = (K + 31) / 32;
    a.lastTile = (M + 63) / 64 * 4 - 1;
    a.w = w;
    a.sm = sAm;
    a.sk = sAk;
    a.p0 = B.p0;
    a.p1 = B.p1;
    a.c0 = B.c0;
    a.c1 = B.c1;
    a.c2 = B.c2;
    a.gate = B.gate;
    a.out = out;
    a.res = res;
    a.psum = psum;
    a.psq = psq;
    a.slabs = p.slabs;
    a.W = p.W;
    a.epi = epi;
    return bf16 ? xk_launch<bf16_t>(a, p, B.pro, st) : xk_launch<float>(a, p, B.pro, st);
}

} // namespace mbk
