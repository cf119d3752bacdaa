// Evaluation mode, fp32: expansion conv, BN1, activation and depthwise conv in one launch.
//
//   d[n][c] = depthwise(act(BN1(W_e x[n]))),   z[n][c] = mean of act(BN2(d[n][c]))
//
// With fixed statistics BN1 is an affine map per channel, so nothing keeps the expansion conv's output e, the
// largest tensor of the block, from staying on the chip.  A workgroup owns 16 expanded channels (the rows of an
// MFMA tile) and a strip of output rows of one image:
//   - the strip's input pixels, with the rows that the filter reaches beyond it, are one contiguous range of the
//     plane; a wavefront takes 16*PX of them at a time, multiplies on fp32 MFMA (A = weights, in registers for the
//     workgroup's life, B = x straight from memory: lane (r, g) holds PX consecutive pixels of channel 4t + g, and
//     element j feeds MFMA number j), applies BN1 and the activation and leaves them in an LDS tile with a zero border;
//   - after one barrier, 16 or 32 threads to a channel convolve runs of four outputs from the tile, store d, and sum
//     act(BN2(d)) for the squeeze.
// What bounds it: small launches the chain of one workgroup (a request of 112 -> 672 channels on 14x14: 1.9 us until all loads
// are issued, 1.3 weights through LDS, 0.7 operands, 1.1 MFMAs, 0.4 into the tile, 1.3 depthwise), large ones the vector
// work of the two activations and the filter beside the MFMAs, which fp32 MFMAs do not overlap with.  24 -> 144 on 56x56,
// 32 images: 21.8 + 21.9 us in two launches (e written and read, 116 MB), 34 here with ReLU6; with Swish 21.1 + 22.2 and 42.4,
// VALUBusy 50 %.
#include "mbconv_dev.h"
#include "mbconv_launch.h"
#include "mbconv_eval.h"

#include <algorithm>

namespace mbk {

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

namespace {

constexpr int kXdRows = 16;     // expanded channels of a workgroup
constexpr int kXdThreads = 512; // 32 to a channel in the depthwise part

struct XdArgs {
    int N, K, C, H, W, Ho, Wo, k, s, Cse;
    int CG, S, R, rin;   // channel groups, strips per image, output rows of a strip, tile rows
    int NI;              // images side by side in the tile (a power of two; S = 1 where it is not 1)
    int pitch, ims, chs; // tile: floats per row (the plane's column 0 at 4), image and channel
    int items, PL;       // (image group, strip) pairs, and how many of them a workgroup takes one after the other
    int groups;          // ceil(items / PL)
    int perDie;          // 0: workgroups in order; else the channel groups of an item group on one XCD
    int rt;              // output rows to a thread: 1 or 2
    int act;             // store act(BN2(d)) in place of d
    FastDiv divCG, divS, divW, divHW, divRuns, divRuns4;
    const float *x, *w, *wdw, *w1;
    float *d, *z;        // z: [strip][n][c] partial means, or null
    float *q;            // or, instead: [n][channel group, strip][Cse] partial sums of W1 z
};

// One row of the window of four outputs, from the plane's column 4*S*j - P on.
template <int K, int S>
__device__ __forceinline__ void xd_window(const float *p, float (&o)[3 * S + K])
{
    constexpr int P = (K - 1) / 2;
    const f32x4 m = *reinterpret_cast<const f32x4 *>(p);
    if (P == 1) {
        o[0] = p[-1];
    } else {
        const f32x2 l = *reinterpret_cast<const f32x2 *>(p - 2);
        o[0] = l[0];
        o[1] = l[1];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        o[P + e] = m[e];
    if (S == 1) {
        if (P == 1) {
            o[5] = p[4];
        } else {
            const f32x2 r = *reinterpret_cast<const f32x2 *>(p + 4);
            o[6] = r[0];
            o[7] = r[1];
        }
    } else {
        const f32x4 m2 = *reinterpret_cast<const f32x4 *>(p + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            o[P + 4 + e] = m2[e];
        if (P == 2)
            o[10] = p[8];
    }
}

struct XdItem {
    int n, ni, strip, ho0, hin0, p0, p1; // first image, images, ..., pixels p0 .. p1-1 (of all images of the item)
};
template <int KD, int SD>
__device__ __forceinline__ XdItem xd_item(const XdArgs &a, int item)
{
    XdItem t;
    const int ng = (int)fdiv((uint32_t)item, a.divS);
    t.n = ng * a.NI;
    t.ni = min(a.NI, a.N - t.n);
    t.strip = item - ng * a.S;
    t.ho0 = t.strip * a.R;
    t.hin0 = t.ho0 * SD - (KD - 1) / 2;
    t.p0 = max(t.hin0, 0) * a.W;
    t.p1 = min(t.hin0 + a.rin, a.H) * a.W + (t.ni - 1) * a.H * a.W;
    return t;
}

// The depthwise convolution of one item.  Thread -> (channel, image, runs): RT rows by four columns at a time, so that a
// row of the tile is read once for all the outputs of the thread that it reaches.
template <int K, int S, int RT>
__device__ __forceinline__ void xd_depthwise(const XdArgs &a, const XdItem &it, int cg, const float *tile,
                                             const float (&wt)[K * K], float *cf, float inv_hw)
{
    const int tid = threadIdx.x, ch = tid >> 5, tpi = 32 / a.NI;
    const int im = a.NI == 1 ? 0 : (tid & 31) / tpi, lt = tid & (tpi - 1);
    const int c = cg * kXdRows + ch;
    const bool live = c < a.C && im < it.ni;
    const float scale = cf[4 * ch + 2], shift = cf[4 * ch + 3];
    const int rw = (a.Wo + 3) >> 2, rows = min(a.R, a.Ho - it.ho0), runs = (rows + RT - 1) / RT * rw;
    const float *tc = tile + ch * a.chs + im * a.ims + 4;
    float *out = a.d + ((size_t)(it.n + (live ? im : 0)) * a.C + min(c, a.C - 1)) * (a.Ho * a.Wo) + it.ho0 * a.Wo;
    const bool sums = a.z || a.q;
    float zs = 0.f;
    for (int i = lt; i < runs; i += tpi) {
        const int rg = (int)fdiv((uint32_t)i, a.divRuns), j = i - rg * rw, oh = RT * rg;
        const float *p = tc + 4 * S * j;
        float o[RT][4];
#pragma unroll
        for (int q = 0; q < RT; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                o[q][r] = 0.f;
        // (rows past the tile, which only outputs past the strip reach, are its last; two rows at a time: the next is on its
        // way while one is multiplied, and no further ones, which would cost registers)
        constexpr int NR = (RT - 1) * S + K;
        const auto at = [&](int ir) { return p + (RT == 1 ? oh * S + ir : min(oh * S + ir, a.rin - 1)) * a.pitch; };
        const auto taps = [&](int ir, const float (&row)[3 * S + K]) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < RT; ++q) {
                const int u = ir - q * S;
                if (u >= 0 && u < K) {
#pragma unroll
                    for (int v = 0; v < K; ++v)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            o[q][r] = fmaf(wt[u * K + v], row[r * S + v], o[q][r]);
                }
            }
        };
        float row[2][3 * S + K];
        xd_window<K, S>(at(0), row[0]);
#pragma unroll
        for (int ir = 0; ir < NR; ++ir) {
            if (ir + 1 < NR)
                xd_window<K, S>(at(ir + 1), row[(ir + 1) % 2]);
            if (RT > 1)
                __builtin_amdgcn_sched_barrier(0);
            taps(ir, row[ir % 2]);
            if (RT > 1)
                __builtin_amdgcn_sched_barrier(0);
        }
        const int left = a.Wo - 4 * j; // outputs of a run that exist
#pragma unroll
        for (int q = 0; q < RT; ++q) {
            if (RT > 1 && oh + q >= rows)
                break;
            if (a.act) { // (uniform)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    o[q][r] = actf(fmaf(o[q][r], scale, shift));
                    zs += r < left ? o[q][r] : 0.f; // by selection: what lies past the row is unspecified
                }
            }
            float *po = out + (oh + q) * a.Wo + 4 * j;
            if (live) {
                if ((a.Wo & 3) == 0) {
                    *reinterpret_cast<f32x4 *>(po) = (f32x4){o[q][0], o[q][1], o[q][2], o[q][3]};
                } else if ((a.Wo & 1) == 0) {
                    *reinterpret_cast<f32x2 *>(po) = (f32x2){o[q][0], o[q][1]};
                    if (left > 2)
                        *reinterpret_cast<f32x2 *>(po + 2) = (f32x2){o[q][2], o[q][3]};
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r < left)
                            po[r] = o[q][r];
                }
            }
            if (sums && !a.act) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float v = actf(fmaf(o[q][r], scale, shift));
                    zs += r < left ? v : 0.f;
                }
            }
        }
    }
    if (sums) {
        if (tpi >= 16) {
            zs = row16_sum(zs);
            if (tpi == 32)
                zs += __shfl_xor(zs, 16, kWave);
        } else {
            for (int o = tpi >> 1; o > 0; o >>= 1)
                zs += __shfl_xor(zs, o, kWave);
        }
        zs *= inv_hw;
        if (lt == 0 && live) {
            if (a.z)
                a.z[((size_t)it.strip * a.N + it.n + im) * a.C + c] = zs;
        }
        if (a.q && lt == 0) // (channels past the end: zero)
            cf[64 + im * kXdRows + ch] = live ? zs : 0.f;
    }
}

// T: steps of four input channels, 4*TP < K <= 4*T.  PX: pixels to a lane.  KD, SD, RT: xd_depthwise.
template <int T, int TP, int PX, int KD, int SD, int RT>
__global__ __launch_bounds__(kXdThreads, T *(PX + 1) > 40 || (KD == 5 && RT == 2) ? 2 : 4) void xd_kernel(XdArgs a, DwEval ev)
{
    constexpr int threads = kXdThreads, nw = threads / 64;
    constexpr int WP = 4 * T + 4;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ __attribute__((aligned(16))) float cf[4 * kXdRows + 8 * kXdRows]; // {BN1 scale, shift, BN2 scale, shift}
                                                                               // per channel; plane sums
    __shared__ float wd[25 * kXdRows]; // depthwise filters
    __shared__ float w1s[64 * kXdRows];
    float *wl = lds, *tile = lds + kXdRows * WP;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    int cg, ig;
    if (a.perDie) {
        if ((int)blockIdx.x >= ev.main) {
            dw_eval_extra(ev, (int)blockIdx.x - ev.main, threads);
            return;
        }
        const int j = (int)(blockIdx.x >> 3), q = (int)fdiv((uint32_t)j, a.divCG);
        cg = j - q * a.CG;
        ig = 8 * q + (int)(blockIdx.x & 7);
        if (ig >= a.groups)
            return;
    } else {
        cg = (int)blockIdx.x;
        ig = (int)blockIdx.y;
        if (ig >= a.groups) {
            dw_eval_extra(ev, (ig - a.groups) * a.CG + cg, threads);
            return;
        }
    }
    const int c0 = cg * kXdRows, K = a.K, HW = a.H * a.W;
    constexpr int KK = KD * KD;
    const int last = min((ig + 1) * a.PL, a.items);
    int item = ig * a.PL;
    XdItem it = xd_item<KD, SD>(a, item);

    float b[T][PX];
    // the pixels of one chunk, past the range's end those of its start
    const auto fetch = [&](const XdItem &t, int chunk) __attribute__((always_inline)) {
        const int pix = t.p0 + (chunk * 16 + r) * PX;
        uint32_t pc = (uint32_t)(pix < t.p1 ? pix : t.p0);
        if (a.NI > 1) // (uniform)
            pc += fdiv(pc, a.divHW) * (uint32_t)((K - 1) * HW);
        // (byte offsets from one uniform base: a base for every step would not fit the scalar registers)
        const char *px = reinterpret_cast<const char *>(a.x + (size_t)t.n * K * HW);
        const uint32_t step = 16u * (uint32_t)HW, off = 4u * ((uint32_t)(g * HW) + pc);
#pragma unroll
        for (int s = 0; s < T; ++s) {
            const float *q = reinterpret_cast<const float *>(
                px + (s < TP ? off + (uint32_t)s * step : 4u * ((uint32_t)(min(4 * s + g, K - 1) * HW) + pc)));
            if (PX == 4) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(q);
#pragma unroll
                for (int e = 0; e < PX; ++e)
                    b[s][e] = v[e];
            } else if (PX == 2) {
                const f32x2 v = *reinterpret_cast<const f32x2 *>(q);
#pragma unroll
                for (int e = 0; e < PX; ++e)
                    b[s][e] = v[e];
            } else {
                b[s][0] = q[0];
            }
        }
    };
    // ---- everything that the workgroup needs from memory is requested here ----
    // weights: 16 rows of K, padded with zeros to 4T; row r, channel 4t + g to [r][g][t]
    constexpr int WN = (64 * T + threads - 1) / threads;
    float wv[WN];
#pragma unroll
    for (int i = 0; i < WN; ++i) {
        const uint32_t idx = (uint32_t)(tid + i * threads), m = idx / (4 * T), kk = idx % (4 * T);
        wv[i] = a.w[(size_t)min(c0 + (int)m, a.C - 1) * K + min((int)kk, K - 1)];
    }
    const float fv = a.wdw[min(c0 * KK + tid, a.C * KK - 1)];
    // the squeezed layer's weights for these channels, [j][channel]
    float w1v[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        w1v[i] = a.q ? a.w1[(size_t)min((tid + i * threads) >> 4, a.Cse - 1) * a.C + min(c0 + (tid & 15), a.C - 1)] : 0.f;
    BnEvalRegs r1 = {}, r2 = {};
    if (tid < kXdRows) {
        const int c = min(c0 + tid, a.C - 1);
        r1 = bn_eval_issue(ev.bn1, c);
        r2 = bn_eval_issue(ev.bn2, c);
    }
    fetch(it, wave);
    __builtin_amdgcn_sched_barrier(0);
    // the tile's rows outside the plane
    const auto border = [&](const XdItem &t) __attribute__((always_inline)) {
        const int top = max(0, -t.hin0), rows = top + max(0, t.hin0 + a.rin - a.H);
        for (int i = wave; i < kXdRows * rows; i += nw) {
            const int rr = i >> 4, row = rr < top ? rr : a.rin - rows + rr;
            float *p = tile + (i & 15) * a.chs + row * a.pitch;
            if (4 * lane < a.pitch)
                for (int im = 0; im < a.NI; ++im)
                    *reinterpret_cast<f32x4 *>(p + im * a.ims + 4 * lane) = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
    };
    border(it);
    // ---- the tile's zero columns, once ----
    for (int row = tid; row < kXdRows * a.NI * a.rin; row += threads) {
        const int rr = row >> 4;
        float *p = tile + (row & 15) * a.chs + rr * a.pitch;
        *reinterpret_cast<f32x4 *>(p) = (f32x4){0.f, 0.f, 0.f, 0.f};
        for (int c = 4 + a.W; c < a.pitch; ++c)
            p[c] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < WN; ++i) {
        const uint32_t idx = (uint32_t)(tid + i * threads), m = idx / (4 * T), kk = idx % (4 * T);
        if (idx < 64 * T)
            wl[m * WP + (kk & 3) * T + (kk >> 2)] = (int)kk < K ? wv[i] : 0.f;
    }
    if (tid < kXdRows * KK)
        wd[tid] = fv;
#pragma unroll
    for (int i = 0; i < 2; ++i)
        w1s[tid + i * threads] = c0 + (tid & 15) < a.C ? w1v[i] : 0.f;
    if (tid < kXdRows) {
        const BnEvalCoef k1 = bn_eval_coef(r1, ev.eps), k2 = bn_eval_coef(r2, ev.eps);
        *reinterpret_cast<f32x4 *>(cf + 4 * tid) = (f32x4){k1.scale, k1.shift, k2.scale, k2.shift};
    }
    __syncthreads();
    float av[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
        av[t] = wl[r * WP + g * T + t];
    float wt[KK];
#pragma unroll
    for (int t = 0; t < KK; ++t)
        wt[t] = wd[(tid >> 5) * KK + t];
    float sc[4], sh[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        sc[v] = cf[4 * (4 * g + v)];
        sh[v] = cf[4 * (4 * g + v) + 1];
    }
    for (;;) {
        const int chunks = (it.p1 - it.p0 + 16 * PX - 1) / (16 * PX);
        for (int ck = wave; ck < chunks; ck += nw) {
            // (long contractions a chain of four steps at a time: in one chain every step rounds the whole sum; the fence keeps
            // the sums from being put off, which takes registers)
            constexpr int CH = T > 6 ? 4 : T;
            f32x4 acc[PX], sum[PX];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                // (past the contraction both operands are zero: what was loaded there may be infinite)
                const uint32_t ok = t < TP || 4 * t + g < K ? 0xffffffffu : 0u;
#pragma unroll
                for (int e = 0; e < PX; ++e) {
                    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                    acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[t], t < TP ? b[t][e] : and_mask(b[t][e], ok),
                                                                  t % CH ? acc[e] : zero, 0, 0, 0);
                    if (t % CH == CH - 1 || t == T - 1)
                        sum[e] = t < CH ? acc[e] : sum[e] + acc[e];
                }
                if (t % CH == CH - 1)
                    __builtin_amdgcn_sched_barrier(0);
            }
            int pix = it.p0 + (ck * 16 + r) * PX;
            const bool in = pix < it.p1;
            if (ck + nw < chunks)
                fetch(it, ck + nw);
            float *p = tile + 4 * g * a.chs + 4;
            if (a.NI > 1) { // (uniform)
                const int im = (int)fdiv((uint32_t)pix, a.divHW);
                pix -= im * HW;
                p += im * a.ims;
            }
            const int h = (int)fdiv((uint32_t)pix, a.divW), w = pix - h * a.W;
            p += (h - it.hin0) * a.pitch + w;
            if (in) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float y[PX];
#pragma unroll
                    for (int e = 0; e < PX; ++e)
                        y[e] = actf(fmaf(sum[e][v], sc[v], sh[v]));
                    if (PX == 4)
                        *reinterpret_cast<f32x4 *>(p + v * a.chs) = (f32x4){y[0], y[PX / 4], y[PX / 2], y[PX - 1]};
                    else if (PX == 2)
                        *reinterpret_cast<f32x2 *>(p + v * a.chs) = (f32x2){y[0], y[PX - 1]};
                    else
                        p[v * a.chs] = y[0];
                }
            }
        }
        const XdItem cur = it;
        ++item;
        __syncthreads();
        xd_depthwise<KD, SD, RT>(a, cur, cg, tile, wt, cf, ev.inv_hw);
        if (a.q) { // (one item to a workgroup; at most 64 squeezed channels and eight images)
            __syncthreads();
            const int qj = tid & 63, qi = tid >> 6;
            if (qj < a.Cse && qi < cur.ni) {
                float s = 0.f;
#pragma unroll
                for (int e = 0; e < kXdRows; ++e)
                    s = fmaf(w1s[qj * kXdRows + e], cf[64 + qi * kXdRows + e], s);
                a.q[((size_t)(cur.n + qi) * (a.CG * a.S) + cg * a.S + cur.strip) * a.Cse + qj] = s;
            }
        }
        if (item >= last)
            return;
        it = xd_item<KD, SD>(a, item);
        fetch(it, wave);
        __syncthreads();
        border(it);
    }
}

constexpr int kXdSteps[] = {4, 6, 10, 16, 20, 28, 48};

// Steps of the contraction (rounded up to one that is built), pixels to a lane
bool xd_form(int K, int W, int *T, int *PX)
{
    for (const int t : kXdSteps)
        if (K <= 4 * t) {
            *T = t;
            *PX = W % 4 == 0 && t <= 16 ? 4 : W % 2 == 0 && t <= 28 ? 2 : 1;
            return true;
        }
    return false;
}

size_t xd_geometry(const DwShape &s, int T, int S, int NI, XdArgs &a)
{
    a.S = S;
    a.NI = NI;
    a.R = (s.Ho + S - 1) / S;
    a.rin = (a.R - 1) * s.s + s.k;
    a.pitch = (s.s == 1 ? 4 : 8) * ((s.Wo + 3) / 4) + 8;
    a.ims = a.rin * a.pitch;
    a.chs = NI * a.ims;
    if (a.chs % 8 == 0) // channels four apart on the two halves of the banks
        a.chs += 4;
    return sizeof(float) * (size_t)kXdRows * (a.chs + 4 * T + 4);
}

} // namespace

// Strips of an image, and the rest of the plan; false: not a shape of this kernel.
static bool xd_plan(const DwShape &s, int K, XdArgs &a, int *T, int *PX, size_t *lds)
{
    // (long contractions as conv_xs takes them: its rows are what this kernel replaces; odd channel counts are with kernels
    // on the bf16 matrix cores, whose sums are the more exact ones)
    if (!xd_form(K, s.W, T, PX) || (*T > 6 && K % 8 != 0))
        return false;
    if ((long long)s.N * s.Ho * ((s.C + 15) / 16) >= (1ll << 30))
        return false;
    // what the depthwise kernels refuse stays refused (kernels_dw2.hip)
    if (s.s == 2 && s.W % 4 == 2 && s.H % 2 == 0 && s.H * ((s.W + 3) / 4) > 1024)
        return false;
    a.CG = (s.C + kXdRows - 1) / kXdRows;
    int S = 1, NI = 1;
    while (S < s.Ho && xd_geometry(s, *T, S, 1, a) > 52 * 1024)
        ++S;
    const int rows = S * std::min(a.rin, s.H); // (rows of e computed, those that strips share more than once)
    while (S < s.Ho && (long long)s.N * a.CG * S < 128 && (s.Ho + S - 1) / S * s.Wo > 128)
        ++S;
    S = (s.Ho + (s.Ho + S - 1) / S - 1) / ((s.Ho + S - 1) / S); // no empty strips
    // small planes: images side by side until every wavefront has a chunk, where that leaves two workgroups per CU
    if (S == 1)
        while (NI < 8 && NI < s.N && NI * s.H * s.W < 6 * 16 * *PX && xd_geometry(s, *T, S, 2 * NI, a) <= 52 * 1024 &&
               (long long)(s.N + 2 * NI - 1) / (2 * NI) * a.CG >= 512)
            NI *= 2;
    *lds = xd_geometry(s, *T, S, NI, a);
    if (*lds > 60 * 1024)
        return false;
    const long long wgs = (long long)((s.N + NI - 1) / NI) * S * a.CG;
    // Where the line lies (one forward pass, the launches it replaces / this kernel, us).  Long contractions hold a compute
    // unit with one or two workgroups, and a second round of them loses to kernels whose operands are split once for all rows:
    // 80 -> 480 on 14x14, 3x3, 16 and 32 images 32.0 / 29.9 and 37.9 / 43.4; 112 -> 672 on 14x14, 5x5, 4 and 8 images 26.0 /
    // 22.3 and 32.4 / 40.8; 192 -> 1152 on 7x7, 2 and 4 images 27.6 / 22.0 and 29.0 / 35.7.  Up to 24 input channels it is the
    // faster one at any size (24 -> 144 on 56x56, 3x3, 32 and 128 images 69.8 / 68.4 and 248 / 205; 16 -> 96 on 112x112, 3x3,
    // stride 2, 64 images 195 / 143), but for 5x5 filters with stride 2 (24 -> 144 on 56x56, 16 and 32 images 36.9 / 32.6 and
    // 51.1 / 52.5), rows of an MFMA tile without a channel (8 -> 24
    // on 108x108, stride 2, 73 images 67.4 / 71.0) and small planes, which leave wavefronts without pixels (24 -> 144, 3x3 on
    // 14x14, 512 images 80.8 / 82.5, 5x5 on 7x7, 1024 images 73.0 / 82.2).
    // 5x5 filters with stride 1 have the matrix unit wait for the filter's vector work: up to one workgroup to a compute unit
    // (24 -> 144, 4 and 16 images of 56x56 28.0 / 21.5 and 51.9 / 55.6, 256 of 28x28 135 / 154).  24x24 is one row too tall for a
    // strip (256 images, 3x3, 89.2 / 97.9).
    const bool large = 10 * s.C >= 8 * kXdRows * a.CG && s.k == 3 && s.H * s.W >= 784;
    if (wgs > (*T > 20 || (s.k == 5 && s.s == 1) ? 256 : *T > 6 ? 512 : large ? 1 << 30 : 1024))
        return false;
    // The strips of wide planes are a few rows, and what they compute twice loses first where every compute unit is busy
    // anyway (16 -> 96 channels, one and eight images: 72x72, 3x3, 1.25 rows for each, 17.8 / 15.0 and 37.2 / 32.1; 96x96, 3x3, 1.4,
    // 20.2 / 18.5 and 44.2 / 46.0; 128x128, 3x3, 1.7, 25.0 / 24.6 and 62.1 / 65.7; 112x112, 5x5, 3, 23.9 / 29.4 and 60.2 / 73.4;
    // stride 2: 112x112, 3x3, 1.25, 19.6 / 15.2 and 38.1 / 37.0; 72x72, 5x5, 1.5, 17.9 / 12.0 and 36.9 / 23.9; 112x112, 5x5, 2.5,
    // 20.7 / 23.3; 24 -> 144, 5x5, 64 images: 48x48, 1.5, 95.8 / 116.7).  Nor, with stride 1, does a last round of workgroups pay that is nearly
    // empty (two to a compute unit; 24 -> 144, 3x3, 16 images: 48x48, 576, 40.2 / 41.2; 64x64, 1152, 52.5 / 53.4;
    // 64 images of 20x20, 576, 33.9 / 35.5).
    const int most = wgs <= 256 || s.s == 2 ? 175 : 130; // per cent
    if (100 * rows > most * s.H || (s.s == 1 && wgs > 512 && 5 * wgs < 4 * 512 * ((wgs + 511) / 512)))
        return false;
    // Rows of whole fours, which the separate launches are fastest on: of long contractions a second workgroup to a compute unit
    // draws or loses (25 shapes, 0.83 to 1.07 of their time; 80 -> 320 on 12x12, 3x3, 16 images 23.4 / 28.1, 32 -> 192 on
    // 64x64, 3x3, 4 images 30.5 / 34.4; 80 -> 240 on 28x28, 5x5, stride 2, 9 images 25.0 / 28.6), but for stride 2 with 3x3, and up
    // to 40 channels stride 2 and planes of one strip (32 -> 192 on 36x36, 3x3, stride 2, 9 images 28.6 / 19.9, on 72x72, 5x5, 3
    // images 33.7 / 23.3; 40 -> 240 on 16x16, 31 images 24.1 / 21.1, but on 12x12, 40 -> 160, 30 images 19.5 / 22.5).
    const bool fours = s.W % 4 == 0;
    const int runs = a.R * ((s.Wo + 3) / 4);
    const bool tail = s.k == 3 && runs > 32 && runs < 43; // a second round of a channel's 32 threads for a few runs
    if (*T > 6 && wgs > 256 && fours && (*T > 10 ? s.s == 1 || s.k == 5 : s.s == 1 && (S > 1 || tail)))
        return false;
    // The longest, which a compute unit has one workgroup of and which take the steps of 192 channels whatever they have, lose
    // where wavefronts have a second chunk of pixels to take (160 -> 960 on 12x12, 3x3, 3 images 26.5 / 33.3, on 8x8 21.0 / 17.2;
    // 144 -> 432 on 16x16, 4 images 21.8 / 25.8; 176 -> 528 on 22x22, 2 images 25.6 / 31.8), unless the launch leaves half of
    // the compute units idle or the channels are whole 64s (192 -> 1152 on 12x12, 3 images 28.0 / 26.2).
    const int strip = std::min(a.rin, s.H) * s.W;
    if (*T > 28 && wgs > 128 && s.s == 1 && K % 64 != 0 && s.H * s.W % 4 == 0 && strip > (fours ? 140 : 200))
        return false;
    // Many channels from 17 to 24, stride 2, on large planes: strips that compute an eighth and more twice lose 2 to 11 % once
    // the launch is several rounds (24 -> 144, 3x3, 56x56, 64 and 72 images 74.0 / 76.1 and 78.0 / 83.0; 64x64, 64 images 85.2 /
    // 87.2; 22 -> 132 on 112x112, 17 images 75.0 / 83.9), until the expanded tensor that they save no longer lies in the last
    // cache (52x52, 92 and 123 images 90 / 94 and 129 / 111).  Strips of less than five rows, which the
    // tile leaves where a plane is wider, bear more (68x68, 119 %, 26 images 64.7 / 56.9).
    if (s.s == 2 && *T == 6 && a.CG >= 8 && s.H * s.W >= 2500 && wgs > 1750 && (long long)s.N * s.C * s.H * s.W < 40000000 &&
        100 * rows >= (a.R >= 5 ? 117 : 125) * s.H)
        return false;
    // (four and eight images side by side, rows of an odd number of pairs: 24 -> 144 on 8x6, 376 images 24.6 / 30.5)
    if (NI >= 4 && s.s == 1 && s.W % 4 == 2 && wgs > 512)
        return false;
    a.rt = s.s == 1 && a.R * ((s.Wo + 3) / 4) >= 3 * 32 ? 2 : 1;
    a.items = (s.N + NI - 1) / NI * S;
    a.PL = 1;
    if (wgs > 4096) // (the weights staged once for several: 128 images of 56x56 above 215 -> 205 us)
        a.PL = (int)std::min<long long>((wgs + 4095) / 4096 * 2, 8);
    a.groups = (a.items + a.PL - 1) / a.PL;
    a.perDie = a.groups >= 64 ? (a.groups + 7) / 8 * a.CG : 0;
    return true;
}

bool eval_expand_dw_plan(const DwShape &s, int K, int *strips)
{
    XdArgs a = {};
    int T, PX;
    size_t lds;
    if (!xd_plan(s, K, a, &T, &PX, &lds))
        return false;
    *strips = a.S;
    return true;
}

// Partial sums per image and squeezed channel that launch_eval_expand_dw writes where it is given `q`; 0: it cannot
int eval_expand_dw_qparts(const DwShape &s, int K, int Cse)
{
    XdArgs a = {};
    int T, PX;
    size_t lds;
    if (Cse > 64 || !xd_plan(s, K, a, &T, &PX, &lds) || a.PL != 1)
        return 0;
    return a.CG * a.S;
}

hipError_t launch_eval_expand_dw(const DwShape &s, int K, const void *x, const void *w_expand, const void *w_dw, void *d,
                                 float *z, float *q, int Cse, const float *w1, bool act, const DwEval &ev_in, hipStream_t st)
{
    XdArgs a = {};
    int T, PX;
    size_t lds;
    if (!xd_plan(s, K, a, &T, &PX, &lds))
        return hipErrorInvalidValue;
    a.N = s.N;
    a.K = K;
    a.C = s.C;
    a.H = s.H;
    a.W = s.W;
    a.Ho = s.Ho;
    a.Wo = s.Wo;
    a.k = s.k;
    a.s = s.s;
    a.Cse = Cse;
    a.divCG = make_div((uint32_t)a.CG);
    a.divS = make_div((uint32_t)a.S);
    a.divW = make_div((uint32_t)s.W);
    a.divHW = make_div((uint32_t)(s.H * s.W));
    a.divRuns = make_div((uint32_t)((s.Wo + 3) / 4));
    a.x = (const float *)x;
    a.w = (const float *)w_expand;
    a.wdw = (const float *)w_dw;
    a.w1 = w1;
    a.d = (float *)d;
    a.z = q ? nullptr : z;
    a.q = q;
    a.act = act;
    DwEval ev = ev_in;
    // small launches: channel group, item group (no division ahead of the loads); workgroups past the items are the extra ones
    const unsigned main = a.perDie ? 8u * (unsigned)a.perDie : (unsigned)(a.groups * a.CG);
    const unsigned extra = dw_eval_extra_blocks(ev, main, kXdThreads);
    const dim3 grid = a.perDie ? dim3(main + extra) : dim3(a.CG, a.groups + (extra + a.CG - 1) / a.CG);
#define MBK_GO(T_, TP_, PX_, K_, S_, RT_)                                                         \
    if (s.k == K_ && s.s == S_ && a.rt == RT_) {                                                  \
        hipLaunchKernelGGL((xd_kernel<T_, TP_, PX_, K_, S_, RT_>), grid, dim3(kXdThreads), lds, st, a, ev); \
        return hipGetLastError();                                                                 \
    }
#define MBK_CASE(T_, TP_, PX_)                                                                    \
    if (T == T_ && PX == PX_) {                                                                   \
        MBK_GO(T_, TP_, PX_, 3, 1, 1)                                                             \
        MBK_GO(T_, TP_, PX_, 5, 1, 1)                                                             \
        MBK_GO(T_, TP_, PX_, 3, 1, 2)                                                             \
        MBK_GO(T_, TP_, PX_, 5, 1, 2)                                                             \
        MBK_GO(T_, TP_, PX_, 3, 2, 1)                                                             \
        MBK_GO(T_, TP_, PX_, 5, 2, 1)                                                             \
    }
    MBK_CASE(4, 0, 1) MBK_CASE(4, 0, 2) MBK_CASE(4, 0, 4)
    MBK_CASE(6, 4, 1) MBK_CASE(6, 4, 2) MBK_CASE(6, 4, 4)
    MBK_CASE(10, 6, 1) MBK_CASE(10, 6, 2) MBK_CASE(10, 6, 4)
    MBK_CASE(16, 10, 1) MBK_CASE(16, 10, 2) MBK_CASE(16, 10, 4)
    MBK_CASE(20, 16, 1) MBK_CASE(20, 16, 2)
    MBK_CASE(28, 20, 1) MBK_CASE(28, 20, 2)
    MBK_CASE(48, 28, 1)
#undef MBK_CASE
#undef MBK_GO
    return hipErrorInvalidValue;
}


// ---- a block without squeeze-and-excitation in one launch ----
//
//   out[n][m] = BN3(sum_c W_p[m][c] act(BN2(depthwise(act(BN1(W_e x[n])))[c]))) (+ x)
//
// Without a gate nothing couples the planes, so a workgroup takes its pixels through the whole block, sixteen expanded
// channels at a time: expansion conv, BN1 and activation into the LDS tile (as above), depthwise conv, BN2 and activation
// into a second one, and the projection conv's products with those sixteen channels into sums that stay in registers.
// Neither e nor d exists in memory.  A wavefront has 64 pixels of the strip's input, which it holds in registers for all
// channels, and 64 of its output; two barriers per sixteen channels.  What bounds it: MFMAs and vector instructions in turn
// (fp32 MFMAs do not overlap with them), a workgroup to a compute unit: 3.9 us for sixteen channels of 504 pixels.  Held to the
// 128 registers that would let two share one it spills inside the loop (32 images of 56x56 39.4 -> 43.6 us, 128 153 -> 169).
// 24 -> 144 -> 24 on 56x56, 32 images: 69.5 us in three launches, 54.7 in two, 39.4 here.
namespace {

struct XfArgs {
    XdArgs x;
    int M, dstr;     // output channels; floats per channel of the second tile
    const float *wp; // [M][C]
    const float *res;
    float *out;
};

template <int T, int TP, int PX, int KD, int MT>
__global__ __launch_bounds__(kXdThreads, 2) void xf_kernel(XfArgs f, DwEval ev)
{
    const XdArgs &a = f.x;
    constexpr int threads = kXdThreads, WP = 4 * T + 4, KK = KD * KD, RT = 2;
    constexpr int WL = kXdRows * WP, WB = WL + 256 * MT + kXdRows * KK; // floats of one group's weights
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ float cf3[2 * 16 * MT]; // BN3 {scale, shift}
    float *cf = lds + 2 * WB;          // {BN1 scale, shift, BN2 scale, shift} of every expanded channel
    float *tile = cf + 4 * kXdRows * a.CG, *dt = tile + kXdRows * a.chs;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int K = a.K, C = a.C, HW = a.H * a.W;
    const XdItem it = xd_item<KD, 1>(a, blockIdx.x);

    // the wavefront's input pixels: column j of the lane is pixel 4r + j, 32 (j/2) + 2r + j%2 or 16j + r
    float b[T][4];
    int toff[4]; // where they go in the tile, -1: nowhere
#pragma unroll
    for (int j = 0; j < 4; j += PX) {
        int pix = it.p0 + 64 * wave + (PX == 4 ? 4 * r : PX == 2 ? 16 * j + 2 * r : 16 * j + r);
        const bool in = pix < it.p1;
        pix = in ? pix : it.p0;
        const int im = a.NI > 1 ? (int)fdiv((uint32_t)pix, a.divHW) : 0, pl = pix - im * HW;
        const int h = (int)fdiv((uint32_t)pl, a.divW), w = pl - h * a.W;
#pragma unroll
        for (int e = 0; e < PX; ++e)
            toff[j + e] = in ? im * a.ims + (h - it.hin0) * a.pitch + 4 + w + e : -1;
        const char *px = reinterpret_cast<const char *>(a.x + (size_t)it.n * K * HW);
        const uint32_t at = (uint32_t)(im * K * HW + pl), off = 4u * ((uint32_t)(g * HW) + at);
#pragma unroll
        for (int s = 0; s < T; ++s) {
            const float *q = reinterpret_cast<const float *>(
                px + (s < TP ? off + (uint32_t)s * (16u * (uint32_t)HW) : 4u * ((uint32_t)(min(4 * s + g, K - 1) * HW) + at)));
            if (PX == 4) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(q);
#pragma unroll
                for (int e = 0; e < PX; ++e)
                    b[s][(j + e) % 4] = v[e];
            } else if (PX == 2) {
                const f32x2 v = *reinterpret_cast<const f32x2 *>(q);
#pragma unroll
                for (int e = 0; e < PX; ++e)
                    b[s][(j + e) % 4] = v[e];
            } else {
                b[s][j] = q[0];
            }
        }
    }
    // one group's weights: requested (load) and parked (park); W_e as in xd_kernel, W_p and the filters in the order of use
    constexpr int WN = (64 * T + threads - 1) / threads, PN = (256 * MT + threads - 1) / threads;
    float wv[WN], pv[PN], fv;
    const auto load = [&](int cg) __attribute__((always_inline)) {
        const int c0 = cg * kXdRows;
#pragma unroll
        for (int i = 0; i < WN; ++i) {
            const uint32_t idx = (uint32_t)(tid + i * threads), m = idx / (4 * T), kk = idx % (4 * T);
            wv[i] = a.w[(size_t)min(c0 + (int)m, C - 1) * K + min((int)kk, K - 1)];
        }
#pragma unroll
        for (int i = 0; i < PN; ++i) { // [row tile][step][lane]
            const int idx = tid + i * threads, ln = idx & 63, st = (idx >> 6) & 3, m = 16 * (idx >> 8) + (ln & 15);
            pv[i] = f.wp[(size_t)min(m, f.M - 1) * C + min(c0 + 4 * st + (ln >> 4), C - 1)];
        }
        fv = a.wdw[min(c0 * KK + tid, C * KK - 1)];
    };
    const auto park = [&](int cg) __attribute__((always_inline)) {
        float *wl = lds + (cg & 1) * WB;
#pragma unroll
        for (int i = 0; i < WN; ++i) {
            const uint32_t idx = (uint32_t)(tid + i * threads), m = idx / (4 * T), kk = idx % (4 * T);
            if (idx < 64 * T)
                wl[m * WP + (kk & 3) * T + (kk >> 2)] = (int)kk < K ? wv[i] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < PN; ++i) {
            const int idx = tid + i * threads, c = cg * kXdRows + 4 * ((idx >> 6) & 3) + ((idx & 63) >> 4);
            if (idx < 256 * MT) // (channels past the end: zero)
                wl[WL + idx] = c < C ? pv[i] : 0.f;
        }
        if (tid < kXdRows * KK)
            wl[WL + 256 * MT + tid] = fv;
    };
    load(0);
    for (int c = tid; c < kXdRows * a.CG; c += threads) {
        const BnEvalRegs r1 = bn_eval_issue(ev.bn1, min(c, C - 1)), r2 = bn_eval_issue(ev.bn2, min(c, C - 1));
        const BnEvalCoef k1 = bn_eval_coef(r1, ev.eps), k2 = bn_eval_coef(r2, ev.eps);
        *reinterpret_cast<f32x4 *>(cf + 4 * c) = (f32x4){k1.scale, k1.shift, k2.scale, k2.shift};
    }
    if (tid < 16 * MT) {
        const BnEvalCoef k3 = bn_eval_coef(bn_eval_issue(ev.bn3, min(tid, f.M - 1)), ev.eps);
        cf3[2 * tid] = k3.scale;
        cf3[2 * tid + 1] = k3.shift;
    }
    // the tile's zero columns, and its rows outside the plane
    for (int row = tid; row < kXdRows * a.NI * a.rin; row += threads) {
        const int rr = row >> 4, h = it.hin0 + rr - (a.NI > 1 ? (int)((uint32_t)rr / (uint32_t)a.rin) * a.rin : 0);
        float *p = tile + (row & 15) * a.chs + rr * a.pitch;
        const bool out = h < 0 || h >= a.H;
        for (int c = 0; c < a.pitch; c += 4)
            if (out || c == 0 || c + 4 > 4 + a.W)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (out || c == 0 || c + e >= 4 + a.W)
                        p[c + e] = 0.f;
    }
    park(0);
    __syncthreads();

    const int rw = (a.Wo + 3) >> 2, rows = min(a.R, a.Ho - it.ho0), opx = 4 * rw; // (a row of the second tile: opx)
    const int ch = tid >> 5, tpi = 32 / a.NI, dim = a.NI == 1 ? 0 : (tid & 31) / tpi, lt = tid & (tpi - 1);
    const int runs = (a.R + RT - 1) / RT * rw;
    f32x4 sum[MT][4];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            sum[m][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    constexpr f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    for (int cg = 0; cg < a.CG; ++cg) {
        const float *wl = lds + (cg & 1) * WB, *wps = wl + WL, *wd = wps + 256 * MT;
        if (cg + 1 < a.CG)
            load(cg + 1);
        // ---- expansion ----
        {
            // (long contractions in chains of five steps, each of which rounds the whole sum so far: in one chain the error of 40 ->
            // 240 -> 40 was 1.72e-7, of the separate launches 1.62, so 1.52; 93.3 -> 94.5 us, 128 images of 28x28)
            constexpr int CH = T > 6 ? 5 : T;
            f32x4 acc[4], e4[4];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const float av = wl[r * WP + g * T + t];
                const uint32_t ok = t < TP || 4 * t + g < K ? 0xffffffffu : 0u;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, t < TP ? b[t][j] : and_mask(b[t][j], ok),
                                                                  t % CH ? acc[j] : zero, 0, 0, 0);
                    if (t % CH == CH - 1 || t == T - 1)
                        e4[j] = t < CH ? acc[j] : e4[j] + acc[j];
                }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const f32x2 k = *reinterpret_cast<const f32x2 *>(cf + 4 * (cg * kXdRows + 4 * g + v));
                float *p = tile + (4 * g + v) * a.chs;
                float y[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    y[j] = actf(fmaf(e4[j][v], k[0], k[1]));
                if (PX == 4) {
                    if (toff[0] >= 0)
                        *reinterpret_cast<f32x4 *>(p + toff[0]) = (f32x4){y[0], y[1], y[2], y[3]};
                } else if (PX == 2) {
#pragma unroll
                    for (int j = 0; j < 4; j += 2)
                        if (toff[j] >= 0)
                            *reinterpret_cast<f32x2 *>(p + toff[j]) = (f32x2){y[j], y[j + 1]};
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (toff[j] >= 0)
                            p[toff[j]] = y[j];
                }
            }
        }
        __syncthreads();
        if (cg + 1 < a.CG) // (the other buffer's readers are past this barrier)
            park(cg + 1);
        // ---- depthwise ----
        {
            float wt[KK];
#pragma unroll
            for (int t = 0; t < KK; ++t)
                wt[t] = wd[ch * KK + t];
            const f32x2 k2 = *reinterpret_cast<const f32x2 *>(cf + 4 * (cg * kXdRows + ch) + 2);
            const float *tc = tile + ch * a.chs + dim * a.ims + 4;
            float *dc = dt + ch * f.dstr + dim * a.R * opx;
            for (int i = lt; i < runs; i += tpi) {
                const int rg = (int)fdiv((uint32_t)i, a.divRuns), j = i - rg * rw, oh = RT * rg;
                const float *p = tc + 4 * j;
                float o[RT][4];
#pragma unroll
                for (int q = 0; q < RT; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        o[q][e] = 0.f;
#pragma unroll
                for (int ir = 0; ir < RT - 1 + KD; ++ir) {
                    float row[3 + KD];
                    xd_window<KD, 1>(p + min(oh + ir, a.rin - 1) * a.pitch, row);
#pragma unroll
                    for (int q = 0; q < RT; ++q) {
                        const int u = ir - q;
                        if (u >= 0 && u < KD) {
#pragma unroll
                            for (int v = 0; v < KD; ++v)
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    o[q][e] = fmaf(wt[u * KD + v], row[e + v], o[q][e]);
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < RT; ++q) {
                    if (oh + q < a.R) {
                        f32x4 y;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            y[e] = actf(fmaf(o[q][e], k2[0], k2[1]));
                        *reinterpret_cast<f32x4 *>(dc + (oh + q) * opx + 4 * j) = y;
                    }
                }
            }
        }
        __syncthreads();
        // ---- projection: (what lies past a row or a strip gives columns that are not stored) ----
        f32x4 acc[MT][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const f32x4 bq = *reinterpret_cast<const f32x4 *>(dt + (4 * s + g) * f.dstr + 64 * wave + 4 * r);
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const float av = wps[m * 256 + s * 64 + lane];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bq[j], s ? acc[m][j] : zero, 0, 0, 0);
            }
        }
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                sum[m][j] += acc[m][j];
    }
    // ---- the lane's four output pixels of its rows ----
    const int q = 64 * wave + 4 * r, row = (int)fdiv((uint32_t)q, a.divRuns4), col = q - row * opx;
    const int im = a.NI == 1 ? 0 : (int)((uint32_t)row / (uint32_t)a.R), oh = row - im * a.R;
    if (im >= it.ni || oh >= rows)
        return;
    const int left = a.Wo - col;
    const size_t HWo = (size_t)a.Ho * a.Wo, base = (size_t)(it.n + im) * f.M * HWo + (size_t)(it.ho0 + oh) * a.Wo + col;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int mm = 16 * m + 4 * g + v;
            if (mm < f.M) {
                const float sc = cf3[2 * mm], sh = cf3[2 * mm + 1];
                const size_t at = base + (size_t)mm * HWo;
                if ((a.Wo & 3) == 0) {
                    f32x4 y;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        y[j] = fmaf(sum[m][j][v], sc, sh);
                    if (f.res)
                        y += *reinterpret_cast<const f32x4 *>(f.res + at);
                    *reinterpret_cast<f32x4 *>(f.out + at) = y;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (j < left)
                            f.out[at + j] = fmaf(sum[m][j][v], sc, sh) + (f.res ? f.res[at + j] : 0.f);
                }
            }
        }
}

} // namespace

// Whether the shape is taken; the plan.
static bool xf_plan(const DwShape &s, int K, int M, XfArgs &f, int *T, int *PX, int *MT, size_t *lds)
{
    XdArgs &a = f.x;
    // (stride 1: with 2 a strip's input is four times its output, 16 -> 96 on 112x112, 64 images 113 us in two launches / 266)
    if (!xd_form(K, s.W, T, PX) || *T > 10 || M > 64 || s.C > 1024 || s.s != 1)
        return false;
    *T = std::max(*T, 6);
    *MT = M <= 16 ? 1 : M <= 32 ? 2 : 4;
    a.CG = (s.C + kXdRows - 1) / kXdRows;
    // strips whose input and output (in runs of four) are at most 64 pixels to a wavefront, or images side by side
    const int opx = 4 * ((s.Wo + 3) / 4);
    int S = 1, NI = 1;
    for (;; ++S) {
        xd_geometry(s, *T, S, 1, a);
        if (std::min(a.rin, s.H) * s.W <= 512 && a.R * opx <= 512)
            break;
        if (S >= s.Ho)
            return false;
    }
    S = (s.Ho + a.R - 1) / a.R; // no empty strips
    if (S == 1)
        while (NI < 8 && NI < s.N && 2 * NI * s.H * s.W <= 512 && 2 * NI * s.Ho * opx <= 512)
            NI *= 2;
    xd_geometry(s, *T, S, NI, a);
    f.dstr = NI * a.R * opx;
    f.dstr = std::max(f.dstr, 512); // (a wavefront reads its 64 pixels whether they exist or not)
    f.dstr += 16;
    const int KK = s.k * s.k, WB = kXdRows * (4 * *T + 4) + 256 * *MT + kXdRows * KK;
    *lds = sizeof(float) * (size_t)(2 * WB + 4 * kXdRows * a.CG + kXdRows * a.chs + kXdRows * f.dstr);
    a.items = (s.N + NI - 1) / NI * S;
    return *lds <= 156 * 1024;
}

bool eval_block_plan(const DwShape &s, int K, int M)
{
    XfArgs f = {};
    int T, PX, MT;
    size_t lds;
    if (!xf_plan(s, K, M, f, &T, &PX, &MT, &lds))
        return false;
    // A workgroup takes as long for a strip of a few pixels as for 512, so a round of 256 takes 4 to 6 us for sixteen
    // channels however much of it is output; the other launches take time by the pixel, and some for being two or three. So:
    // the share of the rounds' places that have an output pixel, with what those launches cost counted as pixels. Where it
    // lies is a fit to 1029 blocks measured on more than one route; of the 604 it takes thirteen are 2 to 12 % slower than
    // in separate launches (one forward pass, ReLU6, best other route / one launch, us). 24 -> 144 -> 24 on 56x56, 3x3, 8
    // workgroups to an image: 10 images 31.5 / 37.7, 13 39.3 / 37.8, 16 38.7 / 37.9, 32 56.5 / 38.9, 33 (a second round)
    // 58.5 / 74.2, 48 76.7 / 74.7, 64 94.5 / 76.4. 32 -> 192 -> 32 on 28x28, 3x3: 56 images 51.6 / 54.2, 72 57.6 / 54.3, 128
    // 84.6 / 55.8, 160 96.3 / 107, 192 115 / 107. 40 -> 240 -> 40, 5x5: on 14x14, 320 images 86.6 / 100.5, 400 105 / 102;
    // 26x28, 270 images 247 / 288. Rows of the output past a multiple of sixteen count, too: 24 -> 96 -> 39 on 40x40, 5x5,
    // 126 images 91 / 116, 32 -> 96 -> 37 on 80x80, 35 images 94 / 107. The other launches are slower on rows that are not
    // whole fours: 32 -> 128 -> 34 on 81x83, 71 images 386 / 315, 28 -> 84 -> 28 on 45x42, 5x5, 315 images 447 / 305. An
    // expanded tensor of more than the 256 MB of the last cache costs them, too: 40 -> 160 -> 40 on 68x68, 88 images 364 /
    // 289. Few workgroups leave the chip empty (24 -> 72 -> 36 on 22x22, 67 images, 134 workgroups, 22.8 / 32.7).
    const long long rounds = (f.x.items + 255) / 256, pixels = (long long)s.N * s.Ho * s.Wo + 4000000 / s.C;
    const bool large = (long long)s.N * s.C * s.H * s.W > 60000000;
    const int share = (s.k == 3 ? 60 : T > 6 ? 70 : 65) + (M > 32 ? 10 : 0) - (s.W % 4 ? 10 : 0) - (large ? 10 : 0); // per cent
    return f.x.items >= (M > 32 ? 160 : 100) && 100 * pixels >= share * rounds * 256 * 512;
}

hipError_t launch_eval_block(const DwShape &s, int K, int M, const void *x, const void *w_expand, const void *w_dw,
                             const void *w_proj, const void *res, void *out, const DwEval &ev, hipStream_t st)
{
    XfArgs f = {};
    int T, PX, MT;
    size_t lds;
    if (!xf_plan(s, K, M, f, &T, &PX, &MT, &lds))
        return hipErrorInvalidValue;
    XdArgs &a = f.x;
    a.N = s.N;
    a.K = K;
    a.C = s.C;
    a.H = s.H;
    a.W = s.W;
    a.Ho = s.Ho;
    a.Wo = s.Wo;
    a.k = s.k;
    a.s = s.s;
    a.divS = make_div((uint32_t)a.S);
    a.divW = make_div((uint32_t)s.W);
    a.divHW = make_div((uint32_t)(s.H * s.W));
    a.divRuns = make_div((uint32_t)((s.Wo + 3) / 4));
    a.divRuns4 = make_div((uint32_t)((s.Wo + 3) / 4 * 4));
    a.x = (const float *)x;
    a.w = (const float *)w_expand;
    a.wdw = (const float *)w_dw;
    f.M = M;
    f.wp = (const float *)w_proj;
    f.res = (const float *)res;
    f.out = (float *)out;
#define MBK_GO(T_, TP_, PX_, K_, MT_)                                                             \
    if (T == T_ && PX == PX_ && s.k == K_ && MT == MT_) {                                         \
        auto kern = xf_kernel<T_, TP_, PX_, K_, MT_>;                                             \
        const hipError_t e_ = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
        if (e_ != hipSuccess)                                                                     \
            return e_;                                                                            \
        hipLaunchKernelGGL(kern, dim3(a.items), dim3(kXdThreads), lds, st, f, ev);                \
        return hipGetLastError();                                                                 \
    }
#define MBK_MT(T_, TP_, PX_, K_) MBK_GO(T_, TP_, PX_, K_, 1) MBK_GO(T_, TP_, PX_, K_, 2) MBK_GO(T_, TP_, PX_, K_, 4)
#define MBK_KS(T_, TP_, PX_) MBK_MT(T_, TP_, PX_, 3) MBK_MT(T_, TP_, PX_, 5)
#define MBK_T(T_, TP_) MBK_KS(T_, TP_, 1) MBK_KS(T_, TP_, 2) MBK_KS(T_, TP_, 4)
    MBK_T(6, 0)
    MBK_T(10, 6)
#undef MBK_T
#undef MBK_KS
#undef MBK_MT
#undef MBK_GO
    return hipErrorInvalidValue;
}

// ---- projection conv of small launches, with the squeeze-and-excitation gate and BN3 ----
//
//   out[n][m] = BN3(sum_k W_p[m][k] act(BN2(d[n][k])) g[n][k]) (+ x),  g = sigmoid(W2 swish(q) + b2)
//
// A request's projection conv is a chain of latencies: with a wavefront for every eighth of the contraction and
// a launch ahead of it for the gate it took 7 to 11 us, and the gate 3 to 6.  A workgroup owns 16 output channels by 16*PX
// pixels of one image and its wavefronts cut the contraction into slices of 4*T channels, everything that a
// wavefront needs (its part of W_p, d, W2, the coefficients) being requested before the first use.  q comes as the
// expansion kernel's partial sums, which the wavefronts share out and add through LDS; the gate of a wavefront's
// channels is its own work, and so needs no barrier.  The slices' tiles are added in a fixed order.
// One image, gate and projection in two launches / here: 1152 -> 192 on 7x7 5.7 + 11.3 / 13.2 us, 672 -> 112 on 14x14
// 4.0 + 9.4 / 7.8, 240 -> 40 on 28x28 2.5 + 6.5 / 4.4, 144 -> 24 on 56x56 2.6 + 7.6 / 5.3; sixteen blocks 349 -> 278 us with
// both kernels of this file.
namespace {

constexpr int kXpWaves = 16;

struct XpArgs {
    int M, K, HW, Cse, parts; // parts == 0: no gate from q
    const float *w, *d, *bn2, *bn3; // [M][K]; normalisation blocks {scale, shift, ...}
    const float *q, *b1, *w2, *b2;  // [n][parts][Cse]
    const float *g;                 // gate [n][K], where there is one in memory
    const float *res;
    float *out;
};

// JR: pieces of 16 squeezed channels (0: no gate from q).  ACT: d is to go through BN2 and the activation (it has not yet).
template <int T, int PX, int JR, bool ACT>
__global__ __launch_bounds__(64 * kXpWaves) void xp_kernel(XpArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int tid = threadIdx.x, lane = tid & 63, KS = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int M = a.M, K = a.K, HW = a.HW;
    const int m0 = 16 * (int)blockIdx.x, p0 = 16 * PX * (int)blockIdx.y, n = blockIdx.z;
    f32x4 *part = reinterpret_cast<f32x4 *>(lds);          // [KS][PX][64]
    float *cs = lds + (size_t)KS * PX * 256 + wave * 16 * T; // the slice's channels: {BN2 scale, shift, gate, b2}
    float *qs = lds + (size_t)KS * PX * 256 + KS * 16 * T;   // [KS][64]

    // ---- the loads ----
    constexpr int QU = 8;
    float qv[QU], b1v = 0.f;
    constexpr int WR = T / 4 < 3 ? T / 4 : 3; // sixteen channels' W2 at a time in flight
    f32x4u w2v[WR][JR > 0 ? JR : 1];
    const int ks0 = 4 * T * wave, part4 = lane & 3;
    if (JR > 0) {
        const int j = min(lane, a.Cse - 1);
#pragma unroll
        for (int u = 0; u < QU; ++u)
            qv[u] = a.q[((size_t)n * a.parts + min(wave + u * KS, a.parts - 1)) * a.Cse + j];
        b1v = a.b1[j];
    }
    float cv[T / 4];
    {
        const float *pc4 = part4 == 0 ? a.bn2 : part4 == 1 ? a.bn2 + K : part4 == 2 ? (a.g ? a.g + (size_t)n * K : a.bn2) : JR > 0 ? a.b2 : a.bn2;
#pragma unroll
        for (int i = 0; i < T / 4; ++i)
            cv[i] = pc4[min(ks0 + 16 * i + (lane >> 2), K - 1)];
    }
    const auto fetch_w2 = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < JR; ++v)
            w2v[i % WR][v] = *reinterpret_cast<const f32x4u *>(a.w2 + (size_t)min(ks0 + 16 * i + (lane >> 2), K - 1) * a.Cse +
                                                               min(4 * (part4 + 4 * v), a.Cse - 4));
    };
#pragma unroll
    for (int i = 0; i < WR; ++i)
        fetch_w2(i);
    // contraction index of slot (i, e): min(kg, K - 4) + e with kg = ks0 + T g + 4 i; what a slot shares with another one
    // is masked, in both factors (either may be infinite)
    f32x4u av[T / 4];
    float b[T][PX];
    const int pix = p0 + PX * r;
    const bool in = pix < HW;
    const uint32_t pc = (uint32_t)(in ? pix : 0);
#pragma unroll
    for (int i = 0; i < T / 4; ++i) {
        const int kk = min(ks0 + T * g + 4 * i, K - 4);
        const float *pb = a.d + ((size_t)n * K + kk) * HW + pc;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (PX == 4) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(pb + (size_t)e * HW);
#pragma unroll
                for (int c = 0; c < PX; ++c)
                    b[4 * i + e][c] = v[c];
            } else if (PX == 2) {
                const f32x2 v = *reinterpret_cast<const f32x2 *>(pb + (size_t)e * HW);
#pragma unroll
                for (int c = 0; c < PX; ++c)
                    b[4 * i + e][c] = v[c];
            } else {
                b[4 * i + e][0] = pb[(size_t)e * HW];
            }
        }
    }
    const auto fetch_w = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < T / 4; ++i)
            av[i] = *reinterpret_cast<const f32x4u *>(a.w + (size_t)min(m0 + r, M - 1) * K + min(ks0 + T * g + 4 * i, K - 4));
    };
    // (long slices: under the gate's arithmetic, when the registers of its loads are free)
    constexpr bool kLateW = JR > 0 && T >= 20;
    if (!kLateW)
        fetch_w();
    // of the thread's output: BN3's coefficients and the residual
    const int orow = tid / (16 * PX), opx = tid % (16 * PX), om = min(m0 + orow, M - 1);
    const size_t oat = ((size_t)n * M + om) * HW + min(p0 + opx, HW - 1);
    const float o3 = a.bn3[om], o3s = a.bn3[M + om], ores = a.res ? a.res[oat] : 0.f;
    __builtin_amdgcn_sched_barrier(0);
    // ---- the gate ----
#pragma unroll
    for (int i = 0; i < T / 4; ++i)
        cs[64 * i + lane] = JR == 0 && part4 == 2 && !a.g ? 1.f : cv[i];
    if (JR > 0) {
        float s = 0.f;
#pragma unroll
        for (int u = 0; u < QU; ++u)
            s += wave + u * KS < a.parts ? qv[u] : 0.f;
        for (int p = wave + QU * KS; p < a.parts; p += KS)
            s += a.q[((size_t)n * a.parts + p) * a.Cse + min(lane, a.Cse - 1)];
        qs[wave * 64 + lane] = s;
        __syncthreads();
        if (kLateW)
            fetch_w();
        float t = b1v;
#pragma unroll
        for (int w = 0; w < kXpWaves; ++w)
            t += w < KS ? qs[min(w, KS - 1) * 64 + lane] : 0.f;
        // the squeezed channels of the lane's pieces, from the lanes that hold them
        const float rq = lane < a.Cse ? swishf(t) : 0.f;
        float rx[JR > 0 ? JR : 1][4];
#pragma unroll
        for (int v = 0; v < JR; ++v)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                rx[v][e] = __shfl(rq, min(4 * (part4 + 4 * v), a.Cse - 4) + e, kWave);
#pragma unroll
        for (int i = 0; i < T / 4; ++i) {
            float acc = 0.f;
#pragma unroll
            for (int v = 0; v < JR; ++v) {
                const int want = 4 * (part4 + 4 * v), at = min(want, a.Cse - 4);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc = fmaf(at + e >= want ? w2v[i % WR][v][e] : 0.f, at + e >= want ? rx[v][e] : 0.f, acc);
            }
            if (i + WR < T / 4)
                fetch_w2(i + WR);
            acc += __shfl_xor(acc, 1, kWave);
            acc += __shfl_xor(acc, 2, kWave);
            if (part4 == 3) // (the lane that has loaded b2)
                cs[64 * i + lane - 1] = sigmoidf_fast(acc + cv[i]);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // ---- the slice's product ----
    // (every instruction with a sum of its own, added in pairs: a chain rounds the whole sum at every step)
    f32x4 acc[PX][4], sum[PX];
#pragma unroll
    for (int i = 0; i < T / 4; ++i) {
        const int kg = ks0 + T * g + 4 * i, kk = min(kg, K - 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            constexpr f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            const int t = 4 * i + e;
            const bool ok = kk + e >= kg;
            const f32x4 k4 = *reinterpret_cast<const f32x4 *>(cs + 4 * max(kk + e - ks0, 0));
            const float w = ok ? av[i][e] : 0.f;
#pragma unroll
            for (int c = 0; c < PX; ++c) {
                const float v = ok ? (ACT ? actf(fmaf(b[t][c], k4[0], k4[1])) : b[t][c]) * k4[2] : 0.f;
                acc[c][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, v, zero, 0, 0, 0);
                if (e == 3) {
                    const f32x4 four = (acc[c][0] + acc[c][1]) + (acc[c][2] + acc[c][3]);
                    sum[c] = i == 0 ? four : sum[c] + four;
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < PX; ++c)
        part[(wave * PX + c) * 64 + lane] = sum[c];
    __syncthreads();
    // ---- the slices added up, BN3 and the residual: thread -> row, pixel ----
    const auto total = [&](int row, int px) __attribute__((always_inline)) {
        const float *ps = lds + 4 * ((px % PX) * 64 + (row >> 2) * 16 + px / PX) + (row & 3);
        float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kXpWaves; ++w)
            s[w & 3] += w < KS ? ps[min(w, KS - 1) * PX * 256] : 0.f;
        return (s[0] + s[1]) + (s[2] + s[3]);
    };
    if (tid < 256 * PX && m0 + orow < M && p0 + opx < HW)
        a.out[oat] = fmaf(total(orow, opx), o3, o3s) + ores;
    for (int o = tid + blockDim.x; o < 256 * PX; o += blockDim.x) { // (fewer threads than outputs)
        const int row = o / (16 * PX), px = o % (16 * PX), m = m0 + row;
        if (m < M && p0 + px < HW) {
            const size_t at = ((size_t)n * M + m) * HW + p0 + px;
            a.out[at] = fmaf(total(row, px), a.bn3[m], a.bn3[M + m]) + (a.res ? a.res[at] : 0.f);
        }
    }
}

long long xp_groups(int N, int M, int HW, int PX)
{
    return (long long)((M + 15) / 16) * ((HW + 16 * PX - 1) / (16 * PX)) * N;
}

// Steps of four channels to a wavefront, wavefronts, pixels to a lane (as many as leave most compute units a workgroup)
bool xp_form(int N, int M, int K, int HW, int Cse, int *T, int *KS, int *PX)
{
    if (K < 4 || K > kXpWaves * 80 || (Cse && (Cse < 4 || Cse > 64)))
        return false;
    for (const int t : {4, 8, 12, 20})
        if (K <= kXpWaves * 4 * t) {
            *T = t;
            *KS = (K + 4 * t - 1) / (4 * t);
            *PX = 1;
            if (HW % 2 == 0 && t <= 12 && xp_groups(N, M, HW, 2) >= 128)
                *PX = 2;
            if (HW % 4 == 0 && t <= 4 && *KS <= 10 && xp_groups(N, M, HW, 4) >= 128)
                *PX = 4;
            return true;
        }
    return false;
}

} // namespace

bool eval_proj_plan(int N, int M, int K, int HW, int Cse, bool act)
{
    int T, KS, PX;
    if (!xp_form(N, M, K, HW, Cse, &T, &KS, &PX) || N > 65535 || HW > 65535)
        return false;
    // Up to one workgroup of sixteen wavefronts to a compute unit; beyond, the gate and W_p that every workgroup fetches again
    // cost more than the launches (the SE stage and the projection conv / this kernel: 672 -> 112 on 14x14, 4 and 8 images 13.0 /
    // 10.4 and 15.5 / 19.7 us; 480 -> 80, 4 and 8 images 11.8 / 11.5, 12.7 / 15.2; 144 -> 24 on 56x56, 4 images 11.8 / 8.5).
    // With the activation still to apply, which each of them repeats, somewhat less (306 -> 34 on 16x16, 15 images, 3600
    // wavefronts, evaluation 23.9 / 24.7; 96 -> 24 on 128x128, one image,
    // 3072, 26.2 / 26.9).
    // With the activation to apply and four pixels to a lane, one workgroup to a compute unit is all that pays (evaluation, SE: 96
    // -> 24 on 12x12, 58 images, 348 workgroups, 20.7 / 22.3; 114 -> 38 on 16x16, 25 images, 300, 21.9 / 23.2; 96 -> 38 on 8x8,
    // 56 images, 168, 19.6 / 18.2; no SE: 48 -> 29 on 48x48, 10 images, 720, 12.1 / 13.5), but for short contractions (24 ->
    // 10 on 68x68, 11 images, 803, 21.7 / 18.5).
    const long long groups = xp_groups(N, M, HW, PX);
    return groups * KS <= (act ? 2600 : 4096) && !(act && PX == 4 && KS > (Cse ? 4 : 2) && groups > 256);
}

hipError_t launch_eval_proj(int N, int M, int K, int HW, int Cse, const void *w, const void *d, const float *bn2,
                            const float *bn3, const float *q, int parts, const float *b1, const float *w2,
                            const float *b2, const float *gate, bool act, const void *res, void *out, hipStream_t st)
{
    int T, KS, PX;
    if (!xp_form(N, M, K, HW, parts ? Cse : 0, &T, &KS, &PX) || (parts && act))
        return hipErrorInvalidValue;
    const XpArgs a = {M, K, HW, Cse, parts, (const float *)w, (const float *)d, bn2, bn3, q, b1, w2, b2, gate,
                      (const float *)res, (float *)out};
    const dim3 grid((M + 15) / 16, (HW + 16 * PX - 1) / (16 * PX), N);
    const size_t lds = sizeof(float) * ((size_t)KS * PX * 256 + KS * 16 * T + (parts ? KS * 64 : 0));
    const int jr = parts ? (Cse + 15) / 16 : 0;
#define MBK_CASE(T_, PX_, JR_, ACT_)                                                              \
    if (T == T_ && PX == PX_ && jr == JR_ && act == ACT_) {                                       \
        hipLaunchKernelGGL((xp_kernel<T_, PX_, JR_, ACT_>), grid, dim3(64 * KS), lds, st, a);     \
        return hipGetLastError();                                                                 \
    }
#define MBK_JR(T_, PX_)                                                                           \
    MBK_CASE(T_, PX_, 0, true) MBK_CASE(T_, PX_, 0, false) MBK_CASE(T_, PX_, 1, false) MBK_CASE(T_, PX_, 2, false) \
    MBK_CASE(T_, PX_, 3, false) MBK_CASE(T_, PX_, 4, false)
    MBK_JR(4, 1) MBK_JR(4, 2) MBK_JR(4, 4)
    MBK_JR(8, 1) MBK_JR(8, 2)
    MBK_JR(12, 1) MBK_JR(12, 2)
    MBK_JR(20, 1)
#undef MBK_JR
#undef MBK_CASE
    return hipErrorInvalidValue;
}

} // namespace mbk
