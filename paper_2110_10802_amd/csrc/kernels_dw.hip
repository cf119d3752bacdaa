// The memory-bound depthwise chain: one (image, channel) plane at a time.
//
// A whole plane (at most 112x112 fp32 = 49 KB) fits in the 160 KB LDS of a gfx950 CU,
// so a group of threads stages the plane once, applying BN + Swish on the way in (each
// activation is evaluated once per input element, not once per filter tap), with the
// zero padding materialised as a border in LDS (the paper's Pad+Conv fusion, section
// "Coarse-Grained Transformations"; MapTiling + LocalStorage, section "Local Data
// Movement Reduction").  The activation a1 = Swish(BN1(e)) therefore never exists in
// HBM: forward reads e and writes d, backward re-derives everything it needs from the
// pre-normalisation tensors (recomputation instead of load/store, section "Guided
// Optimization Case Study: EfficientNet", step "Full fusion and vectorization").
//
// Every reduction (BN partial sums, filter gradients) is a fixed-order tree inside the
// plane's thread group followed by a fixed-order sum over images in a later kernel; no
// atomics anywhere (the same section's "Map fission" step).
#include "mbconv_dev.h"
#include "mbconv_launch.h"
#include "mbconv_bnfin.h"
#include "mbconv_x3.h"
#include "mbconv_eval.h"

#include <algorithm>

namespace mbk {

// kernels_dw4.hip: vectorised variants for stride 1 and W % 4 == 0
bool dw4_supported(const DwShape &s);
hipError_t launch_dw4_fwd(bool bf16, const DwShape &s, const void *e, const float *bn1,
                          const void *w_dw, void *d, float *psum, float *psq, const BnFin *fin,
                          const DwEval *ev, hipStream_t st);
hipError_t launch_dw4_bwd(bool bf16, const DwBwdArgs &h, hipStream_t st);
// kernels_dw2.hip
bool dw2_supported(const DwShape &s);
hipError_t launch_dw2_fwd(bool bf16, const DwShape &s, const void *e, const float *bn1,
                          const void *w_dw, void *d, float *psum, float *psq, const DwEval *ev,
                          hipStream_t st);
hipError_t launch_dw2_bwd(bool bf16, const DwBwdArgs &h, hipStream_t st);
// kernels_dwr.hip
bool dwr_supported(const DwShape &s);
int dwr_num_partials(bool bf16, const DwShape &s, bool bwd);
hipError_t launch_dwr_fwd(bool bf16, const DwShape &s, const void *e, const float *bn1,
                          const void *w_dw, void *d, float *psum, float *psq, const BnFin *fin,
                          const DwEval *ev, hipStream_t st);
hipError_t launch_dwr_bwd(bool bf16, const DwBwdArgs &h, hipStream_t st);

int dw_num_partials(bool bf16, const DwShape &s, bool stores_a1, bool bwd)
{
    if (!stores_a1 && !dw4_supported(s) && dwr_supported(s))
        return dwr_num_partials(bf16, s, bwd);
    return s.N;
}

// Threads per plane: a wavefront for planes up to 16x16, a 256-thread workgroup up to
// 64x64, 1024 threads above.
static int pick_tpp(int plane_elems) { return plane_elems <= 256 ? 64 : plane_elems <= 4096 ? 256 : 1024; }
// The plane reductions and the final elementwise pass give a plane of at most 256 elements to
// 16 lanes (a DPP row): four planes per wavefront share the per-plane overhead (index
// arithmetic, coefficient loads, the reduction), which is most of the work on 14x14 and 7x7 planes.
static int pick_tpp_plane(int plane_elems)
{
    return plane_elems <= 256 ? 16 : plane_elems <= 1024 ? 64 : pick_tpp(plane_elems);
}

struct PlaneId {
    bool active;
    int n, c;
    size_t plane;
};

// CHAN: a workgroup's planes belong to one channel (BLOCK/TPP consecutive images), so that it can
// finalise that channel's normalisation itself, once for all of them.
template <int TPP, bool CHAN = false>
__device__ __forceinline__ PlaneId plane_of_group(int N, int C, FastDiv divC)
{
    constexpr int BLOCK = TPP > 256 ? TPP : 256;
    constexpr int PPB = BLOCK / TPP;
    PlaneId p;
    if (CHAN) {
        const int per = (N + PPB - 1) / PPB, g = threadIdx.x / TPP; // workgroups per channel
        p.c = blockIdx.x / per;
        p.n = (blockIdx.x - p.c * per) * PPB + g;
        p.active = p.n < N;
        p.n = p.active ? p.n : 0;
        p.plane = (size_t)p.n * C + p.c;
        return p;
    }
    const size_t plane = (size_t)blockIdx.x * PPB + threadIdx.x / TPP;
    p.active = plane < (size_t)N * C;
    p.plane = p.active ? plane : 0;
    p.n = (int)fdiv((uint32_t)p.plane, divC);
    p.c = (int)(p.plane - (size_t)p.n * C);
    return p;
}

// ---- forward: d = depthwise(swish(bn1(e))) + BN2 partial statistics ------------------------

struct DwFwdDev {
    DwShape s;
    FastDiv divC, divWp, divWo;
    const void *e;
    const float *bn1;
    const void *w;
    void *d;
    float *psum, *psq;
    void *a1_store;
};

template <typename T, int K, int S, int TPP, typename EVT>
__global__ __launch_bounds__(TPP > 256 ? TPP : 256) void dw_fwd_kernel(DwFwdDev a, EVT ev)
{
    constexpr int P = (K - 1) / 2;
    constexpr int BLOCK = TPP > 256 ? TPP : 256;
    constexpr int PPB = BLOCK / TPP;
    if constexpr (EVT::kEval) {
        if ((int)blockIdx.x >= ev.main) {
            dw_eval_extra(ev, (int)blockIdx.x - ev.main, BLOCK);
            return;
        }
    }
    extern __shared__ float lds[];
    const int H = a.s.H, W = a.s.W, Ho = a.s.Ho, Wo = a.s.Wo, C = a.s.C, N = a.s.N;
    const int Hp = H + 2 * P, Wp = W + 2 * P;
    const int lt = threadIdx.x % TPP;
    float *tile = lds + (threadIdx.x / TPP) * (Hp * Wp);
    float *red = lds + PPB * (Hp * Wp);
    const PlaneId pl = plane_of_group<TPP>(N, C, a.divC);

    float w[K * K];
    float scale = 1.f, shift = 0.f;
    const bool bn = a.bn1 != nullptr;
    BnEvalCoef k2 = {1.f, 0.f, 0.f, 1.f}; // evaluation mode
    if (pl.active) {
#pragma unroll
        for (int t = 0; t < K * K; ++t)
            w[t] = ld<T>((const T *)a.w, (size_t)pl.c * K * K + t);
        if constexpr (EVT::kEval) {
            k2 = bn_eval_coef(bn_eval_issue(ev.bn2, pl.c), ev.eps);
            if (bn) {
                const BnEvalCoef k1 = bn_eval_coef(bn_eval_issue(ev.bn1, pl.c), ev.eps);
                scale = k1.scale;
                shift = k1.shift;
            }
        } else if (bn) {
            scale = a.bn1[pl.c];
            shift = a.bn1[C + pl.c];
        }
        const size_t base = pl.plane * (size_t)H * W;
        for (int idx = lt; idx < Hp * Wp; idx += TPP) {
            const int hp = (int)fdiv((uint32_t)idx, a.divWp);
            const int wp = idx - hp * Wp;
            const int h = hp - P, x = wp - P;
            float v = 0.f;
            if (h >= 0 && h < H && x >= 0 && x < W) {
                v = ld<T>((const T *)a.e, base + (size_t)h * W + x);
                if (bn)
                    v = actf(fmaf(v, scale, shift));
                if (a.a1_store)
                    st<T>((T *)a.a1_store, base + (size_t)h * W + x, v);
            }
            tile[idx] = v;
        }
    }
    __syncthreads();
    float acc2[2] = {0.f, 0.f};
    if (pl.active) {
        const size_t obase = pl.plane * (size_t)Ho * Wo;
        for (int idx = lt; idx < Ho * Wo; idx += TPP) {
            const int i = (int)fdiv((uint32_t)idx, a.divWo);
            const int j = idx - i * Wo;
            const float *t0 = tile + (i * S) * Wp + j * S;
            float acc = 0.f;
#pragma unroll
            for (int u = 0; u < K; ++u)
#pragma unroll
                for (int v = 0; v < K; ++v)
                    acc = fmaf(w[u * K + v], t0[u * Wp + v], acc);
            st<T>((T *)a.d, obase + idx, acc);
            const float sv = as_stored<T>(acc);
            if constexpr (EVT::kEval) {
                if (ev.z)
                    acc2[0] += actf(fmaf(sv, k2.scale, k2.shift));
            } else {
                acc2[0] += sv;
                acc2[1] += sv * sv;
            }
        }
    }
    group_sum<2, TPP>(acc2, red);
    if (pl.active && lt == 0) {
        if constexpr (EVT::kEval) {
            if (ev.z)
                ev.z[pl.plane] = acc2[0] * ev.inv_hw;
        } else {
            a.psum[(size_t)pl.c * N + pl.n] = acc2[0];
            a.psq[(size_t)pl.c * N + pl.n] = acc2[1];
        }
    }
}

size_t dw_fwd_lds_bytes(const DwShape &s)
{
    const int tpp = pick_tpp(s.H * s.W);
    const int block = tpp > 256 ? tpp : 256;
    const int ppb = block / tpp;
    const int p = (s.k - 1) / 2;
    return sizeof(float) * ((size_t)ppb * (s.H + 2 * p) * (s.W + 2 * p) + (block / 64) * 2);
}

template <typename T, int K, int S, typename EVT>
static hipError_t dw_fwd_tpp(const DwFwdDev &a, hipStream_t st, EVT ev)
{
    const DwShape &s = a.s;
    const int tpp = pick_tpp(s.H * s.W);
    const size_t lds = dw_fwd_lds_bytes(s);
    const size_t planes = (size_t)s.N * s.C;
#define MBK_LAUNCH(TPP)                                                                           \
    {                                                                                             \
        constexpr int BLOCK = TPP > 256 ? TPP : 256;                                              \
        auto kern = dw_fwd_kernel<T, K, S, TPP, EVT>;                                             \
        hipError_t e = hipFuncSetAttribute((const void *)kern,                                    \
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
        if (e != hipSuccess)                                                                      \
            return e;                                                                             \
        const unsigned grid = (unsigned)((planes + BLOCK / TPP - 1) / (BLOCK / TPP));             \
        const unsigned extra = dw_eval_extra_blocks(ev, grid, BLOCK);                             \
        hipLaunchKernelGGL(kern, dim3(grid + extra), dim3(BLOCK), lds, st, a, ev);                \
        return hipGetLastError();                                                                 \
    }
    if (tpp == 64)
        MBK_LAUNCH(64)
    if (tpp == 256)
        MBK_LAUNCH(256)
    MBK_LAUNCH(1024)
#undef MBK_LAUNCH
}

template <typename T, typename EVT>
static hipError_t dw_fwd_ks(const DwFwdDev &a, hipStream_t st, const EVT &ev)
{
    const int k = a.s.k, s = a.s.s;
    if (k == 3 && s == 1)
        return dw_fwd_tpp<T, 3, 1>(a, st, ev);
    if (k == 3 && s == 2)
        return dw_fwd_tpp<T, 3, 2>(a, st, ev);
    if (k == 5 && s == 1)
        return dw_fwd_tpp<T, 5, 1>(a, st, ev);
    if (k == 5 && s == 2)
        return dw_fwd_tpp<T, 5, 2>(a, st, ev);
    return hipErrorInvalidValue;
}

// A consumer finalises a normalisation itself where its planes are large enough that the extra
// reduction per plane (overlapped with the plane's first loads) costs less than a launch.
static bool plane_finalize_pays(int HW) { return HW >= 1024; }

bool dw_fwd_finalizes_bn1(const DwShape &s, bool stores_a1)
{
    if (stores_a1)
        return false;
    if (dw4_supported(s)) // (launch_dw_fwd's order of preference)
        return plane_finalize_pays(s.H * s.W);
    return dwr_supported(s); // a wavefront per channel and image range: once per wavefront
}

__global__ __launch_bounds__(256) void dw_eval_coef_kernel(DwEval ev) { dw_eval_extra(ev, (int)blockIdx.x, 256); }

hipError_t launch_dw_eval_coef(DwEval &ev, hipStream_t st)
{
    const unsigned blocks = dw_eval_blocks(ev, 256);
    hipLaunchKernelGGL(dw_eval_coef_kernel, dim3(blocks), dim3(256), 0, st, ev);
    return hipGetLastError();
}

// A launch saved is some 4.5 us; the coefficients and the squeeze are about 130 cycles of every wavefront, 0.06 to 0.1 us
// per thousand of them, where instruction issue is the bound.  Evaluation of a block, with the launches / folded, us:
//  - nothing saved (a launch precedes the expansion conv anyway, no pool): 62 -> 186 -> 93 on 9x9, stride 2, 48 images
//    23.4 / 24.7, 77 -> 462 -> 77 on 6x6, 30 images 25.3 / 25.9;
//  - dw_fwd, a thread group to a plane, one launch saved: 48 -> 288 -> 48 on 25x25, 28 images (32 k wavefronts) 49.7 /
//    48.7, 111 121 / 126; 40 -> 240 -> 88 on 29x29, stride 2, 17 images (16 k) 33.8 / 32.5, 33 (32 k) 43.6 / 46.1; 61 -> 366
//    -> 76 on 17x17, stride 2, with SE, 8 images (12 k) 32.5 / 31.2, 64 (94 k) 74.1 / 78.8;
//  - the pool saved as well, which reads the output once more: with stride 1 folded is as fast or faster at any size
//    (25x25, 222 images 286 / 287; 57x57, 444 images 1484 / 1359); with stride 2 the output is a quarter (17x17, 672
//    channels, 24 images, 65 k, 66.1 / 64.5, 48, 129 k, 91.7 / 93.0, 95 158 / 167; 64 -> 384 -> 89 on 9x9, bf16, 164 images,
//    63 k, 143.6 / 146.6);
//  - dw4 and dw2, 5x5, fp32, planes of 1024 threads: 64 registers and more, which is one workgroup to a compute unit, not two, with
//    stride 2: 24 -> 144 -> 40 on 72x72, stride 2, 4 images (9 k) 36.6 / 30.8, 16 59.5 / 69.0, 64 162 / 201, 8 -> 48 -> 12 on
//    104x100 without SE, 17 images (13 k) 37.6 / 40.6; stride 1, 16
//    images (37 k) 90.8 / 84.9, 64 311 / 326, without SE 16 images 74.8 / 80.3; 42 -> 252 -> 40, a launch ahead, stride 2,
//    one image (4 k) 28.1 / 26.2, 3 39.2 / 40.4.
// dw_fwd with 1024 threads and 5x5: the folded form is the faster kernel (16 -> 96 -> 16 on 82x82, ReLU6, 61 images 310 / 251;
// 43 -> 31 on 69x69, stride 2, 64 images 74 / 57).  dw4, dw2 and dwr otherwise, where a wavefront has more pixels: folded is as fast or faster at every size measured.
bool dw_eval_folds(bool bf16, const DwShape &s, bool se, bool coef_ahead)
{
    const int saved = (se ? 1 : 0) + (coef_ahead ? 0 : 1);
    if (!saved)
        return false;
    const bool runs = dw4_supported(s) || dw2_supported(s); // (of four pixels)
    if (!runs && dwr_supported(s))
        return true;
    const int items = runs ? s.H * ((s.W + 3) / 4) : s.H * s.W; // and threads to a plane, as the launchers choose them
    const int threads = items <= 256 ? 64 : items <= (runs ? 1024 : 4096) ? 256 : 1024;
    const long long waves = (long long)s.N * s.C * (threads / 64);
    if (s.k == 5 && threads == 1024 && !runs)
        return true;
    if (!bf16 && s.k == 5 && threads == 1024)
        return waves <= (se && s.s == 1 ? 48 : coef_ahead ? 4 : 10) * 1024;
    return runs || (se && s.s == 1) || waves <= (saved == 2 ? 48 : 28) * 1024;
}

hipError_t launch_dw_fwd(bool bf16, const DwShape &s, const void *e, const float *bn1,
                         const void *w_dw, void *d, float *psum, float *psq, void *a1_store,
                         const BnFin *fin, const DwEval *ev, hipStream_t st)
{
    if (fin && !dw_fwd_finalizes_bn1(s, a1_store != nullptr))
        return hipErrorInvalidValue;
    if (!a1_store && dw4_supported(s))
        return launch_dw4_fwd(bf16, s, e, bn1, w_dw, d, psum, psq, fin, ev, st);
    if (!a1_store && dwr_supported(s))
        return launch_dwr_fwd(bf16, s, e, bn1, w_dw, d, psum, psq, fin, ev, st);
    if (!a1_store && dw2_supported(s))
        return launch_dw2_fwd(bf16, s, e, bn1, w_dw, d, psum, psq, ev, st);
    DwFwdDev a;
    a.s = s;
    a.divC = make_div((uint32_t)s.C);
    a.divWp = make_div((uint32_t)(s.W + 2 * s.p));
    a.divWo = make_div((uint32_t)s.Wo);
    a.e = e;
    a.bn1 = bn1;
    a.w = w_dw;
    a.d = d;
    a.psum = psum;
    a.psq = psq;
    a.a1_store = a1_store;
    if (ev)
        return bf16 ? dw_fwd_ks<bf16_t>(a, st, *ev) : dw_fwd_ks<float>(a, st, *ev);
    return bf16 ? dw_fwd_ks<bf16_t>(a, st, DwTrain()) : dw_fwd_ks<float>(a, st, DwTrain());
}

// ---- backward ---------------------------------------------------------------------------------

struct DwBwdDev {
    DwShape s;
    FastDiv divC, divWp, divWq, divWo, divW;
    FastDiv divWc0, divWc1; // stride 2: columns per parity class starting at column 0 / 1
    const void *G, *d, *e;
    const float *g, *dzs, *bn2, *coef2, *bn1;
    const void *w;
    const void *a1_saved;
    void *dy1_out;
    const void *res;
    float *pdw, *psb, *psr;
};

template <typename T, int K, int S, int TPP>
__global__ __launch_bounds__(TPP > 256 ? TPP : 256, (K == 3 && TPP == 1024) ? 8 : 1) void dw_bwd_kernel(DwBwdDev a)
{
    constexpr int P = (K - 1) / 2;
    constexpr int BLOCK = TPP > 256 ? TPP : 256;
    constexpr int PPB = BLOCK / TPP;
    constexpr int NV = K * K + 2;
    extern __shared__ float lds[];
    const int H = a.s.H, W = a.s.W, Ho = a.s.Ho, Wo = a.s.Wo, C = a.s.C, N = a.s.N;
    const int Hp = H + 2 * P, Wp = W + 2 * P;    // a1 tile, border P
    const int Hq = Ho + 2 * P, Wq = Wo + 2 * P;  // dd tile, border P
    const int lt = threadIdx.x % TPP, grp = threadIdx.x / TPP;
    float *a1t = lds + grp * (Hp * Wp + Hq * Wq);
    float *ddt = a1t + Hp * Wp;
    float *red = lds + PPB * (Hp * Wp + Hq * Wq);
    const PlaneId pl = plane_of_group<TPP>(N, C, a.divC);
    const bool bn = a.bn1 != nullptr;

    float w[K * K];
    float scale1 = 1.f, shift1 = 0.f, mean1 = 0.f, rstd1 = 0.f;
    if (pl.active) {
#pragma unroll
        for (int t = 0; t < K * K; ++t)
            w[t] = ld<T>((const T *)a.w, (size_t)pl.c * K * K + t);
        if (bn) {
            scale1 = a.bn1[pl.c];
            shift1 = a.bn1[C + pl.c];
            mean1 = a.bn1[2 * C + pl.c];
            rstd1 = a.bn1[3 * C + pl.c];
        }
        // depthwise input a1 with a zero border
        const size_t ebase = pl.plane * (size_t)H * W;
        for (int idx = lt; idx < Hp * Wp; idx += TPP) {
            const int hp = (int)fdiv((uint32_t)idx, a.divWp);
            const int wp = idx - hp * Wp;
            const int h = hp - P, x = wp - P;
            float v = 0.f;
            if (h >= 0 && h < H && x >= 0 && x < W) {
                if (a.a1_saved) {
                    v = ld<T>((const T *)a.a1_saved, ebase + (size_t)h * W + x);
                } else {
                    v = ld<T>((const T *)a.e, ebase + (size_t)h * W + x);
                    if (bn)
                        v = actf(fmaf(v, scale1, shift1));
                }
            }
            a1t[idx] = v;
        }
        // gradient w.r.t. the depthwise output, dd, with a zero border
        const float scale2 = a.bn2[pl.c], shift2 = a.bn2[C + pl.c];
        const float c0 = a.coef2[pl.c], c1 = a.coef2[C + pl.c], c2 = a.coef2[2 * C + pl.c];
        const float gate = a.g[pl.plane], dzs = a.dzs[pl.plane];
        const size_t dbase = pl.plane * (size_t)Ho * Wo;
        for (int idx = lt; idx < Hq * Wq; idx += TPP) {
            const int ip = (int)fdiv((uint32_t)idx, a.divWq);
            const int jp = idx - ip * Wq;
            const int i = ip - P, j = jp - P;
            float v = 0.f;
            if (i >= 0 && i < Ho && j >= 0 && j < Wo) {
                const float Gv = ld<T>((const T *)a.G, dbase + (size_t)i * Wo + j);
                const float dv = ld<T>((const T *)a.d, dbase + (size_t)i * Wo + j);
                float val, grad;
                act_both(fmaf(dv, scale2, shift2), val, grad);
                const float dy2 = fmaf(Gv, gate, dzs) * grad;
                v = fmaf(c0, dy2, fmaf(c1, dv, c2));
            }
            ddt[idx] = v;
        }
    }
    __syncthreads();

    float acc[NV];
#pragma unroll
    for (int t = 0; t < NV; ++t)
        acc[t] = 0.f;
    if (pl.active) {
        // filter gradient: dw[u,v] += dd[i,j] * a1[i*S+u-P, j*S+v-P]
        for (int idx = lt; idx < Ho * Wo; idx += TPP) {
            const int i = (int)fdiv((uint32_t)idx, a.divWo);
            const int j = idx - i * Wo;
            const float ddv = ddt[(i + P) * Wq + j + P];
            const float *t0 = a1t + (i * S) * Wp + j * S;
#pragma unroll
            for (int u = 0; u < K; ++u)
#pragma unroll
                for (int v = 0; v < K; ++v)
                    acc[u * K + v] = fmaf(ddv, t0[u * Wp + v], acc[u * K + v]);
        }
        // input gradient: da1[h,x] = sum_{u,v} w[u,v]*dd[(h+P-u)/S, (x+P-v)/S] over the taps
        // for which both quotients are exact; in border coordinates the row is
        // (h+P-u+S*P)/S, always non-negative.
        const size_t ebase = pl.plane * (size_t)H * W;
        auto finish = [&](int idx, float da) { // Swish', store, BN1 partial sums
            if (bn) {
                const float raw = ld<T>((const T *)a.e, ebase + idx);
                float val, grad;
                act_both(fmaf(raw, scale1, shift1), val, grad);
                const float dy1 = da * grad;
                st<T>((T *)a.dy1_out, ebase + idx, dy1);
                const float sv = as_stored<T>(dy1);
                acc[K * K] += sv;
                acc[K * K + 1] = fmaf(sv, (raw - mean1) * rstd1, acc[K * K + 1]);
            } else {
                if (a.res)
                    da += ld<T>((const T *)a.res, ebase + idx);
                st<T>((T *)a.dy1_out, ebase + idx, da);
            }
        };
        if (S == 1) {
            for (int idx = lt; idx < H * W; idx += TPP) {
                const int h = (int)fdiv((uint32_t)idx, a.divW);
                const int x = idx - h * W;
                float da = 0.f;
#pragma unroll
                for (int u = 0; u < K; ++u)
#pragma unroll
                    for (int v = 0; v < K; ++v)
                        da = fmaf(w[u * K + v], ddt[(h + 2 * P - u) * Wq + x + 2 * P - v], da);
                finish(idx, da);
            }
        } else {
            // stride 2: an input pixel only meets the taps u = ph (mod 2), v = pw (mod 2) with
            // ph = (h+P)&1, pw = (x+P)&1.  The four parity classes are walked one after the
            // other so that the tap set, and hence the weight registers, are compile-time.
#pragma unroll
            for (int ph = 0; ph < 2; ++ph)
#pragma unroll
                for (int pw = 0; pw < 2; ++pw) {
                    const int hs = ph ^ (P & 1), xs = pw ^ (P & 1); // first row / column of the class
                    const int Hc = (H - hs + 1) >> 1, Wc = (W - xs + 1) >> 1;
                    const FastDiv dv = xs ? a.divWc1 : a.divWc0;
                    for (int idx = lt; idx < Hc * Wc; idx += TPP) {
                        const int hh = (int)fdiv((uint32_t)idx, dv);
                        const int h = hs + 2 * hh, x = xs + 2 * (idx - hh * Wc);
                        const int r0 = ((h + P - ph) >> 1) + P, c0 = ((x + P - pw) >> 1) + P;
                        float da = 0.f;
#pragma unroll
                        for (int ua = 0; ph + 2 * ua < K; ++ua)
#pragma unroll
                            for (int vb = 0; pw + 2 * vb < K; ++vb)
                                da = fmaf(w[(ph + 2 * ua) * K + pw + 2 * vb],
                                          ddt[(r0 - ua) * Wq + c0 - vb], da);
                        finish(h * W + x, da);
                    }
                }
        }
    }
    group_sum<NV, TPP>(acc, red);
    if (pl.active && lt == 0) {
        float *dst = a.pdw + ((size_t)pl.c * N + pl.n) * (K * K);
#pragma unroll
        for (int t = 0; t < K * K; ++t)
            dst[t] = acc[t];
        if (bn) {
            a.psb[(size_t)pl.c * N + pl.n] = acc[K * K];
            a.psr[(size_t)pl.c * N + pl.n] = acc[K * K + 1];
        }
    }
}

size_t dw_bwd_lds_bytes(const DwShape &s)
{
    const int tpp = pick_tpp(s.H * s.W);
    const int block = tpp > 256 ? tpp : 256;
    const int ppb = block / tpp;
    const int p = (s.k - 1) / 2;
    const size_t per = (size_t)(s.H + 2 * p) * (s.W + 2 * p) + (size_t)(s.Ho + 2 * p) * (s.Wo + 2 * p);
    return sizeof(float) * (ppb * per + (size_t)(block / 64) * (s.k * s.k + 2));
}

template <typename T, int K, int S>
static hipError_t dw_bwd_tpp(const DwBwdDev &a, hipStream_t st)
{
    const DwShape &s = a.s;
    const int tpp = pick_tpp(s.H * s.W);
    const size_t lds = dw_bwd_lds_bytes(s);
    const size_t planes = (size_t)s.N * s.C;
#define MBK_LAUNCH(TPP)                                                                           \
    {                                                                                             \
        constexpr int BLOCK = TPP > 256 ? TPP : 256;                                              \
        auto kern = dw_bwd_kernel<T, K, S, TPP>;                                                  \
        hipError_t e = hipFuncSetAttribute((const void *)kern,                                    \
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
        if (e != hipSuccess)                                                                      \
            return e;                                                                             \
        const unsigned grid = (unsigned)((planes + BLOCK / TPP - 1) / (BLOCK / TPP));             \
        hipLaunchKernelGGL(kern, dim3(grid), dim3(BLOCK), lds, st, a);                            \
        return hipGetLastError();                                                                 \
    }
    if (tpp == 64)
        MBK_LAUNCH(64)
    if (tpp == 256)
        MBK_LAUNCH(256)
    MBK_LAUNCH(1024)
#undef MBK_LAUNCH
}

template <typename T>
static hipError_t dw_bwd_ks(const DwBwdDev &a, hipStream_t st)
{
    const int k = a.s.k, s = a.s.s;
    if (k == 3 && s == 1)
        return dw_bwd_tpp<T, 3, 1>(a, st);
    if (k == 3 && s == 2)
        return dw_bwd_tpp<T, 3, 2>(a, st);
    if (k == 5 && s == 1)
        return dw_bwd_tpp<T, 5, 1>(a, st);
    if (k == 5 && s == 2)
        return dw_bwd_tpp<T, 5, 2>(a, st);
    return hipErrorInvalidValue;
}

hipError_t launch_dw_bwd(bool bf16, const DwBwdArgs &h, hipStream_t st)
{
    if (!h.a1_saved && dw4_supported(h.s))
        return launch_dw4_bwd(bf16, h, st);
    if (!h.a1_saved && dwr_supported(h.s))
        return launch_dwr_bwd(bf16, h, st);
    if (!h.a1_saved && !h.res && dw2_supported(h.s))
        return launch_dw2_bwd(bf16, h, st);
    DwBwdDev a;
    a.s = h.s;
    const int p = h.s.p;
    a.divC = make_div((uint32_t)h.s.C);
    a.divWp = make_div((uint32_t)(h.s.W + 2 * p));
    a.divWq = make_div((uint32_t)(h.s.Wo + 2 * p));
    a.divWo = make_div((uint32_t)h.s.Wo);
    a.divW = make_div((uint32_t)h.s.W);
    a.divWc0 = make_div((uint32_t)std::max(1, (h.s.W + 1) / 2));
    a.divWc1 = make_div((uint32_t)std::max(1, h.s.W / 2));
    a.G = h.G;
    a.d = h.d;
    a.e = h.e;
    a.g = h.g;
    a.dzs = h.dzs;
    a.bn2 = h.bn2;
    a.coef2 = h.coef2;
    a.bn1 = h.bn1;
    a.w = h.w_dw;
    a.a1_saved = h.a1_saved;
    a.dy1_out = h.dy1_out;
    a.res = h.res;
    a.pdw = h.pdw;
    a.psb = h.psb;
    a.psr = h.psr;
    return bf16 ? dw_bwd_ks<bf16_t>(a, st) : dw_bwd_ks<float>(a, st);
}

// ---- per-plane reductions and the final elementwise pass --------------------------------------

struct PlaneArgs {
    int N, C, HW;
    FastDiv divC;
    const void *t0, *t1;
    const float *bn; // {scale, shift, mean, rstd}[C]
    float *o0, *o1, *o2;
    int layoutCN; // 1: outputs indexed [c][n]; 0: [n][c]
    float o0_scale; // multiplies the first output (1/HW turns a plane sum into a mean)
    void *out;    // elementwise output (bn_apply)
    const void *res;
    BnFin fin;    // pool and bn_apply, fin.psum non-null: `bn` is derived there from the partial sums
    X3PrepArgs prep; // weight images that the workgroups past the planes' write (channel form of the pool)
};

// Four consecutive elements at once (16 bytes per lane for fp32, 8 for bf16).
template <typename T>
__device__ __forceinline__ void ldvec4(const T *p, size_t i, float (&v)[4]);
template <>
__device__ __forceinline__ void ldvec4<float>(const float *p, size_t i, float (&v)[4])
{
    const float4 t = *reinterpret_cast<const float4 *>(p + i);
    v[0] = t.x;
    v[1] = t.y;
    v[2] = t.z;
    v[3] = t.w;
}
template <>
__device__ __forceinline__ void ldvec4<bf16_t>(const bf16_t *p, size_t i, float (&v)[4])
{
    const uint2 t = *reinterpret_cast<const uint2 *>(&p[i]);
    v[0] = bf16_bits_to_float(t.x & 0xffffu);
    v[1] = bf16_bits_to_float(t.x >> 16);
    v[2] = bf16_bits_to_float(t.y & 0xffffu);
    v[3] = bf16_bits_to_float(t.y >> 16);
}
template <typename T>
__device__ __forceinline__ void stvec4(T *p, size_t i, const float (&v)[4]);
template <>
__device__ __forceinline__ void stvec4<float>(float *p, size_t i, const float (&v)[4])
{
    *reinterpret_cast<float4 *>(p + i) = make_float4(v[0], v[1], v[2], v[3]);
}
template <>
__device__ __forceinline__ void stvec4<bf16_t>(bf16_t *p, size_t i, const float (&v)[4])
{
    uint2 t;
    t.x = bf16_pack2(v[0], v[1]);
    t.y = bf16_pack2(v[2], v[3]);
    *reinterpret_cast<uint2 *>(&p[i]) = t;
}

// z = mean swish(y), s3 = sum swish'(y), s4 = sum swish'(y)*xhat, y = BN(t0)
struct OpPool {
    static constexpr int NV = 3;
    static constexpr bool kTwo = false;
    static __device__ __forceinline__ void eval(float v, float, float sc, float sh, float mu,
                                                float rs, float (&acc)[NV])
    {
        float val, grad;
        act_both(fmaf(v, sc, sh), val, grad);
        acc[0] += val;
        acc[1] += grad;
        acc[2] = fmaf(grad, (v - mu) * rs, acc[2]);
    }
};
// sums of dy (t0) and dy*xhat(t1)
struct OpDot {
    static constexpr int NV = 2;
    static constexpr bool kTwo = true;
    static __device__ __forceinline__ void eval(float dy, float raw, float, float, float mu,
                                                float rs, float (&acc)[NV])
    {
        acc[0] += dy;
        acc[1] = fmaf(dy, (raw - mu) * rs, acc[1]);
    }
};
// G (t0) against a2, swish'(y2), swish'(y2)*dhat rebuilt from d (t1)
struct OpGate {
    static constexpr int NV = 3;
    static constexpr bool kTwo = true;
    static __device__ __forceinline__ void eval(float Gv, float v, float sc, float sh, float mu,
                                                float rs, float (&acc)[NV])
    {
        float val, grad;
        act_both(fmaf(v, sc, sh), val, grad);
        acc[0] = fmaf(Gv, val, acc[0]);
        acc[1] = fmaf(Gv, grad, acc[1]);
        acc[2] = fmaf(Gv * grad, (v - mu) * rs, acc[2]);
    }
};

template <typename T, int TPP, typename OP>
__global__ __launch_bounds__(TPP > 256 ? TPP : 256) void plane_reduce_kernel(PlaneArgs a)
{
    constexpr int BLOCK = TPP > 256 ? TPP : 256;
    __shared__ float red[(BLOCK / 64) * OP::NV];
    const int lt = threadIdx.x % TPP;
    const PlaneId pl = plane_of_group<TPP>(a.N, a.C, a.divC);
    float acc[OP::NV];
#pragma unroll
    for (int t = 0; t < OP::NV; ++t)
        acc[t] = 0.f;
    if (pl.active) {
        const float sc = a.bn[pl.c], sh = a.bn[a.C + pl.c];
        const float mu = a.bn[2 * a.C + pl.c], rs = a.bn[3 * a.C + pl.c];
        const size_t base = pl.plane * (size_t)a.HW;
        // Four strides of the plane per round: all loads of a round are issued before any of
        // them is consumed (the scheduler fence keeps the compiler from pairing each load with
        // its arithmetic, which would cost one memory round trip per stride).
        if ((a.HW & 3) == 0) {
            float v0[4][4], v1[4][4];
            const auto load_round = [&](int idx0) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int idx = idx0 + 4 * TPP * u;
                    // past the end: reread an element of the plane, masked when consumed
                    const int ic = idx < a.HW ? idx : (idx0 < a.HW ? idx0 : 0);
                    ldvec4<T>((const T *)a.t0, base + ic, v0[u]);
                    if (OP::kTwo)
                        ldvec4<T>((const T *)a.t1, base + ic, v1[u]);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            int idx0 = 4 * lt;
            load_round(idx0);
            while (true) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (idx0 + 4 * TPP * u < a.HW) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            OP::eval(v0[u][r], OP::kTwo ? v1[u][r] : 0.f, sc, sh, mu, rs, acc);
                    }
                }
                idx0 += 16 * TPP;
                if (idx0 >= a.HW)
                    break;
                load_round(idx0);
            }
        } else {
            for (int idx0 = lt; idx0 < a.HW; idx0 += 4 * TPP) {
                float v0[4], v1[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int idx = idx0 + TPP * u;
                    const int ic = idx < a.HW ? idx : idx0;
                    v0[u] = ld<T>((const T *)a.t0, base + ic);
                    v1[u] = OP::kTwo ? ld<T>((const T *)a.t1, base + ic) : 0.f;
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (idx0 + TPP * u < a.HW)
                        OP::eval(v0[u], v1[u], sc, sh, mu, rs, acc);
            }
        }
    }
    group_sum<OP::NV, TPP>(acc, red);
    if (pl.active && lt == 0) {
        const size_t o = a.layoutCN ? (size_t)pl.c * a.N + pl.n : pl.plane;
        float *outs[3] = {a.o0, a.o1, a.o2};
#pragma unroll
        for (int t = 0; t < OP::NV; ++t)
            outs[t][o] = t == 0 ? acc[t] * a.o0_scale : acc[t];
    }
}

// The pool of small planes with BN2's finalise step: a workgroup works on one channel, on the planes of
// `rounds` x 256/TPP consecutive images.  Its first wavefront finalises (all four would put more
// instructions into the sum than the pool itself has: 64 x 1152 planes of 7x7 13.7 us, now 10.8; the
// finalise launch and the pool without it took 5.4 + 6.3); the
// first planes are requested before.  The workgroups ahead of the planes' write the weight images of
// convolutions later in the sequence.
template <typename T, int TPP>
__global__ __launch_bounds__(256) void pool_chan_kernel(PlaneArgs a, int rounds, int per)
{
    constexpr int PPB = 256 / TPP;
    __shared__ float cf[4];
    if ((int)blockIdx.x < a.prep.tiles) {
        x3_prep_tile(a.prep, blockIdx.x, threadIdx.x);
        return;
    }
    // per: workgroups of a channel.  Neighbouring channels go to one XCD (blockIdx.x mod 8): their results
    // lie next to each other, and a line written from several L2s costs a partial write each.
    const int total = a.C * per, i = blockIdx.x - a.prep.tiles;
    const int b = (i & 7) * ((total + 7) >> 3) + (i >> 3), c = b / per, part = b - c * per;
    if (b >= total)
        return;
    const int lt = threadIdx.x % TPP;
    BnFinRegs fr;
    if (threadIdx.x < 64)
        bn_fin_issue<64>(a.fin, c, threadIdx.x, fr);
    float sc, sh, mu, rs;
    const auto coefs = [&]() {
        if (threadIdx.x < 64) {
            bn_fin_finish<64>(a.fin, a.C, c, threadIdx.x, part == 0, nullptr, fr, sc, sh, mu, rs);
            if (threadIdx.x == 0) {
                cf[0] = sc;
                cf[1] = sh;
                cf[2] = mu;
                cf[3] = rs;
            }
        }
        __syncthreads();
        sc = cf[0];
        sh = cf[1];
        mu = cf[2];
        rs = cf[3];
    };
    int n = part * rounds * PPB + threadIdx.x / TPP;
    for (int r = 0; r < rounds; ++r, n += PPB) {
        const size_t plane = (size_t)(n < a.N ? n : 0) * a.C + c, base = plane * a.HW;
        float acc[3] = {0.f, 0.f, 0.f};
        if ((a.HW & 3) == 0) { // at most 16 * TPP elements
            float v[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int idx = 4 * (lt + TPP * u);
                ldvec4<T>((const T *)a.t0, base + (idx < a.HW ? idx : 0), v[u]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (r == 0)
                coefs();
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (4 * (lt + TPP * u) < a.HW) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        OpPool::eval(v[u][j], 0.f, sc, sh, mu, rs, acc);
                }
        } else {
            for (int idx0 = lt; idx0 - lt < a.HW; idx0 += 4 * TPP) { // (equally often in all threads)
                float v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int idx = idx0 + TPP * u;
                    v[u] = ld<T>((const T *)a.t0, base + (idx < a.HW ? idx : 0));
                }
                __builtin_amdgcn_sched_barrier(0);
                if (r == 0 && idx0 == lt)
                    coefs();
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (idx0 + TPP * u < a.HW)
                        OpPool::eval(v[u], 0.f, sc, sh, mu, rs, acc);
            }
        }
        group_sum<3, TPP>(acc, nullptr);
        if (n < a.N && lt == 0) {
            a.o0[plane] = acc[0] * a.o0_scale;
            a.o1[plane] = acc[1];
            a.o2[plane] = acc[2];
        }
    }
}

// CHAN (planes of at most 1024 elements, training): the workgroup's planes belong to one channel, whose
// BN3 it finalises first; the launch that did it before took 4.7 us in front of one of 5.
template <typename T, int TPP, bool CHAN>
__global__ __launch_bounds__(TPP > 256 ? TPP : 256) void bn_apply_kernel(PlaneArgs a)
{
    constexpr int BLOCK = TPP > 256 ? TPP : 256;
    __shared__ double redd[2 * (BLOCK / 64)];
    const int lt = threadIdx.x % TPP;
    const PlaneId pl = plane_of_group<TPP, CHAN>(a.N, a.C, a.divC);
    if (!CHAN && !pl.active) // (TPP > 64: one plane per workgroup, always active)
        return;
    // the threads that finalise together: the plane's, or with CHAN the workgroup
    constexpr int FIN = CHAN || TPP < 64 ? 256 : TPP;
    const bool fin = CHAN || (TPP > 64 && a.fin.psum);
    float sc, sh;
    BnFinRegs fr;
    if (fin) {
        bn_fin_issue<FIN>(a.fin, pl.c, CHAN ? (int)threadIdx.x : lt, fr);
    } else {
        sc = a.bn[pl.c];
        sh = a.bn[a.C + pl.c];
    }
    __builtin_amdgcn_sched_barrier(0);
    const auto coefs = [&]() {
        float mu, rs;
        if constexpr (CHAN || TPP > 64) {
            const bool writer =
                CHAN ? blockIdx.x % ((a.N + BLOCK / TPP - 1) / (BLOCK / TPP)) == 0 : pl.n == 0;
            if (fin)
                bn_fin_finish<FIN>(a.fin, a.C, pl.c, CHAN ? (int)threadIdx.x : lt, writer, redd, fr, sc, sh, mu, rs);
        }
    };
    const size_t base = pl.plane * (size_t)a.HW;
    if ((a.HW & 3) == 0) {
        // (coefficient requests in front of the first round's loads, as in plane_reduce_kernel)
        float v[4][4], rr[4][4];
        const auto load_round = [&](int idx0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int idx = idx0 + 4 * TPP * u;
                const int ic = idx < a.HW ? idx : (idx0 < a.HW ? idx0 : 0);
                ldvec4<T>((const T *)a.t0, base + ic, v[u]);
                if (a.res)
                    ldvec4<T>((const T *)a.res, base + ic, rr[u]);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        int idx0 = 4 * lt;
        load_round(idx0);
        coefs();
        __builtin_amdgcn_sched_barrier(0);
        if (CHAN && !pl.active)
            return;
        while (true) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int idx = idx0 + 4 * TPP * u;
                if (idx < a.HW) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        v[u][r] = fmaf(v[u][r], sc, sh);
                        if (a.res)
                            v[u][r] += rr[u][r];
                    }
                    stvec4<T>((T *)a.out, base + idx, v[u]);
                }
            }
            idx0 += 16 * TPP;
            if (idx0 >= a.HW)
                break;
            load_round(idx0);
        }
    } else {
        coefs();
        if (CHAN && !pl.active)
            return;
        for (int idx = lt; idx < a.HW; idx += TPP) {
            float v = fmaf(ld<T>((const T *)a.t0, base + idx), sc, sh);
            if (a.res)
                v += ld<T>((const T *)a.res, base + idx);
            st<T>((T *)a.out, base + idx, v);
        }
    }
}

// BN3's backward reductions and their finalise step in one launch: a workgroup owns a channel, TPP
// lanes a plane.  The planes' sums are added over the workgroup in fp64, in a fixed order, and one
// thread turns them into dgamma, dbeta and the coefficients {c0, c1, c2}.  Latency is all it costs:
// 64 x 320 planes of 7x7 5.9 us, 4.8 + 4.7 as two launches.
template <typename T, int TPP>
__global__ __launch_bounds__(1024) void bn_bwd_chan_kernel(PlaneArgs a, BnBwdFin f)
{
    constexpr int G = 1024 / TPP; // planes in flight
    __shared__ double red[2][16];
    const int c = blockIdx.x, lt = threadIdx.x % TPP;
    const float gm = f.gamma[c], mu = a.bn[2 * a.C + c], rs = a.bn[3 * a.C + c];
    double sb = 0.0, sr = 0.0;
    for (int n = threadIdx.x / TPP; n < a.N; n += G) {
        const size_t base = ((size_t)n * a.C + c) * a.HW;
        float acc[2] = {0.f, 0.f};
        if ((a.HW & 3) == 0) { // at most 16 * TPP elements: one round
            float v0[4][4], v1[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int idx = 4 * (lt + TPP * u), ic = idx < a.HW ? idx : 0;
                ldvec4<T>((const T *)a.t0, base + ic, v0[u]);
                ldvec4<T>((const T *)a.t1, base + ic, v1[u]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (4 * (lt + TPP * u) < a.HW) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        OpDot::eval(v0[u][r], v1[u][r], 0.f, 0.f, mu, rs, acc);
                }
        } else {
            for (int idx0 = lt; idx0 < a.HW; idx0 += 4 * TPP) {
                float v0[4], v1[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int ic = idx0 + TPP * u < a.HW ? idx0 + TPP * u : idx0;
                    v0[u] = ld<T>((const T *)a.t0, base + ic);
                    v1[u] = ld<T>((const T *)a.t1, base + ic);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (idx0 + TPP * u < a.HW)
                        OpDot::eval(v0[u], v1[u], 0.f, 0.f, mu, rs, acc);
            }
        }
        sb += (double)acc[0];
        sr += (double)acc[1];
    }
    sb = wave_sum_d(sb);
    sr = wave_sum_d(sr);
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = sb;
        red[1][threadIdx.x >> 6] = sr;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        sb = sr = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            sb += red[0][w];
            sr += red[1][w];
        }
        f.dbeta[c] = (float)sb;
        f.dgamma[c] = (float)sr;
        bn_bwd_coef_vals(a.C, c, f.inv_m, sr, sb, gm, mu, rs, f.coef);
    }
}

template <typename T, typename OP>
static hipError_t plane_reduce_launch(const PlaneArgs &a, hipStream_t st)
{
    const int tpp = pick_tpp_plane(a.HW);
    const size_t planes = (size_t)a.N * a.C;
#define MBK_LAUNCH(TPP)                                                                           \
    {                                                                                             \
        constexpr int BLOCK = TPP > 256 ? TPP : 256;                                              \
        const unsigned grid = (unsigned)((planes + BLOCK / TPP - 1) / (BLOCK / TPP));             \
        hipLaunchKernelGGL((plane_reduce_kernel<T, TPP, OP>), dim3(grid), dim3(BLOCK), 0, st, a); \
        return hipGetLastError();                                                                 \
    }
    if (tpp == 16)
        MBK_LAUNCH(16)
    if (tpp == 64)
        MBK_LAUNCH(64)
    if (tpp == 256)
        MBK_LAUNCH(256)
    MBK_LAUNCH(1024)
#undef MBK_LAUNCH
}

static PlaneArgs plane_args(int N, int C, int HW, const void *t0, const void *t1, const float *bn)
{
    PlaneArgs a = {};
    a.N = N;
    a.C = C;
    a.HW = HW;
    a.divC = make_div((uint32_t)C);
    a.t0 = t0;
    a.t1 = t1;
    a.bn = bn;
    a.o0_scale = 1.f;
    return a;
}

// Small planes (16 or 64 lanes each): the pool finalises BN2's statistics itself, a channel's planes to
// a workgroup, in at most two rounds of images.  Larger planes have workgroups of their own and would
// repeat the sum for each of them; there the finalise step is a launch, and so it is where there are
// more workgroups than a round and a half of eight per compute unit: the workgroups of the following
// rounds wait for their coefficients again, or with four rounds of images each have too few loads in
// flight (with / without the step inside, one forward pass: 384 channels, 256 images of 12x12 105.9 /
// 106.9 us, 512 of 14x14 258.7 / 254.1; 96 channels, 2048 of 17x17 826 / 794).
static long long pool_chan_groups(int N, int C, int HW, int rounds)
{
    const int per = rounds * (256 / pick_tpp_plane(HW));
    return (long long)C * ((N + per - 1) / per);
}
bool plane_channel_form(int N, int C, int HW) { return HW <= 1024 && pool_chan_groups(N, C, HW, 2) <= 3 * 1024; }

hipError_t launch_pool(bool bf16, int N, int C, int HW, const void *d, const float *bn2, float *z,
                       float *s3, float *s4, const BnFin *fin, const X3PrepArgs *prep, hipStream_t st)
{
    PlaneArgs a = plane_args(N, C, HW, d, nullptr, bn2);
    a.o0 = z;
    a.o1 = s3;
    a.o2 = s4;
    a.layoutCN = 0;
    a.o0_scale = 1.f / (float)HW;
    if (fin) {
        a.fin = *fin;
        if (prep)
            a.prep = *prep;
        // images per workgroup: two rounds where that leaves eight workgroups per compute unit
        const int ppb = 256 / pick_tpp_plane(HW);
        const int rounds = pool_chan_groups(N, C, HW, 2) >= 2048 ? 2 : 1;
        const int per = (N + rounds * ppb - 1) / (rounds * ppb);
        const dim3 grid((unsigned)((C * per + 7) / 8 * 8 + a.prep.tiles));
        if (ppb == 16 && bf16)
            hipLaunchKernelGGL((pool_chan_kernel<bf16_t, 16>), grid, dim3(256), 0, st, a, rounds, per);
        else if (ppb == 16)
            hipLaunchKernelGGL((pool_chan_kernel<float, 16>), grid, dim3(256), 0, st, a, rounds, per);
        else if (bf16)
            hipLaunchKernelGGL((pool_chan_kernel<bf16_t, 64>), grid, dim3(256), 0, st, a, rounds, per);
        else
            hipLaunchKernelGGL((pool_chan_kernel<float, 64>), grid, dim3(256), 0, st, a, rounds, per);
        return hipGetLastError();
    }
    return bf16 ? plane_reduce_launch<bf16_t, OpPool>(a, st) : plane_reduce_launch<float, OpPool>(a, st);
}

// A workgroup per channel reads 2*N*HW elements: with more than two planes to a thread group it
// would take longer than the launch that it saves.
bool bn_bwd_chan_supported(int N, int HW)
{
    return HW <= 1024 && N <= 2 * 1024 / pick_tpp_plane(HW);
}

hipError_t launch_bn_bwd_chan(bool bf16, int N, int C, int HW, const void *dy, const void *raw, const float *bn,
                              const BnBwdFin &f, hipStream_t st)
{
    const PlaneArgs a = plane_args(N, C, HW, dy, raw, bn);
    if (pick_tpp_plane(HW) == 16) {
        if (bf16)
            hipLaunchKernelGGL((bn_bwd_chan_kernel<bf16_t, 16>), dim3((unsigned)C), dim3(1024), 0, st, a, f);
        else
            hipLaunchKernelGGL((bn_bwd_chan_kernel<float, 16>), dim3((unsigned)C), dim3(1024), 0, st, a, f);
    } else {
        if (bf16)
            hipLaunchKernelGGL((bn_bwd_chan_kernel<bf16_t, 64>), dim3((unsigned)C), dim3(1024), 0, st, a, f);
        else
            hipLaunchKernelGGL((bn_bwd_chan_kernel<float, 64>), dim3((unsigned)C), dim3(1024), 0, st, a, f);
    }
    return hipGetLastError();
}

hipError_t launch_plane_dot(bool bf16, int N, int C, int HW, const void *dy, const void *raw,
                            const float *bn, float *psb, float *psr, hipStream_t st)
{
    PlaneArgs a = plane_args(N, C, HW, dy, raw, bn);
    a.o0 = psb;
    a.o1 = psr;
    a.layoutCN = 1;
    return bf16 ? plane_reduce_launch<bf16_t, OpDot>(a, st) : plane_reduce_launch<float, OpDot>(a, st);
}

hipError_t launch_gate_sums(bool bf16, int N, int C, int HW, const void *G, const void *d,
                            const float *bn2, float *dg, float *A1, float *A2, hipStream_t st)
{
    PlaneArgs a = plane_args(N, C, HW, G, d, bn2);
    a.o0 = dg;
    a.o1 = A1;
    a.o2 = A2;
    a.layoutCN = 0;
    return bf16 ? plane_reduce_launch<bf16_t, OpGate>(a, st) : plane_reduce_launch<float, OpGate>(a, st);
}

// Every workgroup that finalises BN3 reads all of its channel's partial sums (one per 32 pixels of the
// whole batch behind conv_xk), so the repeated reads grow with the square of the batch, the launch they
// save does not.  Up to two and a half rounds of eight workgroups per compute unit they are hidden
// (with / without the step inside, one forward pass of a block with Cout channels: 112, 64 images of
// 17x17 78.3 / 80.3 us; 40, 128 images of 112x112 987 / 1014), beyond that they are not (112, 512 of
// 17x17 492 / 474; 64, 1024 of 24x24 437 / 364; 112, 256 of 56x56 1728 / 1514).
bool bn_apply_finalizes(int N, int C, int HW)
{
    const int tpp = pick_tpp_plane(HW), ppb = tpp < 256 ? 256 / tpp : 1;
    return (long long)C * ((N + ppb - 1) / ppb) <= 5 * 1024;
}

hipError_t launch_bn_apply(bool bf16, int N, int C, int HW, const void *p, const float *bn3,
                           const void *res, void *out, const BnFin *fin, hipStream_t st)
{
    PlaneArgs a = plane_args(N, C, HW, p, nullptr, bn3);
    if (fin)
        a.fin = *fin;
    a.out = out;
    a.res = res;
    const int tpp = pick_tpp_plane(HW);
    const size_t planes = (size_t)N * C;
#define MBK_LAUNCH(TPP, CHAN)                                                                     \
    {                                                                                             \
        constexpr int BLOCK = TPP > 256 ? TPP : 256, PPB = BLOCK / TPP;                           \
        const unsigned grid = (unsigned)(CHAN ? (size_t)C * ((N + PPB - 1) / PPB) : (planes + PPB - 1) / PPB); \
        if (bf16)                                                                                 \
            hipLaunchKernelGGL((bn_apply_kernel<bf16_t, TPP, CHAN>), dim3(grid), dim3(BLOCK), 0, st, a);       \
        else                                                                                      \
            hipLaunchKernelGGL((bn_apply_kernel<float, TPP, CHAN>), dim3(grid), dim3(BLOCK), 0, st, a);        \
        return hipGetLastError();                                                                 \
    }
    if (fin && tpp == 16)
        MBK_LAUNCH(16, true)
    if (fin && tpp == 64)
        MBK_LAUNCH(64, true)
    if (tpp == 16)
        MBK_LAUNCH(16, false)
    if (tpp == 64)
        MBK_LAUNCH(64, false)
    if (tpp == 256)
        MBK_LAUNCH(256, false)
    MBK_LAUNCH(1024, false)
#undef MBK_LAUNCH
}

} // namespace mbk
