// fp32 1x1 convolutions and weight gradients of the wide blocks on the bf16 matrix cores.
//
// An fp32 MFMA (v_mfma_f32_32x32x2_f32) runs at the rate of the vector ALU and blocks it; the
// bf16 MFMA (v_mfma_f32_32x32x16_bf16) does sixteen times the work per cycle and runs beside
// the vector ALU.  An fp32 value is the exact sum of three bf16 values (8 + 8 + 8 significant
// bits: h = bf16(x), m = bf16(x - h), l = bf16(x - h - m), every subtraction exact), and a
// product of two bf16 values is exact in fp32, so
//     a*b = ah*bh + (ah*bm + am*bh) + (am*bm + ah*bl + al*bh) + O(2^-24 |a*b|):
// six bf16 MFMAs with fp32 accumulation reproduce the fp32 contraction to fp32 rounding level
// (the dropped terms are of the size of one fp32 rounding of the product) at 6/16 of the fp32
// MFMA's matrix-core time, and that time overlaps with the staging arithmetic.  Storage stays
// fp32 in HBM; the three planes of an activation exist in LDS and registers only, those of the conv
// weights are written once per forward pass (x3_prep_kernel) in the order the kernels read them.
#include <algorithm>
#include "mbconv_x3.h"


namespace mbk {

__device__ __forceinline__ void x3_ld4(const float *p, size_t i, float (&v)[4])
{
    const float4 t = *reinterpret_cast<const float4 *>(p + i);
    v[0] = t.x;
    v[1] = t.y;
    v[2] = t.z;
    v[3] = t.w;
}
// four consecutive floats at an address that is only 4-byte aligned (pixel runs of planes whose
// size is not a multiple of four)
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void x3_ld4u(const float *p, size_t i, float (&v)[4])
{
    const float4u t = *reinterpret_cast<const float4u *>(p + i);
    v[0] = t[0];
    v[1] = t[1];
    v[2] = t[2];
    v[3] = t[3];
}

// acc += a*b for the three-plane operands (small terms first)
__device__ __forceinline__ float16v x3_mfma6(const bf16x8 (&a)[3], const bf16x8 (&b)[3], float16v acc)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[2], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], acc, 0, 0, 0);
    return acc;
}

// the five small products of x3_mfma6 (all but a[0]*b[0])
__device__ __forceinline__ float16v x3_mfma5(const bf16x8 (&a)[3], const bf16x8 (&b)[3], float16v acc)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[2], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], acc, 0, 0, 0);
    return acc;
}

// Halfword offset of element (row, k) in a plane of rows of 64 bytes (32 k) whose four 16-byte groups
// are permuted by bits 2-3 of the row: the 16-byte reads of 16 consecutive rows fall on distinct banks
// without padding.
__device__ __forceinline__ int x3_img_at(int row, int k)
{
    return row * 32 + ((((k >> 3) ^ (row >> 2)) & 3) << 3) + (k & 7);
}

// ---- weight images -------------------------------------------------------------------------
// The A operand of a convolution (rows m, contraction index k) as bf16 planes (three for fp32 weights,
// one for bf16), cut into tiles of 64 rows x 32 k in the lane order of v_mfma_f32_16x16x32_bf16:
// tile (mt, ch) is [row tile of 16][plane][lane][8 k] with lane = row % 16 + 16 * (k / 8), so that a
// wavefront reads an operand as 64 consecutive 16-byte pieces.  Rows and k past the end are zeros.
__global__ __launch_bounds__(256) void x3_prep_kernel(X3PrepArgs a) { x3_prep_tile(a, blockIdx.x, threadIdx.x); }

size_t x3_weight_image_bytes(bool bf16, int M, int K)
{
    return (size_t)((M + 63) / 64) * ((K + 31) / 32) * (bf16 ? 1 : 3) * 2048 * sizeof(uint16_t);
}

hipError_t launch_x3_prep(const X3PrepArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(x3_prep_kernel, dim3((unsigned)a.tiles), dim3(256), 0, st, a);
    return hipGetLastError();
}

// ---- weight gradient -------------------------------------------------------------------------
// dW[a,b] = sum_q op(U)[a,q] * op(V)[b,q].  Both operands are pixel-contiguous in memory, which
// is the [row][k] layout the instruction wants, so a run of four pixels goes through its
// prologue, is split and lands in LDS as one 8-byte store per plane.  A workgroup of eight
// wavefronts owns 128 rows of U by 128 rows of V (each wavefront 64 x 32) and a range of
// 32-pixel chunks; with the narrow operand inside one tile the wide one is staged, and sent
// through its prologue, once in the whole grid.  Chunks are loaded two iterations ahead into a
// ring of two register slots, so HBM stays busy while a chunk is split and multiplied.  The
// splits' partial tiles are added by a fixed-order second stage.
//
// bf16 storage (T = bf16_t): the same kernel with one plane per operand, rounded once after the fp32
// prologue, and one MFMA per product block (the accumulation is fp32 either way).  128 images of 14x14,
// 112 -> 672 -> 112: 75 us in two launches of 64-row tiles, 43 for the pair here; chunks of 64 pixels
// 70, their registers spill.
struct X3WgradOperand {
    const void *p0, *p1;
    const float *c0, *c1, *c2, *gate;
};
struct X3WgradArgs {
    int Ma, Mb, HW;
    uint32_t runs;      // runs of four pixels: (HW + 3)/4 per image
    int chunksPerSplit; // chunks of eight runs
    int tilesA, tilesB, splits;
    FastDiv divRuns; // by the runs of an image
    X3WgradOperand U, V;
    float *partial;
};

constexpr int kWgRuns = 8; // runs of a chunk
template <typename T>
constexpr int kWgPlanes = sizeof(T) == 4 ? 3 : 1;
// a run of four pixels as it comes from memory
template <typename T>
struct X3Run;
template <>
struct X3Run<float> {
    float v[4];
    template <bool RAG>
    __device__ __forceinline__ void load(const void *p, size_t i)
    {
        if (RAG)
            x3_ld4u((const float *)p, i, v);
        else
            x3_ld4((const float *)p, i, v);
    }
    __device__ __forceinline__ float get(int j) const { return v[j]; }
};
template <>
struct X3Run<bf16_t> {
    uint2 v;
    template <bool RAG>
    __device__ __forceinline__ void load(const void *p, size_t i)
    {
        v = *reinterpret_cast<const uint2 *>((const bf16_t *)p + i);
    }
    __device__ __forceinline__ float get(int j) const
    {
        const uint32_t w = j < 2 ? v.x : v.y;
        return __uint_as_float(j & 1 ? w & 0xffff0000u : w << 16);
    }
};

// What a thread keeps per operand for the whole kernel: rows rr + 64*i (i < NP) of the tile.  Rows past
// the last one are read at the last one and never stored; eight of them (a wavefront's) are not sent
// through the prologue either, their place in LDS then holds anything (96 of 128 rows, gated side, 256
// images of 28x28: 46.5 us with the prologue, 41.1 without).
template <int PRO, int NP>
struct X3RowConst {
    float k0[NP], k1[NP], k2[NP];
    int row[NP];
    uint32_t at[NP]; // offset of the row within an image
    bool live[NP];   // uniform: the wavefront's rows of this pass are not all past the end
    __device__ __forceinline__ void init(const X3WgradOperand &o, int row0, int rr, int wave, int M, int HW)
    {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int r = min(row0 + rr + 64 * i, M - 1);
            row[i] = r;
            at[i] = (uint32_t)r * (uint32_t)HW;
            live[i] = row0 + 64 * i + 8 * wave < M;
            k0[i] = k1[i] = k2[i] = 0.f;
            if (PRO != PRO_NONE) {
                k0[i] = o.c0[r];
                k1[i] = o.c1[r];
                if (PRO == PRO_BNBWD)
                    k2[i] = o.c2[r];
            }
        }
    }
};
// one ring slot of an operand: the raw pixel runs (four pixels at 4*qg) of the thread's rows
template <typename T, int PRO, int NP>
struct X3RowData {
    X3Run<T> v0[NP], v1[PRO == PRO_BNBWD ? NP : 1];
    float g[NP];
    // n, pix: image and first pixel of the run (it lies inside one plane).  Both rows load, also past
    // the last row: a branch around a load would make the loads behind it wait.
    template <bool RAG>
    __device__ __forceinline__ void load(const X3WgradOperand &o, const X3RowConst<PRO, NP> &c, int M, uint32_t img,
                                         uint32_t n, uint32_t pix)
    {
        const size_t base = (size_t)n * img + pix;
        const uint32_t gbase = n * (uint32_t)M;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const size_t idx = base + c.at[i];
            v0[i].template load<RAG>(o.p0, idx);
            if constexpr (PRO == PRO_BNBWD)
                v1[i].template load<RAG>(o.p1, idx);
            if constexpr (PRO == PRO_BNSWISH_GATE)
                g[i] = o.gate[gbase + (uint32_t)c.row[i]];
        }
    }
    // prologue, split, an 8-byte LDS store per row and plane; MASK: pixel j survives under mask[j]
    template <bool MASK>
    __device__ __forceinline__ void store(const X3RowConst<PRO, NP> &c, uint16_t *planes, int rr, int qg,
                                          const uint32_t (&mask)[4]) const
    {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            if (!c.live[i])
                continue;
            float y[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                y[j] = x3_apply<PRO>(v0[i].get(j), PRO == PRO_BNBWD ? v1[PRO == PRO_BNBWD ? i : 0].get(j) : 0.f, c.k0[i],
                                     c.k1[i], PRO == PRO_BNSWISH_GATE ? g[i] : c.k2[i]);
                if (MASK)
                    y[j] = and_mask(y[j], mask[j]);
            }
            uint16_t *at = planes + x3_img_at(rr + 64 * i, 4 * qg);
            if constexpr (kWgPlanes<T> == 1) {
                *reinterpret_cast<uint2 *>(at) = make_uint2(bf16_pack2(y[0], y[1]), bf16_pack2(y[2], y[3]));
            } else {
                uint32_t w0[3], w1[3];
                x3_split2(y[0], y[1], w0);
                x3_split2(y[2], y[3], w1);
#pragma unroll
                for (int pl = 0; pl < 3; ++pl)
                    *reinterpret_cast<uint2 *>(at + pl * (NP * 64 * 32)) = make_uint2(w0[pl], w1[pl]);
            }
        }
    }
};

// VB: rows of the V tile, 128 or 64 (a narrow second operand: each wavefront then owns 32 x 32).
// TR: the partial tile is written transposed (the host swaps the operands when the first one is
// the narrow one).
// (`bid`: the workgroup's index within this weight gradient's grid; Us, Vs: LDS for three planes
// of 128 and of VB rows)
// RAG: the plane size is no multiple of four.  The contraction runs over runs of four pixels, image by
// image; the last run of an image starts at HW - 4 and its pixels that the run before has are masked, so
// a 15x15 plane takes 57 runs (228 for its 225 pixels), every access stays 16 bytes wide (4-byte aligned)
// inside its plane, and both operands see the same order.
// These planes were the fp32 matrix cores' before, whose sums over many images are closer than those of
// a single accumulator here (the bf16 MFMA truncates a small addend to a large accumulator), so the small
// cross products have an accumulator of their own, on tiles of 128 x 64.
template <typename T, int PROU, int PROV, int VB, bool TR, bool RAG>
__device__ __forceinline__ void wgrad_x3_body(const X3WgradArgs &a, int bid, uint16_t *Us, uint16_t *Vs)
{
    constexpr int QG = kWgRuns, NPL = kWgPlanes<T>, BQ = 4 * QG, NPU = 2, NPV = VB / 64;
    constexpr int kPlane = 128 * 32, kPlaneV = VB * 32; // planes in the layout of x3_img_at
    constexpr int NA = VB == 128 ? 2 : 1;                        // 32-row blocks of U per wavefront
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // first row of this wavefront's part of the U tile and of the V tile
    const int ua = VB == 128 ? 64 * (wave >> 2) : 32 * (wave >> 1);
    const int vb = VB == 128 ? 32 * (wave & 3) : 32 * (wave & 1);
    // The (split, tile) pairs in order, an eighth of them to each XCD (blockIdx.x mod 8): workgroups
    // that read the same pixels (all tiles of one split) mostly share an XCD's L2, and no XCD has more
    // than one workgroup above the others, whatever the number of splits.  (Whole splits dealt to the
    // XCDs: ten of them gave two XCDs twice the work; 1152 x (320 + 192) over 3136 pixels: 66.7
    // us, 51.5 this way.)
    const int tiles = a.tilesA * a.tilesB, perXcd = (tiles * a.splits + 7) >> 3;
    const int item = (bid & 7) * perXcd + (bid >> 3);
    const int split = item / tiles, tile = item % tiles;
    if (split >= a.splits)
        return;
    const int a0 = (tile % a.tilesA) * 128, b0 = (tile / a.tilesA) * VB;
    const int numChunks = (int)((a.runs + QG - 1) / QG);
    const int cbeg = split * a.chunksPerSplit;
    const int cend = min(cbeg + a.chunksPerSplit, numChunks);
    const int qg = tid % QG, rr = tid / QG;
    X3RowConst<PROU, NPU> cu;
    X3RowConst<PROV, NPV> cv;
    cu.init(a.U, a0, rr, wave, a.Ma, a.HW);
    cv.init(a.V, b0, rr, wave, a.Mb, a.HW);
    const uint32_t imgU = (uint32_t)a.Ma * (uint32_t)a.HW, imgV = (uint32_t)a.Mb * (uint32_t)a.HW;
    const bool work = a0 + ua < a.Ma && b0 + vb < a.Mb; // uniform: the wavefront's part is not all padding
    X3RowData<T, PROU, NPU> du[2];
    X3RowData<T, PROV, NPV> dv[2];
    uint32_t qmask[2] = {0u, 0u};
    int fresh[2] = {0, 0};
    // unconditional clamped loads; the validity of a pixel is an AND mask on V's way into LDS
    auto load = [&](int s, int chunk) __attribute__((always_inline)) {
        const uint32_t run = (uint32_t)chunk * QG + (uint32_t)qg;
        qmask[s] = run < a.runs ? 0xffffffffu : 0u;
        const uint32_t rc = qmask[s] ? run : 0u;
        const uint32_t n = fdiv(rc, a.divRuns);
        const uint32_t want = 4u * (rc - n * a.divRuns.d), pix = RAG ? min(want, (uint32_t)a.HW - 4u) : want;
        fresh[s] = (int)(want - pix);
        du[s].template load<RAG>(a.U, cu, a.Ma, imgU, n, pix);
        dv[s].template load<RAG>(a.V, cv, a.Mb, imgV, n, pix);
    };
    auto store = [&](int s) __attribute__((always_inline)) {
        uint32_t mask[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            mask[j] = (RAG && j < fresh[s]) ? 0u : qmask[s];
        du[s].template store<false>(cu, Us, rr, qg, mask);
        dv[s].template store<true>(cv, Vs, rr, qg, mask);
    };

    static_assert(!RAG || VB == 64, "two accumulators per output: 32 x 32 per wavefront");
    float16v acc[NA], low; // low: RAG only
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        low[r] = 0.f;
#pragma unroll
        for (int i = 0; i < NA; ++i)
            acc[i][r] = 0.f;
    }
    if (cbeg < cend) { // uniform over the workgroup; an empty split writes zeros
        load(0, cbeg);
        load(1, min(cbeg + 1, cend - 1));
        store(0);
        __syncthreads();
        auto step = [&](int u, int cc) __attribute__((always_inline)) {
            load(u, min(cc + 2, cend - 1)); // slot u is free: its chunk went to LDS last iteration
            // the loads are all issued before the MFMAs start and nothing that uses their data
            // moves up among the MFMAs (the scheduler would otherwise wait for them there)
            __builtin_amdgcn_sched_barrier(0);
            if (work) {
#pragma unroll
                for (int s = 0; s < BQ / 16; ++s) {
                    const int ko = 16 * s + 8 * (lane >> 5);
                    bf16x8 av[NA][NPL], bv[NPL];
#pragma unroll
                    for (int pl = 0; pl < NPL; ++pl) {
#pragma unroll
                        for (int i = 0; i < NA; ++i)
                            av[i][pl] = x3_lds8(Us + pl * kPlane + x3_img_at(ua + 32 * i + (lane & 31), ko));
                        bv[pl] = x3_lds8(Vs + pl * kPlaneV + x3_img_at(vb + (lane & 31), ko));
                    }
#pragma unroll
                    for (int i = 0; i < NA; ++i) {
                        if constexpr (NPL == 1) {
                            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i][0], bv[0], acc[i], 0, 0, 0);
                        } else if constexpr (RAG) {
                            low = x3_mfma5(av[i], bv, low);
                            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i][0], bv[0], acc[i], 0, 0, 0);
                        } else {
                            acc[i] = x3_mfma6(av[i], bv, acc[i]);
                        }
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads(); // every wavefront has read the chunk
            store(u ^ 1);    // the repeated last chunk is stored but never consumed
            __syncthreads();
        };
        int cc = cbeg;
        for (; cc + 1 < cend; cc += 2) {
            step(0, cc);
            step(1, cc + 1);
        }
        if (cc < cend) // uniform over the workgroup
            step(0, cc);
    }
    float *dst = a.partial + (size_t)split * a.Ma * a.Mb;
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int ai = a0 + ua + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            const int bi = b0 + vb + (lane & 31);
            if (ai < a.Ma && bi < a.Mb)
                dst[TR ? (size_t)bi * a.Ma + ai : (size_t)ai * a.Mb + bi] = RAG ? acc[i][r] + low[r] : acc[i][r];
        }
}

template <typename T, int PROU, int PROV, int VB, bool TR, bool RAG>
__global__ __launch_bounds__(512) void wgrad_x3_kernel(X3WgradArgs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t Us[kWgPlanes<T> * 128 * 32];
    __shared__ __attribute__((aligned(16))) uint16_t Vs[kWgPlanes<T> * VB * 32];
    wgrad_x3_body<T, PROU, PROV, VB, TR, RAG>(a, (int)blockIdx.x, Us, Vs);
}

// The six forms of the kernel above, by number (x3_wgrad_variant).
template <typename T, int VAR, bool RAG>
__device__ __forceinline__ void wgrad_x3_variant(const X3WgradArgs &a, int bid, uint16_t *Us, uint16_t *Vs)
{
    if (VAR == 0)
        wgrad_x3_body<T, PRO_BNBWD, PRO_NONE, 128, false, false>(a, bid, Us, Vs);
    else if (VAR == 1)
        wgrad_x3_body<T, PRO_BNBWD, PRO_BNSWISH_GATE, 128, false, false>(a, bid, Us, Vs);
    else if (VAR == 2)
        wgrad_x3_body<T, PRO_BNBWD, PRO_NONE, 64, false, RAG>(a, bid, Us, Vs);
    else if (VAR == 3)
        wgrad_x3_body<T, PRO_BNBWD, PRO_BNSWISH_GATE, 64, false, RAG>(a, bid, Us, Vs);
    else if (VAR == 4)
        wgrad_x3_body<T, PRO_NONE, PRO_BNBWD, 64, true, RAG>(a, bid, Us, Vs);
    else
        wgrad_x3_body<T, PRO_BNSWISH_GATE, PRO_BNBWD, 64, true, RAG>(a, bid, Us, Vs);
}

// Two weight gradients in one launch (a block's projection and expansion conv: independent of
// each other, each about one workgroup per compute unit and bound by the latency of its own
// load-stage-multiply chain): the first gridA workgroups work on `a`, the others on `b`, and
// with at most 128 registers two workgroups, one of each, share a compute unit.
template <typename T, int VARA, int VARB, bool RAG>
__global__ __launch_bounds__(512, 4) void wgrad_x3_pair_kernel(X3WgradArgs a, X3WgradArgs b, int gridA)
{
    __shared__ __attribute__((aligned(16))) uint16_t Us[kWgPlanes<T> * 128 * 32];
    __shared__ __attribute__((aligned(16))) uint16_t Vs[kWgPlanes<T> * 128 * 32];
    if ((int)blockIdx.x < gridA) // uniform over the workgroup
        wgrad_x3_variant<T, VARA, RAG>(a, (int)blockIdx.x, Us, Vs);
    else
        wgrad_x3_variant<T, VARB, RAG>(b, (int)blockIdx.x - gridA, Us, Vs);
}

// Tile and splits.  The wider operand gets 128-row tiles; the other one 128-row tiles, or one
// 64-row tile when it has at most 64 rows (and more than 32).  Splits of the contraction: at most one workgroup (eight
// wavefronts) per compute unit, at least two chunks each.
bool x3_wgrad_plan(bool bf16, int Ma, int Mb, int N, int HW, int *splits)
{
    const long long Q = (long long)N * HW;
    // (a side of at most 32 channels belongs to the fused backward kernels of kernels_wave.hip,
    // which size their partial tiles by the plan of that file)
    // Planes of at most 64 pixels that are no multiple of four (7x7) stay on the fp32 matrix cores, the
    // engine that mbconv_step_engine has answered for them so far.  Neither speed nor accuracy asks for
    // it (64 x 7x7, 192 -> 1152 -> 320: 66 us for the pair there, 51 here; error against 64 bits 3.9e-7 and
    // 4.9e-7 there, 2.7e-7 and 3.5e-7 here).
    if (HW % 4 != 0 && HW <= 64)
        return false;
    // bf16: operands are rounded here; up to 64 x 256 rows, and on planes that are no multiple of four, the fp32
    // kernels (wgrad_lt, wgrad_rd) take them as they are
    if (bf16 && (HW % 4 != 0 || (std::min(Ma, Mb) <= 64 && std::max(Ma, Mb) <= 256)))
        return false;
    if (Q >= (1ll << 31) || (long long)std::max(Ma, Mb) * HW >= (1ll << 31) || HW < 4 || (!bf16 && std::min(Ma, Mb) <= 32) || std::max(Ma, Mb) < 64)
        return false;
    const int wide = std::max(Ma, Mb), narrow = std::min(Ma, Mb), vb = narrow <= 64 || HW % 4 != 0 ? 64 : 128;
    const long long tiles = (long long)((wide + 127) / 128) * ((narrow + vb - 1) / vb);
    const long long chunks = ((long long)N * ((HW + 3) / 4) + kWgRuns - 1) / kWgRuns;
    // (rounded down: two gradients that share a launch then just fit, two workgroups per compute unit;
    // 512 workgroups of one gradient measured slower: twice the partial tiles)
    long long s = 256 / tiles;
    const long long smax = (chunks + 1) / 2;
    if (s > smax)
        s = smax;
    if (s < 1)
        s = 1;
    const long long per = (chunks + s - 1) / s;
    *splits = (int)((chunks + per - 1) / per);
    return true;
}

static X3Operand to_x3(const Operand &o)
{
    X3Operand d;
    d.p0 = (const float *)o.p0;
    d.p1 = (const float *)o.p1;
    d.c0 = o.c0;
    d.c1 = o.c1;
    d.c2 = o.c2;
    d.gate = o.gate;
    return d;
}

static X3WgradOperand to_wgrad(const Operand &o) { return {o.p0, o.p1, o.c0, o.c1, o.c2, o.gate}; }

// Arguments, grid and kernel form (0..5, see wgrad_x3_variant) of one weight gradient.
// rag: the launch's kernel is the form for planes that are no multiple of four (either one's of a pair).
// The other one's plane then goes through 64-row tiles too, in the splits planned for 128-row ones: up
// to 512 workgroups, which measured as fast as fewer splits (18x18 -> 9x9, 64 images, 48 -> 288 -> 80:
// backward 94.5 / 94.0 us) or faster (192 -> 1152 -> 320, 32 images 219 / 230), and faster than two
// launches (100 and 232) but where both are long (34x34 -> 17x17, 64 images, 112 -> 448 -> 192: 461, 448).
static bool x3_wgrad_setup(bool bf16, bool rag, int N, int Ma, int Mb, int HW, const Operand &U, const Operand &V,
                           float *partial, X3WgradArgs *out, unsigned *grid, int *variant, int *splits_out)
{
    int splits;
    if (!x3_wgrad_plan(bf16, Ma, Mb, N, HW, &splits))
        return false;
    // a narrow first operand: the kernel computes the transposed product and writes it transposed
    const bool swap = Ma < 64 && Mb >= 64;
    const int vb = std::min(Ma, Mb) <= 64 || rag ? 64 : 128;
    X3WgradArgs a;
    a.Ma = swap ? Mb : Ma;
    a.Mb = swap ? Ma : Mb;
    a.HW = HW;
    const int perImage = (HW + 3) / 4;
    a.runs = (uint32_t)((long long)N * perImage);
    const int chunks = (int)((a.runs + kWgRuns - 1u) / kWgRuns);
    a.chunksPerSplit = (chunks + splits - 1) / splits;
    a.divRuns = make_div((uint32_t)perImage);
    a.U = to_wgrad(swap ? V : U);
    a.V = to_wgrad(swap ? U : V);
    a.partial = partial;
    *splits_out = splits;
    a.tilesA = (a.Ma + 127) / 128;
    a.tilesB = (a.Mb + vb - 1) / vb;
    a.splits = splits;
    *grid = (unsigned)((splits * a.tilesA * a.tilesB + 7) / 8 * 8);
    const int pu = swap ? V.pro : U.pro, pv = swap ? U.pro : V.pro;
    int var = -1;
    if (!swap && pu == PRO_BNBWD && pv == PRO_NONE)
        var = vb == 128 ? 0 : 2;
    else if (!swap && pu == PRO_BNBWD && pv == PRO_BNSWISH_GATE)
        var = vb == 128 ? 1 : 3;
    else if (swap && vb == 64 && pu == PRO_NONE && pv == PRO_BNBWD)
        var = 4;
    else if (swap && vb == 64 && pu == PRO_BNSWISH_GATE && pv == PRO_BNBWD)
        var = 5;
    if (var < 0)
        return false;
    *out = a;
    *variant = var;
    return true;
}

hipError_t launch_x3_wgrad(bool bf16, int N, int Ma, int Mb, int HW, const Operand &U, const Operand &V,
                           float *partial, int *splits_out, hipStream_t st)
{
    X3WgradArgs a;
    unsigned grid;
    int var;
    if (!x3_wgrad_setup(bf16, HW % 4 != 0, N, Ma, Mb, HW, U, V, partial, &a, &grid, &var, splits_out))
        return hipErrorInvalidValue;
#define MBK_CASE(VAR, PU, PV, VB_, TR_)                                                           \
    if (var == VAR) {                                                                             \
        constexpr bool kRag = VB_ == 64; /* (the other forms never see such planes) */            \
        if (bf16)                                                                                 \
            hipLaunchKernelGGL((wgrad_x3_kernel<bf16_t, PU, PV, VB_, TR_, false>), dim3(grid), dim3(512), 0, st, a); \
        else if (kRag && HW % 4 != 0)                                                             \
            hipLaunchKernelGGL((wgrad_x3_kernel<float, PU, PV, VB_, TR_, kRag>), dim3(grid), dim3(512), 0, st, a);   \
        else                                                                                      \
            hipLaunchKernelGGL((wgrad_x3_kernel<float, PU, PV, VB_, TR_, false>), dim3(grid), dim3(512), 0, st, a);  \
        return hipGetLastError();                                                                 \
    }
    MBK_CASE(0, PRO_BNBWD, PRO_NONE, 128, false)
    MBK_CASE(1, PRO_BNBWD, PRO_BNSWISH_GATE, 128, false)
    MBK_CASE(2, PRO_BNBWD, PRO_NONE, 64, false)
    MBK_CASE(3, PRO_BNBWD, PRO_BNSWISH_GATE, 64, false)
    MBK_CASE(4, PRO_NONE, PRO_BNBWD, 64, true)
    MBK_CASE(5, PRO_BNSWISH_GATE, PRO_BNBWD, 64, true)
#undef MBK_CASE
    return hipErrorInvalidValue;
}

// The projection conv's weight gradient (A: dp x sc) and the expansion conv's (B: de x x) in one
// launch.  Returns hipErrorNotSupported, nothing launched, when one of them is not a shape of
// this file or their forms are not a pair the launch has.
hipError_t launch_x3_wgrad_pair(bool bf16, int N, int MaA, int MbA, int HWA, const Operand &UA, const Operand &VA,
                                float *partialA, int *splitsA, int MaB, int MbB, int HWB,
                                const Operand &UB, const Operand &VB, float *partialB, int *splitsB,
                                hipStream_t st)
{
    X3WgradArgs a, b;
    unsigned ga, gb;
    int va, vb;
    const bool rag = HWA % 4 != 0 || HWB % 4 != 0;
    if (!x3_wgrad_setup(bf16, rag, N, MaA, MbA, HWA, UA, VA, partialA, &a, &ga, &va, splitsA) ||
        !x3_wgrad_setup(bf16, rag, N, MaB, MbB, HWB, UB, VB, partialB, &b, &gb, &vb, splitsB))
        return hipErrorNotSupported;
#define MBK_CASE(VA_, VB_)                                                                        \
    if (va == VA_ && vb == VB_) {                                                                 \
        constexpr bool kRag = VA_ >= 2 && VB_ >= 2;                                               \
        const dim3 grid(ga + gb);                                                                 \
        if (bf16)                                                                                 \
            hipLaunchKernelGGL((wgrad_x3_pair_kernel<bf16_t, VA_, VB_, false>), grid, dim3(512), 0, st, a, b, (int)ga); \
        else if (kRag && rag)                                                                     \
            hipLaunchKernelGGL((wgrad_x3_pair_kernel<float, VA_, VB_, kRag>), grid, dim3(512), 0, st, a, b, (int)ga);   \
        else                                                                                      \
            hipLaunchKernelGGL((wgrad_x3_pair_kernel<float, VA_, VB_, false>), grid, dim3(512), 0, st, a, b, (int)ga);  \
        return hipGetLastError();                                                                 \
    }
    // projection side: dp (BN backward) with the gated activation, 128- or 64-row tile, or
    // swapped; expansion side: de (BN backward) with the block's input, likewise
    MBK_CASE(1, 0)
    MBK_CASE(1, 2)
    MBK_CASE(3, 2)
    MBK_CASE(3, 0)
    MBK_CASE(5, 2)
    MBK_CASE(5, 0)
    MBK_CASE(1, 4)
    MBK_CASE(3, 4)
    MBK_CASE(5, 4)
#undef MBK_CASE
    return hipErrorNotSupported;
}

// ---- 1x1 convolution with a short contraction: weights resident in LDS, a wavefront per chunk ----
// out[n][m][q] = sum_k W[m][k] * op(B)[n][k][q] for K <= 192 and many rows (the expansion conv,
// K = Cin, and the projection conv's data gradient, K = Cout, of the wide blocks).  With
// 64 x 64 output tiles every tile stages its own copy of the B operand (load, split into planes, LDS
// stores, two barriers per 32 values of k) and lasts 2-3 us per 32 values of k for 0.2 us of
// matrix-core time; with a short contraction the tile's prologue and epilogue are most of it.
// Here the roles are turned round:
//   - a workgroup owns a slab of 64 output rows; the slab's weights, all of K, are read once, split
//     into planes and kept in LDS (at most 72 KB) in the lane order of the MFMA's A operand, so an
//     operand is one 16-byte LDS read per lane and plane, conflict-free (24 to 48 values to split
//     per thread: no weight image, and no launch ahead of the expansion conv to write one);
//   - a wavefront owns whole chunks of 32 pixels: lane (r, g) loads, for every 32 values of k,
//     the values k = 8g .. 8g+7 of its two pixels (2r and 2r+1 of the chunk when the plane size
//     is even: eight-byte loads, sixteen lanes cover a 128-byte line; r and 16+r otherwise),
//     which after the prologue and the split into planes ARE the B operands of
//     v_mfma_f32_16x16x32_bf16 (column = pixel, contraction = k): no LDS stores, no barrier in
//     the loop, and the operand is split once per pixel chunk and slab instead of once per tile;
//   - the next chunk's values of a k step are requested as soon as this chunk's have been
//     consumed; the accumulators (4 row tiles x 2 pixel tiles) are stored straight from
//     registers, eight bytes per lane, sixteen lanes to a 128-byte line;
//   - BN statistics of the output (EPI_STATS) are kept per lane over the wavefront's chunks and
//     reduced once at the end: lanes of a row, then the four wavefronts in order through LDS.
// The workgroups of all slabs that read the same pixel chunks run on the same die (most of them) and share
// its L2.
struct X3WArgs {
    int M, K, HW;
    uint32_t Q;
    int numChunks;
    FastDiv divHW;
    const float *w; // A(m, k) = w[m*sm + k*sk], sm or sk = 1
    int sm, sk;
    X3Operand B;
    float *out;
    float *psum, *psq; // EPI_STATS: [M][NT]
    int NT;            // chunk sets (= statistics partials per row)
    int slabs, perDie;
};

template <int KS, bool PAIR, int PRO, int EPI>
__global__ __launch_bounds__(256, 2) void conv_xw_kernel(X3WArgs a)
{
    static_assert(PRO == PRO_NONE || PRO == PRO_BNBWD, "prologues of the short-contraction roles");
    static_assert(EPI == EPI_NONE || EPI == EPI_STATS, "epilogues of the short-contraction roles");
    constexpr int NP = PRO == PRO_BNBWD ? 2 : 1;
    constexpr int STEP_HW = 4 * 3 * 64 * 8; // halfwords of the slab per k step: 4 row tiles, 3 planes
    extern __shared__ uint16_t lds16[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int M = a.M, K = a.K, HW = a.HW;
    // die = workgroup mod 8: all slabs of a chunk set on one, sets in turn; of the sets left over an eighth of the
    // (set, slab) pairs each
    const int die = blockIdx.x & 7, bi = blockIdx.x >> 3, whole = (a.NT >> 3) * a.slabs;
    const int rest = die * (a.perDie - whole) + bi - whole;
    const int slab = (bi < whole ? bi : rest) % a.slabs;
    const int cs = bi < whole ? (bi / a.slabs) * 8 + die : (a.NT & ~7) + rest / a.slabs;
    if (cs >= a.NT) // uniform over the workgroup
        return;

    // the slab's weights: thread -> (row r16, k group) pieces of eight k, of every 32-deep step one;
    // requested here, split into planes and parked in LDS below, after the first chunk's values have
    // been requested as well.  (Rows and k past the end: clamped loads, masked to zero.)
    float slabv[KS][8];
    const int sr = 16 * (tid >> 6) + (tid & 15), sg = (tid >> 4) & 3; // row of the slab, k group
    {
        const float *wr = a.w + (size_t)min(64 * slab + sr, M - 1) * a.sm;
        if (a.sk == 1) { // (uniform) rows of the matrix: 16-byte loads, K and every k group multiples of 8
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 v = *reinterpret_cast<const f32x4 *>(wr + min(32 * s + 8 * sg, K - 8) + 4 * h);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        slabv[s][4 * h + e] = v[e];
                }
        } else { // columns: sixteen lanes read sixteen consecutive rows
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    slabv[s][t] = wr[(size_t)min(32 * s + 8 * sg + t, K - 1) * a.sk];
        }
    }
    // BN-backward coefficients per contraction index, {c0, c1, c2, -} (zero past K)
    f32x4 *Cl = reinterpret_cast<f32x4 *>(lds16 + KS * STEP_HW); // [32*KS] (PRO_BNBWD)
    float *Rd = reinterpret_cast<float *>(lds16 + KS * STEP_HW); // [4][128]  (EPI_STATS, at the end)
    if (PRO == PRO_BNBWD) {
        for (int k = tid; k < 32 * KS; k += 256) {
            const int kk = k < K ? k : K - 1;
            const uint32_t m = k < K ? 0xffffffffu : 0u;
            Cl[k] = (f32x4){and_mask(a.B.c0[kk], m), and_mask(a.B.c1[kk], m), and_mask(a.B.c2[kk], m), 0.f};
        }
    }
    // the lane's eight contraction rows of step s start at row 32s + 8g, clamped to the last
    // group of eight (K % 8 == 0; the slab is zero past K)
    uint32_t vrow[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s)
        vrow[s] = (uint32_t)min(32 * s + 8 * g, K - 8) * (uint32_t)HW;
    const uint32_t mrow = (uint32_t)(64 * slab + 4 * g) * (uint32_t)HW; // output row 16i + v above it
    const uint32_t bimg = (uint32_t)K * (uint32_t)HW, oimg = (uint32_t)M * (uint32_t)HW;

    // pixel tile pt of chunk c: pixel 2r + pt (pairs) or r + 16 pt
    const auto locate = [&](int c, uint32_t (&bo)[2], uint32_t (&oo)[2], uint32_t (&okm)[2]) {
#pragma unroll
        for (int pt = 0; pt < (PAIR ? 1 : 2); ++pt) {
            const uint32_t q = (uint32_t)c * 32u + (PAIR ? 2u * (uint32_t)r : 16u * pt + (uint32_t)r);
            okm[pt] = q < a.Q ? 0xffffffffu : 0u;
            const uint32_t qs = q < a.Q ? q : 0u;
            const uint32_t n = fdiv(qs, a.divHW), pix = qs - n * (uint32_t)HW;
            bo[pt] = n * bimg + pix;
            oo[pt] = n * oimg + pix;
        }
        if (PAIR) {
            bo[1] = bo[0];
            oo[1] = oo[0];
            okm[1] = okm[0];
        }
    };
    float xv[NP][KS][2][8];
    const auto fetch_step = [&](int s, const uint32_t (&bo)[2]) {
        const uint32_t o0 = bo[0] + vrow[s], o1 = bo[1] + vrow[s];
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float *pb = (p == 0 ? a.B.p0 : a.B.p1) + (size_t)t * HW; // uniform
                if (PAIR) {
                    const f32x2 v2 = *reinterpret_cast<const f32x2 *>(pb + o0);
                    xv[p][s][0][t] = v2[0];
                    xv[p][s][1][t] = v2[1];
                } else {
                    xv[p][s][0][t] = pb[o0];
                    xv[p][s][1][t] = pb[o1];
                }
            }
    };

    f32x4 acc[4][2];
    float s1[4][4], s2[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            s1[i][v] = s2[i][v] = 0.f;

    const int cStep = 4 * a.NT;
    int ch = 4 * cs + wv;
    uint32_t bo[2], oo[2], okm[2];
    locate(ch < a.numChunks ? ch : 0, bo, oo, okm);
#pragma unroll
    for (int s = 0; s < KS; ++s)
        fetch_step(s, bo);
    __builtin_amdgcn_sched_barrier(0);
    {
        const bool mok = 64 * slab + sr < M;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            uint32_t p[4][3];
            bf16x8 o[3];
#pragma unroll
            for (int t = 0; t < 8; ++t)
                slabv[s][t] = and_mask(slabv[s][t], mok && 32 * s + 8 * sg + t < K ? 0xffffffffu : 0u);
            x3_split8(slabv[s], p, o);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
                *reinterpret_cast<bf16x8 *>(lds16 + s * STEP_HW + (((tid >> 6) * 3 + pl) * 64 + lane) * 8) = o[pl];
        }
    }
    __syncthreads(); // the slab, Cl

    for (; ch < a.numChunks; ch += cStep) {
        const int nx = ch + cStep < a.numChunks ? ch + cStep : ch;
        uint32_t nbo[2], noo[2], nokm[2];
        locate(nx, nbo, noo, nokm);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            acc[i][0] = acc[i][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            float d0[8], d1[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                if (PRO == PRO_BNBWD) {
                    const f32x4 k = Cl[32 * s + 8 * g + t];
                    d0[t] = fmaf(k[0], xv[0][s][0][t], fmaf(k[1], xv[NP - 1][s][0][t], k[2]));
                    d1[t] = fmaf(k[0], xv[0][s][1][t], fmaf(k[1], xv[NP - 1][s][1][t], k[2]));
                } else {
                    d0[t] = xv[0][s][0][t];
                    d1[t] = xv[0][s][1][t];
                }
                d0[t] = and_mask(d0[t], okm[0]);
                d1[t] = and_mask(d1[t], okm[1]);
            }
            fetch_step(s, nbo);
            uint32_t p0[4][3], p1[4][3];
            bf16x8 b0[3], b1[3];
            x3_split8(d0, p0, b0);
            x3_split8(d1, p1, b1);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                bf16x8 av[3];
#pragma unroll
                for (int pl = 0; pl < 3; ++pl)
                    av[pl] = x3_lds8(lds16 + s * STEP_HW + ((i * 3 + pl) * 64 + lane) * 8);
                acc[i][0] = x3_mfma6_16(av, b0, acc[i][0]);
                acc[i][1] = x3_mfma6_16(av, b1, acc[i][1]);
            }
            // (one step at a time: the scheduler would otherwise split every step's operands
            // ahead of the first MFMA and run out of registers)
            __builtin_amdgcn_sched_barrier(0);
        }
        // rows 64 slab + 16i + 4g + v, the lane's two pixels
        const bool ok0 = okm[0] != 0u, ok1 = okm[1] != 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float *po = a.out + (size_t)(16 * i + v) * HW; // uniform
                const float x0 = acc[i][0][v], x1 = acc[i][1][v];
                const bool mok = 64 * slab + 16 * i + 4 * g + v < M;
                if (PAIR) {
                    if (ok0 && mok)
                        *reinterpret_cast<f32x2 *>(po + oo[0] + mrow) = (f32x2){x0, x1};
                } else {
                    if (ok0 && mok)
                        po[oo[0] + mrow] = x0;
                    if (ok1 && mok)
                        po[oo[1] + mrow] = x1;
                }
                if (EPI == EPI_STATS) { // (pixels past the end were masked to zero on the way in)
                    s1[i][v] += x0 + x1;
                    s2[i][v] = fmaf(x0, x0, fmaf(x1, x1, s2[i][v]));
                }
            }
#pragma unroll
        for (int pt = 0; pt < 2; ++pt) {
            bo[pt] = nbo[pt];
            oo[pt] = noo[pt];
            okm[pt] = nokm[pt];
        }
    }
    if (EPI == EPI_STATS) {
        // lanes of a row hold the same 16 channels: add them, then the wavefronts in order
        __syncthreads(); // (Rd lies over Cl)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float t1 = row16_sum(s1[i][v]), t2 = row16_sum(s2[i][v]);
                if (r == 0) {
                    Rd[wv * 128 + 16 * i + 4 * g + v] = t1;
                    Rd[wv * 128 + 64 + 16 * i + 4 * g + v] = t2;
                }
            }
        __syncthreads();
        if (tid < 128) {
            const int mm = 64 * slab + (tid & 63);
            const float t = (Rd[tid] + Rd[128 + tid]) + (Rd[256 + tid] + Rd[384 + tid]);
            if (mm < M)
                (tid < 64 ? a.psum : a.psq)[(size_t)mm * a.NT + cs] = t;
        }
    }
}

// Shapes and roles served: contraction of at most 192 (96 with the two-tensor prologue), a
// multiple of 8; at least one 64-row slab of output; fp32.  `nt`: chunk sets = statistics
// partials per row.
bool xw_conv_plan(int N, int M, int K, int HW, int pro, int epi, int *nt)
{
    const long long Q = (long long)N * HW;
    if (K % 8 != 0 || K < 32 || K > (pro == PRO_BNBWD ? 96 : 192) || M < 64 || M < K)
        return false;
    if ((pro != PRO_NONE && pro != PRO_BNBWD) || (epi != EPI_NONE && epi != EPI_STATS))
        return false;
    if (Q * M >= (1ll << 30) || Q * K >= (1ll << 30)) // 32-bit byte offsets in the kernel
        return false;
    const int slabs = (M + 63) / 64;
    const long long chunks = (Q + 31) / 32;
    // about two workgroups per CU in all; of the counts that need the same number of rounds over the chunk
    // groups (four chunks, one per wavefront), a small one, and never more than there are groups (192 -> 1152
    // on 64 planes of 7x7 was 32 sets for 25 groups, 576 workgroups, an eighth of them in a second round: 28.3
    // us, 22.1 with 25).  Rounded up to a multiple of 8: the smallest leaves too few wavefronts in flight
    // (80 -> 480, 32 planes of 28x28: step 287 us with 56 sets, 292 with 49).
    const long long groups = (chunks + 3) / 4;
    long long sets = ((512 + slabs - 1) / slabs + 7) / 8 * 8;
    const long long rounds = (groups + sets - 1) / sets;
    sets = std::min(groups, ((groups + rounds - 1) / rounds + 7) / 8 * 8);
    *nt = (int)sets;
    return true;
}

hipError_t launch_xw_conv1x1(int N, int M, int K, int HW, const void *w, int sAm, int sAk, const Operand &B,
                             void *out, int epi, float *psum, float *psq, hipStream_t st)
{
    int nt;
    if (!xw_conv_plan(N, M, K, HW, B.pro, epi, &nt))
        return hipErrorInvalidValue;
    X3WArgs a;
    a.M = M;
    a.K = K;
    a.HW = HW;
    a.Q = (uint32_t)((long long)N * HW);
    a.numChunks = (int)((a.Q + 31u) / 32u);
    a.divHW = make_div((uint32_t)HW);
    a.w = (const float *)w;
    a.sm = sAm;
    a.sk = sAk;
    a.B = to_x3(B);
    a.out = (float *)out;
    a.psum = psum;
    a.psq = psq;
    a.NT = nt;
    a.slabs = (M + 63) / 64;
    a.perDie = (nt >> 3) * a.slabs + ((nt & 7) * a.slabs + 7) / 8;
    const int ks = (K + 31) / 32;
    const bool pair = HW % 2 == 0;
    const dim3 grid((unsigned)(8 * a.perDie));
    const size_t lds = (size_t)ks * 12288 + (B.pro == PRO_BNBWD ? std::max((size_t)ks * 512, (size_t)2048) : 2048);
#define MBK_CASE(KS_, PAIR_, PRO_, EPI_)                                                          \
    if (ks == KS_ && pair == PAIR_ && B.pro == PRO_ && epi == EPI_) {                             \
        auto kern = conv_xw_kernel<KS_, PAIR_, PRO_, EPI_>;                                       \
        const hipError_t e_ = hipFuncSetAttribute(                                                \
            (const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);            \
        if (e_ != hipSuccess)                                                                     \
            return e_;                                                                            \
        hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, a);                                    \
        return hipGetLastError();                                                                 \
    }
#define MBK_KS(KS_)                                                                               \
    MBK_CASE(KS_, true, PRO_NONE, EPI_STATS)                                                      \
    MBK_CASE(KS_, false, PRO_NONE, EPI_STATS)                                                     \
    MBK_CASE(KS_, true, PRO_NONE, EPI_NONE)                                                       \
    MBK_CASE(KS_, false, PRO_NONE, EPI_NONE)
    MBK_KS(1)
    MBK_KS(2)
    MBK_KS(3)
    MBK_KS(4)
    MBK_KS(5)
    MBK_KS(6)
#undef MBK_KS
#define MBK_KS(KS_)                                                                               \
    MBK_CASE(KS_, true, PRO_BNBWD, EPI_NONE)                                                      \
    MBK_CASE(KS_, false, PRO_BNBWD, EPI_NONE)                                                     \
    MBK_CASE(KS_, true, PRO_BNBWD, EPI_STATS)                                                     \
    MBK_CASE(KS_, false, PRO_BNBWD, EPI_STATS)
    MBK_KS(1)
    MBK_KS(2)
    MBK_KS(3)
    MBK_KS(4)
#undef MBK_KS
#undef MBK_CASE
    return hipErrorInvalidValue;
}

// ---- 1x1 convolution with a short contraction and few pixels: a workgroup per tile ----
// The expansion conv of a request or a small batch has a few chunks of 32 pixels, and conv_xw, which keeps 64 rows
// of weights in LDS for many chunks, then spends a chain of latencies on a handful of workgroups: load the slab, split it,
// barrier, then every step of the contraction in turn on one wavefront (192 -> 1152 channels on one 7x7 plane: 24
// workgroups, half of whose wavefronts have no chunk, 11.7 us); so does conv_pe, up to 40 input channels, with a
// workgroup for all rows of 64 pixels (40 -> 240 on one 28x28 plane: 13 workgroups, 12.0 us).  Here a workgroup
// owns 16 rows by 32 pixels and has a wavefront for each step of 32 of the contraction: everything is requested at
// once, and the steps are added in order through LDS.  On fp32 MFMA: sixteen instructions of a wavefront take as long as splitting its operands would.
// Evaluation of the blocks named, 33.3 -> 25.6 and 24.9 -> 17.5 us.
struct X3SArgs {
    int M, K, HW;
    uint32_t Q;
    FastDiv divHW, divTiles;
    const float *w, *x; // [M][K], [n][K][HW]
    float *out;
    float *psum, *psq;  // [M][chunks]
    int tiles, chunks;
};

template <int KS, bool PAIR>
__global__ __launch_bounds__(64 * KS) void conv_xs_kernel(X3SArgs a)
{
    __shared__ f32x4 part[KS][2][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int s = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int M = a.M, K = a.K, HW = a.HW;
    const int chunk = (int)fdiv(blockIdx.x, a.divTiles), m0 = 16 * ((int)blockIdx.x - chunk * a.tiles);
    // A: row m0 + r, contraction 32s + 8g .. +7 (past the end clamped; K % 8 == 0).  Instruction t takes k = 8g + t of
    // every g, the contraction's order being free.
    const int k0 = min(32 * s + 8 * g, K - 8);
    const uint32_t kok = 32 * s + 8 * g < K ? 0xffffffffu : 0u;
    float av[8], d0[8], d1[8];
    {
        const float *wr = a.w + (size_t)min(m0 + r, M - 1) * K + k0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 v = *reinterpret_cast<const f32x4 *>(wr + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                av[4 * h + e] = v[e];
        }
    }
    // pixel tile pt: pixel 2r + pt of the chunk (pairs: one image, HW being even) or r + 16 pt
    uint32_t bo[2], oo[2], okm[2];
#pragma unroll
    for (int pt = 0; pt < 2; ++pt) {
        const uint32_t q = (uint32_t)chunk * 32u + (PAIR ? 2u * (uint32_t)r : 16u * pt + (uint32_t)r);
        okm[pt] = q < a.Q ? 0xffffffffu : 0u;
        const uint32_t qs = q < a.Q ? q : 0u;
        const uint32_t n = fdiv(qs, a.divHW), pix = qs - n * (uint32_t)HW;
        bo[pt] = (n * (uint32_t)K + (uint32_t)k0) * (uint32_t)HW + pix;
        oo[pt] = n * (uint32_t)M * (uint32_t)HW + pix;
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float *pb = a.x + (size_t)t * HW; // uniform
        if (PAIR) {
            const f32x2 v = *reinterpret_cast<const f32x2 *>(pb + bo[0]);
            d0[t] = v[0];
            d1[t] = v[1];
        } else {
            d0[t] = pb[bo[0]];
            d1[t] = pb[bo[1]];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // (past the contraction both operands are zero: what was loaded there may be infinite)
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float w = and_mask(av[t], kok);
        acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(w, and_mask(d0[t], okm[0] & kok), acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(w, and_mask(d1[t], okm[1] & kok), acc1, 0, 0, 0);
    }
    if (KS > 1) {
        part[s][0][lane] = acc0;
        part[s][1][lane] = acc1;
        __syncthreads();
        if (s != 0) // uniform over the wavefront
            return;
#pragma unroll
        for (int j = 1; j < KS; ++j) {
            acc0 += part[j][0][lane];
            acc1 += part[j][1][lane];
        }
    }
    // rows m0 + 4g + v, the lane's two pixels
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int m = m0 + 4 * g + v;
        const float x0 = acc0[v], x1 = acc1[v];
        if (m < M) {
            float *po = a.out + (size_t)m * HW;
            if (PAIR) {
                if (okm[0])
                    *reinterpret_cast<f32x2 *>(po + oo[0]) = (f32x2){x0, x1};
            } else {
                if (okm[0])
                    po[oo[0]] = x0;
                if (okm[1])
                    po[oo[1]] = x1;
            }
        }
        // statistics of the output (pixels past the end were masked to zero on the way in)
        const float t1 = row16_sum(x0 + x1), t2 = row16_sum(fmaf(x0, x0, x1 * x1));
        if (r == 0 && m < M) {
            a.psum[(size_t)m * a.chunks + chunk] = t1;
            a.psq[(size_t)m * a.chunks + chunk] = t2;
        }
    }
}

int wave_conv_kind(int M, int K, int HW); // kernels_pv16.hip

// `nt`: chunks = statistics partials per row.
bool xs_conv_plan(int N, int M, int K, int HW, int pro, int epi, int *nt)
{
    const long long Q = (long long)N * HW, chunks = (Q + 31) / 32;
    // (the expansion conv's role, and shapes whose rows are whole 32-byte pieces)
    if (K % 8 != 0 || K < 8 || K > 192 || pro != PRO_NONE || epi != EPI_STATS)
        return false;
    if (Q * M >= (1ll << 30) || Q * K >= (1ll << 30)) // 32-bit byte offsets in the kernel
        return false;
    bool ok;
    // Where the other kernel is conv_pe (kernels_pv16.hip: planes of a multiple of four pixels, up to 40 input and 384 output
    // channels), which leaves BN1 fewer partial sums: as many as its finalise step adds beside the planes for nothing.
    // (Forward, times as fast as conv_pe: 24 -> 144 on 28x28 at 588, 1151 and 1739 chunks 1.12, 1.05, 0.96; 16 -> 96 on 56x56 at
    // 784 and 1176 1.05, 1.03; 8 -> 24 on 112x112 at 1176 and 1960 1.03, 1.01, on 56x56 at 1960 0.97; 40 -> 120 on 56x56 at 980 and
    // 1960 1.06, 0.98; 40 -> 240 on 14x14 at 1065 and 2131 1.12, 1.00; 16 -> 192 on 56x56 at 784 and 1568 1.02, 0.97; 40 -> 384 on
    // 28x28 at 759, 1543 and 3062 1.06, 1.03, 0.86.)
    if (wave_conv_kind(M, K, HW))
        ok = chunks <= 1200;
    // Elsewhere up to one and a half times what is resident at once; beyond, the rows that every workgroup reads again cost
    // more than the latencies (80 -> 480 on 14x14 and 15x15 at 8, 16 and 32 thousand wavefronts 1.02 to 1.04, 1.00, 0.9;
    // 24 -> 144 on 57x57 1.04, 1.02, 1.00).  conv_xw catches up sooner where it has few rows to stage and reads
    // the pixels once: 64 -> 64 on 14x14, 251, 502 and 998 chunks 1.07, 1.01, 0.92; 32 -> 96
    // on 27x27, 660 and 1344 1.05, 0.97; 56 -> 168 on 17x17, 524, evaluation of the block 49.9 / 48.5 us.
    else {
        int sets;
        const long long waves = chunks * ((M + 15) / 16) * ((K + 31) / 32);
        ok = waves <= 12 * 1024 && (chunks <= 600 || !xw_conv_plan(N, M, K, HW, pro, epi, &sets));
    }
    if (!ok)
        return false;
    *nt = (int)chunks;
    return true;
}

hipError_t launch_xs_conv1x1(int N, int M, int K, int HW, const void *w, int sAm, int sAk, const Operand &B, void *out,
                             int epi, float *psum, float *psq, hipStream_t st)
{
    int nt;
    if (!xs_conv_plan(N, M, K, HW, B.pro, epi, &nt) || sAm != K || sAk != 1)
        return hipErrorInvalidValue;
    X3SArgs a;
    a.M = M;
    a.K = K;
    a.HW = HW;
    a.Q = (uint32_t)((long long)N * HW);
    a.divHW = make_div((uint32_t)HW);
    a.w = (const float *)w;
    a.x = (const float *)B.p0;
    a.out = (float *)out;
    a.psum = psum;
    a.psq = psq;
    a.tiles = (M + 15) / 16;
    a.chunks = nt;
    a.divTiles = make_div((uint32_t)a.tiles);
    const int ks = (K + 31) / 32;
    const bool pair = HW % 2 == 0;
    const dim3 grid((unsigned)(a.tiles * nt));
#define MBK_KS(KS_)                                                                               \
    if (ks == KS_) {                                                                              \
        if (pair)                                                                                 \
            hipLaunchKernelGGL((conv_xs_kernel<KS_, true>), grid, dim3(64 * KS_), 0, st, a);      \
        else                                                                                      \
            hipLaunchKernelGGL((conv_xs_kernel<KS_, false>), grid, dim3(64 * KS_), 0, st, a);     \
        return hipGetLastError();                                                                 \
    }
    MBK_KS(1)
    MBK_KS(2)
    MBK_KS(3)
    MBK_KS(4)
    MBK_KS(5)
    MBK_KS(6)
#undef MBK_KS
    return hipErrorInvalidValue;
}

} // namespace mbk
