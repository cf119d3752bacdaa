// Weight gradient of a 1x1 convolution on fp32 MFMA: the planes and channel counts that the bf16 matrix cores'
// kernel (kernels_x3.hip) and the one for few channels on even planes (kernels_wave.hip) do not take, 7x7 above all.
//
//   dW[a][b] = sum_{n,q} op(U)[n][a][q] * op(V)[n][b][q]
//
// A workgroup owns 64 rows of U by 64 of V (each of its four wavefronts 32 x 32) and a range of 32-pixel
// chunks.  Both operands are contiguous in pixels and the matrix cores want rows across lanes, so a chunk is
// loaded a pixel (or, on planes of a multiple of four pixels, a run of four) per lane, goes through its
// prologue and is transposed on its way into one of two LDS buffers while the other is multiplied.
//
// fp32 MFMA runs at the vector rate and blocks it, so every vector instruction of the staging is paid in
// matrix time: per chunk and wavefront 1024 cycles of MFMA next to some 600 for V (normalisation, activation,
// gate) and U.  Hence one 32-bit add per load (row offsets kept, uniform bases; with 64-bit products of image,
// row and plane it was three times as much): the pair 1152 x (320 + 192) on 64 planes of 7x7, 85 us before,
// 71 now, 24 at the rate of the unit.  (Operands loaded straight into registers, sixteen rows of
// 64 bytes to an instruction, no LDS: 92 us, the rows of odd planes are not aligned and the cache then takes
// an access per lane.)
#include <algorithm>
#include "mbconv_wgr_plan.h"
#include "mbconv_x3.h"

namespace mbk {

struct WgrOperand {
    const void *p0, *p1;
    const float *c0, *c1, *c2, *gate;
};
struct WgrArgs {
    int Ma, Mb, HW;
    uint32_t Q;
    int chunks, perSplit; // of 32 pixels
    FastDiv divHW;
    WgrOperand U, V;
    float *partial;       // [splits][Ma][Mb]
    int tilesA, tilesB, splits;
    int perDie;           // items a die takes
};

constexpr int kWgrPitch = 66; // floats per pixel of a chunk in LDS: 64 rows + 2

// VEC consecutive pixels of a row
template <typename T, int VEC>
struct WgrRaw;
template <>
struct WgrRaw<float, 1> {
    float v;
    __device__ __forceinline__ void load(const char *p) { v = *reinterpret_cast<const float *>(p); }
    __device__ __forceinline__ float get(int) const { return v; }
};
template <>
struct WgrRaw<float, 4> {
    f32x4 v;
    __device__ __forceinline__ void load(const char *p) { v = *reinterpret_cast<const f32x4 *>(p); }
    __device__ __forceinline__ float get(int j) const { return v[j]; }
};
template <>
struct WgrRaw<bf16_t, 1> {
    uint16_t v;
    __device__ __forceinline__ void load(const char *p) { v = *reinterpret_cast<const uint16_t *>(p); }
    __device__ __forceinline__ float get(int) const { return bf16_bits_to_float(v); }
};
template <>
struct WgrRaw<bf16_t, 4> {
    u32x2 v;
    __device__ __forceinline__ void load(const char *p) { v = *reinterpret_cast<const u32x2 *>(p); }
    __device__ __forceinline__ float get(int j) const
    {
        return __uint_as_float(j & 1 ? v[j >> 1] & 0xffff0000u : v[j >> 1] << 16);
    }
};

template <typename T, int PROV, int VEC>
__device__ __forceinline__ void wgr_body(const WgrArgs &a, int item, float (*Us)[32 * kWgrPitch],
                                         float (*Vs)[32 * kWgrPitch])
{
    constexpr int QC = 32 / VEC;               // runs of a chunk
    constexpr int RR = 256 / QC, NR = 64 / RR; // rows a pass, passes
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wa = wave >> 1, wb = wave & 1;
    // items: the wider side's tiles outermost, then the other's, then the splits, so that what shares the
    // wider operand's rows shares a die
    const int split = item % a.splits, t = item / a.splits;
    const int cbeg = split * a.perSplit, cend = min(cbeg + a.perSplit, a.chunks);
    const bool wideA = a.tilesA >= a.tilesB;
    const int minor = wideA ? a.tilesB : a.tilesA;
    const int ta = wideA ? t / minor : t % minor, tb = wideA ? t % minor : t / minor;
    const int Ma = a.Ma, Mb = a.Mb;
    const uint32_t HW = (uint32_t)a.HW;
    // byte offsets are 32 bits, from the split's first image on: its images lie within 4 GiB (wgr_least)
    const uint32_t q0 = (uint32_t)min(cbeg, a.chunks - 1) * 32u, n0 = fdiv(q0, a.divHW);
    const size_t fromU = (size_t)n0 * Ma * HW * sizeof(T), fromV = (size_t)n0 * Mb * HW * sizeof(T);
    const char *u0 = (const char *)a.U.p0 + fromU, *u1 = (const char *)a.U.p1 + fromU, *v0 = (const char *)a.V.p0 + fromV;
    const char *gates = (const char *)a.V.gate + (size_t)n0 * Mb * 4u;
    const int qcol = tid % QC, rrow = tid / QC;

    // rows rrow + RR*i of the tiles (past the end the last one: never stored), byte offsets within an image
    uint32_t atU[NR], atV[NR], atG[NR];
    float ku[NR][3], kv[NR][2];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int ra = min(64 * ta + rrow + RR * i, Ma - 1), rb = min(64 * tb + rrow + RR * i, Mb - 1);
        atU[i] = (uint32_t)ra * HW * (uint32_t)sizeof(T);
        atV[i] = (uint32_t)rb * HW * (uint32_t)sizeof(T);
        atG[i] = (uint32_t)rb * 4u;
        ku[i][0] = a.U.c0[ra];
        ku[i][1] = a.U.c1[ra];
        ku[i][2] = a.U.c2[ra];
        kv[i][0] = kv[i][1] = 0.f;
        if (PROV != PRO_NONE) {
            kv[i][0] = a.V.c0[rb];
            kv[i][1] = a.V.c1[rb];
        }
    }
    WgrRaw<T, VEC> xu[NR], yu[NR], xv[NR];
    float gate[NR];
    uint32_t okm = 0; // the run is inside the batch
    const auto fetch = [&](int chunk) __attribute__((always_inline)) {
        const uint32_t q = (uint32_t)chunk * 32u + (uint32_t)(qcol * VEC), qc = q < a.Q ? q : q0;
        okm = q < a.Q ? 0xffffffffu : 0u;
        const uint32_t image = fdiv(qc, a.divHW), pix = qc - image * HW, n = image - n0;
        const uint32_t bu = (n * (uint32_t)Ma * HW + pix) * (uint32_t)sizeof(T);
        const uint32_t bv = (n * (uint32_t)Mb * HW + pix) * (uint32_t)sizeof(T), bg = n * (uint32_t)Mb * 4u;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            xv[i].load(v0 + (bv + atV[i]));
            if (PROV == PRO_BNSWISH_GATE)
                gate[i] = *reinterpret_cast<const float *>(gates + (bg + atG[i]));
            xu[i].load(u0 + (bu + atU[i]));
            yu[i].load(u1 + (bu + atU[i]));
        }
    };
    const auto store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                const int at = (qcol * VEC + j) * kWgrPitch + rrow + RR * i;
                const float v = x3_apply<PROV>(xv[i].get(j), 0.f, kv[i][0], kv[i][1], PROV == PRO_NONE ? 0.f : gate[i]);
                Vs[buf][at] = and_mask(v, okm);
                Us[buf][at] = and_mask(fmaf(ku[i][0], xu[i].get(j), fmaf(ku[i][1], yu[i].get(j), ku[i][2])), okm);
            }
    };

    float16v acc;
#pragma unroll
    for (int k = 0; k < 16; ++k)
        acc[k] = 0.f;
    const int ua = (lane >> 5) * kWgrPitch + 32 * wa + (lane & 31), va = (lane >> 5) * kWgrPitch + 32 * wb + (lane & 31);
    if (cbeg < cend) { // uniform over the workgroup; an empty split writes zeros
        fetch(cbeg);
        store(0);
        __syncthreads();
        for (int c = cbeg; c < cend; ++c) {
            const int buf = (c - cbeg) & 1;
            fetch(min(c + 1, cend - 1)); // (the repeated last chunk is stored but never consumed)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 32; k += 2)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(Us[buf][ua + k * kWgrPitch], Vs[buf][va + k * kWgrPitch], acc, 0, 0,
                                                           0);
            __builtin_amdgcn_sched_barrier(0);
            store(buf ^ 1);
            __syncthreads();
        }
    }
    float *dst = a.partial + (size_t)split * Ma * Mb;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int m = 64 * ta + 32 * wa + 8 * (k >> 2) + 4 * (lane >> 5) + (k & 3), n = 64 * tb + 32 * wb + (lane & 31);
        if (m < Ma && n < Mb)
            dst[(size_t)m * Mb + n] = acc[k];
    }
}

// The first 8*a.perDie workgroups work on `a`, the others on `b` (the two weight gradients of a block, which do
// not depend on each other).  die = workgroup mod 8.
template <typename T, int PVA, int PVB, int VEC>
__global__ __launch_bounds__(256, 4) void wgrad_rd_kernel(WgrArgs a, WgrArgs b)
{
    __shared__ float Us[2][32 * kWgrPitch], Vs[2][32 * kWgrPitch];
    const int die = blockIdx.x & 7, k = blockIdx.x >> 3;
    if (k < a.perDie) { // uniform over the workgroup
        const int item = die * a.perDie + k;
        if (item < a.tilesA * a.tilesB * a.splits)
            wgr_body<T, PVA, VEC>(a, item, Us, Vs);
    } else {
        const int item = die * b.perDie + k - a.perDie;
        if (item < b.tilesA * b.tilesB * b.splits)
            wgr_body<T, PVB, VEC>(b, item, Us, Vs);
    }
}

// Workgroups that are resident at once (four to a compute unit), less what eight dies' remainders can add
constexpr int kWgrResident = 4 * 256 - 16;
static int wgr_tiles(int Ma, int Mb) { return ((Ma + 63) / 64) * ((Mb + 63) / 64); }
static int wgr_chunks(int N, int HW) { return (int)(((long long)N * HW + 31) / 32); }

// The fewest splits whose images each lie within 4 GiB, the span of the kernel's byte offsets; 0: not even a chunk's do.
static int wgr_least(bool bf16, int Ma, int Mb, int N, int HW)
{
    const long long image = (long long)std::max(Ma, Mb) * std::max(HW * (bf16 ? 2 : 4), 4); // (its gates: 4 bytes a row)
    const long long images = ((1ll << 32) - 1) / image;
    const long long chunks = images > 2 ? (images - 2) * HW / 32 : 0; // 32*chunks pixels touch that many images at most
    return chunks ? (int)((wgr_chunks(N, HW) + chunks - 1) / chunks) : 0;
}

// As many splits as are resident at once, of four chunks or more (the last one fewer: 117 -> 171 channels on 29 planes of
// 3x3, nine chunks, training step 75.0 us with two splits, 71.5 with three).
bool wgr_plan(bool bf16, int Ma, int Mb, int N, int HW, int *splits)
{
    const int most = (wgr_chunks(N, HW) + 3) / 4, least = wgr_least(bf16, Ma, Mb, N, HW);
    *splits = std::max(least, std::min(std::min(640, kWgrResident) / wgr_tiles(Ma, Mb), most));
    return least > 0;
}

static WgrArgs wgr_args(int N, int Ma, int Mb, int HW, const Operand &U, const Operand &V, float *partial, int splits)
{
    WgrArgs a;
    a.Ma = Ma;
    a.Mb = Mb;
    a.HW = HW;
    a.Q = (uint32_t)((long long)N * HW);
    a.chunks = wgr_chunks(N, HW);
    a.perSplit = (a.chunks + splits - 1) / splits;
    a.divHW = make_div((uint32_t)HW);
    a.U = {U.p0, U.p1, U.c0, U.c1, U.c2, nullptr};
    a.V = {V.p0, nullptr, V.c0, V.c1, nullptr, V.gate};
    a.partial = partial;
    a.tilesA = (Ma + 63) / 64;
    a.tilesB = (Mb + 63) / 64;
    a.splits = splits;
    a.perDie = (a.tilesA * a.tilesB * splits + 7) / 8;
    return a;
}

static hipError_t wgr_go(bool bf16, bool gated, const WgrArgs &a, const WgrArgs &b, hipStream_t st)
{
    const dim3 grid((unsigned)(8 * (a.perDie + b.perDie)));
    const bool v4 = a.HW % 4 == 0 && b.HW % 4 == 0;
#define MBK_CASE(T, PVA, VEC)                                                                     \
    {                                                                                             \
        hipLaunchKernelGGL((wgrad_rd_kernel<T, PVA, PRO_NONE, VEC>), grid, dim3(256), 0, st, a, b); \
        return hipGetLastError();                                                                 \
    }
#define MBK_T(T)                                                                                  \
    {                                                                                             \
        if (gated && v4)                                                                          \
            MBK_CASE(T, PRO_BNSWISH_GATE, 4)                                                      \
        if (gated)                                                                                \
            MBK_CASE(T, PRO_BNSWISH_GATE, 1)                                                      \
        if (v4)                                                                                   \
            MBK_CASE(T, PRO_NONE, 4)                                                              \
        MBK_CASE(T, PRO_NONE, 1)                                                                  \
    }
    if (bf16)
        MBK_T(bf16_t)
    MBK_T(float)
#undef MBK_T
#undef MBK_CASE
}

hipError_t launch_wgr(bool bf16, int N, int Ma, int Mb, int HW, const Operand &U, const Operand &V, float *partial,
                      int *splits_out, hipStream_t st)
{
    int splits;
    if (!wgr_plan(bf16, Ma, Mb, N, HW, &splits) || U.pro != PRO_BNBWD || V.pro == PRO_BNBWD)
        return hipErrorInvalidValue;
    *splits_out = splits;
    const WgrArgs a = wgr_args(N, Ma, Mb, HW, U, V, partial, splits);
    WgrArgs none = a;
    none.perDie = 0;
    return wgr_go(bf16, V.pro != PRO_NONE, a, none, st);
}

// Two of them in one launch (A: the projection conv's, B: the expansion conv's), which leave each other's
// workgroups room (mbconv_wgr_plan.h).
hipError_t launch_wgr_pair(bool bf16, int N, int MaA, int MbA, int HWA, const Operand &UA, const Operand &VA,
                           float *partialA, int *splitsA, int MaB, int MbB, int HWB, const Operand &UB,
                           const Operand &VB, float *partialB, int *splitsB, hipStream_t st)
{
    int sa, sb;
    if (!wgr_plan(bf16, MaA, MbA, N, HWA, &sa) || !wgr_plan(bf16, MaB, MbB, N, HWB, &sb) || UA.pro != PRO_BNBWD ||
        UB.pro != PRO_BNBWD || VA.pro == PRO_BNBWD || VB.pro != PRO_NONE)
        return hipErrorNotSupported;
    const WgrSide a = {wgr_tiles(MaA, MbA), wgr_chunks(N, HWA), VA.pro == PRO_NONE ? 12 : 16, sa};
    const WgrSide b = {wgr_tiles(MaB, MbB), wgr_chunks(N, HWB), 12, sb};
    wgr_pair_splits(a, b, kWgrResident, splitsA, splitsB);
    *splitsA = std::max(*splitsA, wgr_least(bf16, MaA, MbA, N, HWA));
    *splitsB = std::max(*splitsB, wgr_least(bf16, MaB, MbB, N, HWB));
    return wgr_go(bf16, VA.pro != PRO_NONE, wgr_args(N, MaA, MbA, HWA, UA, VA, partialA, *splitsA),
                  wgr_args(N, MaB, MbB, HWB, UB, VB, partialB, *splitsB), st);
}

} // namespace mbk
