// bf16 storage, 1x1 convolutions with a short contraction and many rows (the expansion conv, K = Cin, and the projection
// conv's data gradient, K = Cout, of the wide blocks): weights resident in LDS, a wavefront per pixel chunk.
//
//   out[n][m][q] = sum_k W[m][k] * op(B)[n][k][q],  operands rounded to bf16 once after the fp32 prologue, fp32 sums
//
// With tiles of 64 pixels by 64 or 128 rows (kernels_bf.hip) every tile stages its own activations through LDS, with a
// barrier for every 32 values of k and an epilogue through LDS, and with four to six of them that is its life: 672 <- 112
// channels on 128 planes of 14x14 take 27 us and the data gradient 35, for 39 and 45 MB.  Here, as in conv_xw for fp32,
//   - a workgroup owns 64 rows whose weights, all of K, lie in LDS (4 KB per 32 values of k) in lane order, one
//     conflict-free 16-byte read per lane and operand;
//   - a wavefront owns whole chunks of 64 pixels: lane (r, g) loads, for every 32 values of k, the values k = 8g .. 8g+7
//     of its four pixels 4r .. 4r+3 (eight-byte loads, sixteen lanes to a 128-byte line), turns them in registers (one
//     byte permutation per pair of values; with a prologue it is the conversion to bf16 that pairs them) and has the B
//     operands of v_mfma_f32_16x16x32_bf16, pixel 4r + j feeding instruction j: no LDS store and no barrier in the loop;
//   - a step's values of the next chunk, or of the step after the next, are requested as soon as its registers are free,
//     and results leave the same way, eight bytes per lane;
//   - BN1's statistics leave as one fp32 partial for every chunk, 64 pixels, with the additions of conv_bf in its order (kept in
//     fp32 over a wavefront's chunks they take 18.8 us instead of 19.5, and lose bits with every chunk).
// The same two, here: 19.5 and 26.1 us.  What bounds it is a wavefront's chain at the two or three workgroups of a
// compute unit that the registers allow (16 tiles of sums): 2.9 us until the weights lie in LDS, then 2.5 to 3.5 a chunk.
#include "mbconv_x3.h"

#include <algorithm>

namespace mbk {

constexpr uint32_t kBwNowhere = 0x80000000u; // a byte offset past every tensor that the plan lets through

struct BwArgs {
    int M, K, HW;
    uint32_t Q;
    int numChunks;
    FastDiv divHW;
    const bf16_t *w;     // [M][K] (PRO_NONE)
    const uint16_t *img; // weight image (PRO_BNBWD; kernels_x3.hip), CH steps of 32
    int CH;
    const bf16_t *p0, *p1;
    const float *c0, *c1, *c2;
    bf16_t *out;
    float *psum, *psq; // EPI_STATS: [M][numChunks]
    int NT;            // chunk sets
    int slabs, perDie;
};

__device__ __forceinline__ uint32_t bw_lo(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t bw_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

template <int CTRL>
__device__ __forceinline__ float bw_add_dpp(float v)
{
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
// (by value: a choice between two elements of an array is a choice of addresses to the compiler, and the array in memory)
__device__ __forceinline__ float bw_pick(bool second, float a, float b) { return second ? b : a; }

// Sums over the 16 lanes of a row of eight values per lane, two of them to each quad: lane r ends with the total of value
// r % 8.  The additions are those of row16_sum, in its order (so the same bits), but of half as many values after each step
// but the first.
__device__ __forceinline__ float bw_sum8(float (&v)[8], int r)
{
#pragma unroll
    for (int i = 0; i < 8; ++i)
        v[i] = bw_add_dpp<0x124>(bw_add_dpp<0x128>(v[i])); // row_ror:8, row_ror:4
#pragma unroll
    for (int i = 0; i < 4; ++i)
        v[i] = bw_add_dpp<0x4e>(bw_pick(r & 4, v[i], v[i + 4])); // quad_perm: the lane two further on
#pragma unroll
    for (int i = 0; i < 2; ++i)
        v[i] = bw_add_dpp<0xb1>(bw_pick(r & 2, v[i], v[i + 2])); // quad_perm: the neighbour
    return bw_pick(r & 1, v[0], v[1]);
}

// Workgroups of a compute unit that the registers allow
constexpr int bw_waves(int pro, int ks) { return pro == PRO_BNBWD && ks <= 4 ? 3 : 2; }

// KS: steps of 32 of the contraction; RD: steps in flight (a divisor of KS)
template <int KS, int RD, int PRO, int EPI>
__global__ __launch_bounds__(256, bw_waves(PRO, KS)) void conv_bw_kernel(BwArgs a)
{
    static_assert(PRO == PRO_NONE || PRO == PRO_BNBWD, "prologues of the short-contraction roles");
    static_assert(KS % RD == 0, "a step's slot is the same in every chunk");
    constexpr int NP = PRO == PRO_BNBWD ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) uint16_t lds16[]; // [KS][4 row tiles][64 lanes][8]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int M = a.M, K = a.K, HW = a.HW;
    // die = workgroup mod 8: the slabs of a chunk set on one, which then reads the set's pixels from memory once
    const int die = blockIdx.x & 7, bi = blockIdx.x >> 3, whole = (a.NT >> 3) * a.slabs;
    const int rest = die * (a.perDie - whole) + bi - whole;
    const int slab = (bi < whole ? bi : rest) % a.slabs;
    const int cs = bi < whole ? (bi / a.slabs) * 8 + die : (a.NT & ~7) + rest / a.slabs;
    if (cs >= a.NT) // uniform over the workgroup
        return;

    // the slab's weights, requested here and parked below: thread -> (row, eight k) of every step, or, where there is a
    // weight image (the data gradient's columns are not contiguous), the same pieces in its order, zero past the ends
    u32x4 wreg[KS];
    const int sr = 64 * slab + 16 * (tid >> 6) + (tid & 15), sg = (tid >> 4) & 3;
    if (PRO == PRO_BNBWD) {
        const uint16_t *im = a.img + (size_t)slab * a.CH * 2048 + tid * 8;
#pragma unroll
        for (int s = 0; s < KS; ++s)
            wreg[s] = *reinterpret_cast<const u32x4 *>(im + min(s, a.CH - 1) * 2048);
    } else {
        const bf16_t *wr = a.w + (size_t)min(sr, M - 1) * K;
#pragma unroll
        for (int s = 0; s < KS; ++s)
            wreg[s] = *reinterpret_cast<const u32x4 *>(wr + min(32 * s + 8 * sg, K - 8)); // (K % 8 == 0)
    }
    f32x4 *Cl = reinterpret_cast<f32x4 *>(lds16 + KS * 2048); // [32*KS] {c0, c1, c2, -} (PRO_BNBWD), zero past K
    f32x4 cv = {0.f, 0.f, 0.f, 0.f};
    if (PRO == PRO_BNBWD) {
        const int kk = min(tid, K - 1);
        cv = (f32x4){a.c0[kk], a.c1[kk], a.c2[kk], 0.f};
    }
    const uint32_t mrow = (uint32_t)(64 * slab + 4 * g) * (uint32_t)HW; // output row 16i + v above it
    const uint32_t bimg = (uint32_t)K * (uint32_t)HW, oimg = (uint32_t)M * (uint32_t)HW;
    // where the lane's four pixels are (HW % 4 == 0: in one image, and all there or none)
    const auto locate = [&](int c, uint32_t &bo, uint32_t &oo, uint32_t &okm) __attribute__((always_inline)) {
        const uint32_t q = (uint32_t)c * 64u + 4u * (uint32_t)r;
        okm = q < a.Q ? 0xffffffffu : 0u;
        const uint32_t qs = q < a.Q ? q : 0u;
        const uint32_t n = fdiv(qs, a.divHW), pix = qs - n * (uint32_t)HW;
        bo = n * bimg + pix;
        oo = n * oimg + pix;
    };
    // (buffer accesses: a row's distance from the lane's first is a scalar, not an address in registers)
    const auto rs0 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(a.p0), 0, (int)(2u * a.Q * (uint32_t)K), 0x00020000);
    const auto rs1 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(NP == 2 ? a.p1 : a.p0), 0,
                                                       (int)(2u * a.Q * (uint32_t)K), 0x00020000);
    u32x2 raw[RD][NP][8];
    const auto fetch = [&](int s, uint32_t bo) __attribute__((always_inline)) {
        const int o = (int)(2u * (bo + (uint32_t)min(32 * s + 8 * g, K - 8) * (uint32_t)HW));
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int t = 0; t < 8; ++t)
                raw[s % RD][p][t] = __builtin_amdgcn_raw_buffer_load_b64(p == 0 ? rs0 : rs1, o, 2 * t * HW, 0);
    };

    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(a.out, 0, (int)(2u * a.Q * (uint32_t)M), 0x00020000);
    const int cStep = 4 * a.NT;
    int ch = 4 * cs + wv;
    uint32_t bo, oo, okm;
    locate(ch < a.numChunks ? ch : 0, bo, oo, okm);
#pragma unroll
    for (int s = 0; s < RD; ++s)
        fetch(s, bo);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const uint32_t m = PRO == PRO_BNBWD ? (s < a.CH ? 0xffffffffu : 0u)
                                            : (sr < M && 32 * s + 8 * sg < K ? 0xffffffffu : 0u);
        *reinterpret_cast<u32x4 *>(lds16 + s * 2048 + tid * 8) =
            (u32x4){wreg[s][0] & m, wreg[s][1] & m, wreg[s][2] & m, wreg[s][3] & m};
    }
    if (PRO == PRO_BNBWD && tid < 32 * KS) {
        const uint32_t m = tid < K ? 0xffffffffu : 0u;
        Cl[tid] = (f32x4){and_mask(cv[0], m), and_mask(cv[1], m), and_mask(cv[2], m), 0.f};
    }
    __syncthreads(); // the slab, Cl

    // (the lane's row of the statistics: row tile r / 4, row 4g + r % 4 of it)
    const int srow = 64 * slab + 16 * (r >> 2) + 4 * g + (r & 3), snum = EPI == EPI_STATS ? (int)(4u * (uint32_t)a.numChunks * (uint32_t)M) : 0;
    const auto rsum = __builtin_amdgcn_make_buffer_rsrc(a.psum, 0, snum, 0x00020000);
    const auto rsq = __builtin_amdgcn_make_buffer_rsrc(a.psq, 0, snum, 0x00020000);
    const uint32_t sv = srow < M ? 4u * (uint32_t)srow * (uint32_t)a.numChunks : kBwNowhere;
    for (; ch < a.numChunks; ch += cStep) {
        uint32_t nbo, noo, nokm;
        locate(ch + cStep < a.numChunks ? ch + cStep : ch, nbo, noo, nokm);
        f32x4 acc[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            // (values past K, in the last step: zero, as what was loaded there may be infinite)
            const uint32_t m = 32 * s + 8 * g >= K ? 0u : 0xffffffffu;
            const auto mask = [&](uint32_t v) { return s == KS - 1 ? v & m : v; };
            u32x4 b[4];
            const u32x2(&x)[8] = raw[s % RD][0];
            if (PRO == PRO_NONE) {
#pragma unroll
                for (int w = 0; w < 4; ++w)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        b[2 * h][w] = mask(bw_lo(x[2 * w][h], x[2 * w + 1][h]));
                        b[2 * h + 1][w] = mask(bw_hi(x[2 * w][h], x[2 * w + 1][h]));
                    }
            } else {
                const u32x2(&y)[8] = raw[s % RD][NP - 1];
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    float d[2][4];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const f32x4 k = Cl[32 * s + 8 * g + 2 * w + e];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const uint32_t xw = x[2 * w + e][j >> 1], yw = y[2 * w + e][j >> 1];
                            const float xf = __uint_as_float(j & 1 ? xw & 0xffff0000u : xw << 16);
                            const float yf = __uint_as_float(j & 1 ? yw & 0xffff0000u : yw << 16);
                            d[e][j] = fmaf(k[0], xf, fmaf(k[1], yf, k[2]));
                        }
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        b[j][w] = mask(bf16_pack2(d[0][j], d[1][j]));
                }
            }
            if (s + RD < KS)
                fetch(s + RD, bo);
            else
                fetch(s + RD - KS, nbo);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bf16x8 av = x3_lds8(lds16 + s * 2048 + (i * 64 + lane) * 8);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, b[j]), acc[i][j],
                                                                        0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0); // (one step's operands at a time in registers)
        }
        // rows 64 slab + 16i + 4g + v, the lane's four pixels.  Buffer stores, which drop what lies past the tensor's
        // end: behind a branch around a store the next loads' wait would be one for every store before them.
        float s1[2], s2[2], p1[8], p2[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t ov = okm && 64 * slab + 16 * i + 4 * g < M ? 2u * (oo + mrow) : kBwNowhere; // (M % 8 == 0)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const u32x2 o = {bf16_pack2(acc[i][0][v], acc[i][1][v]), bf16_pack2(acc[i][2][v], acc[i][3][v])};
                __builtin_amdgcn_raw_buffer_store_b64(o, rsrc, (int)ov, (int)(2u * (uint32_t)(16 * i + v) * (uint32_t)HW), 0);
                if (EPI == EPI_STATS) { // of the values as stored
                    const uint32_t xl = o[0] & okm, xh = o[1] & okm;
                    const float x0 = __uint_as_float(xl << 16), x1 = __uint_as_float(xl & 0xffff0000u);
                    const float x2 = __uint_as_float(xh << 16), x3 = __uint_as_float(xh & 0xffff0000u);
                    p1[4 * (i & 1) + v] = ((x0 + x1) + x2) + x3;
                    p2[4 * (i & 1) + v] = fmaf(x3, x3, fmaf(x2, x2, fmaf(x1, x1, x0 * x0)));
                }
            }
            if (EPI == EPI_STATS && i & 1) {
                s1[i >> 1] = bw_sum8(p1, r);
                s2[i >> 1] = bw_sum8(p2, r);
            }
        }
        if (EPI == EPI_STATS) { // a partial sum for every 64 pixels, as the tiles leave them: the rest is added in fp64
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, bw_pick(r & 8, s1[0], s1[1])), rsum, (int)sv, 4 * ch, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, bw_pick(r & 8, s2[0], s2[1])), rsq, (int)sv, 4 * ch, 0);
        }
        bo = nbo;
        oo = noo;
        okm = nokm;
    }
}

// `sets`: chunk sets, each a workgroup's for every slab of rows.
bool bw_conv_plan(int N, int M, int K, int HW, int pro, int epi, int *sets)
{
    const long long Q = (long long)N * HW;
    // the shapes that kernels_bf.hip multiplies with bf16 operands, in the roles of a short contraction
    if (K % 8 != 0 || M % 8 != 0 || HW % 4 != 0 || K < 32 || K > 192 || M < 64 || M < K)
        return false;
    if (!(pro == PRO_NONE && epi == EPI_STATS) && !(pro == PRO_BNBWD && epi == EPI_NONE))
        return false;
    if (Q * M >= (1ll << 30) || Q * K >= (1ll << 30)) // byte offsets below 2 GiB in the kernel
        return false;
    const int slabs = (M + 63) / 64;
    const long long groups = ((Q + 63) / 64 + 3) / 4; // of four chunks, one per wavefront
    // Fewer workgroups than this are no faster than the tiles (training step, tiles / here: 64 -> 384 channels on four planes
    // of 16x16, 24 groups of chunks and rows, 68.8 / 70.9 us; evaluation, 72 -> 288 on 38 of 20x20, 300, 30.3 / 30.8; training
    // steps, 112 -> 672 on 14x14, 32 images, 275, 140.4 / 138.3, 512 images 1110 / 1043; 48 -> 288 on 28x28, 64 images 212 / 196).
    if (groups * slabs < (pro == PRO_NONE ? 320 : 128))
        return false;
    // one round of workgroups, with as many chunks to a wavefront as that takes (544 workgroups on 512 places: 22.3 us above)
    const long long wgs = 256 * bw_waves(pro, (K + 31) / 32), rounds = (groups * slabs + wgs - 1) / wgs;
    *sets = (int)((groups + rounds - 1) / rounds);
    return true;
}

hipError_t launch_bw_conv1x1(int N, int M, int K, int HW, const void *w, int sAm, int sAk, const void *wimg, const Operand &B,
                             void *out, int epi, float *psum, float *psq, hipStream_t st)
{
    int nt;
    if (!bw_conv_plan(N, M, K, HW, B.pro, epi, &nt) || (B.pro == PRO_NONE ? sAm != K || sAk != 1 : !wimg))
        return hipErrorInvalidValue;
    BwArgs a;
    a.M = M;
    a.K = K;
    a.HW = HW;
    a.Q = (uint32_t)((long long)N * HW);
    a.numChunks = (int)((a.Q + 63u) / 64u);
    a.divHW = make_div((uint32_t)HW);
    a.w = (const bf16_t *)w;
    a.img = (const uint16_t *)wimg;
    a.CH = (K + 31) / 32;
    a.p0 = (const bf16_t *)B.p0;
    a.p1 = (const bf16_t *)B.p1;
    a.c0 = B.c0;
    a.c1 = B.c1;
    a.c2 = B.c2;
    a.out = (bf16_t *)out;
    a.psum = psum;
    a.psq = psq;
    a.NT = nt;
    a.slabs = (M + 63) / 64;
    a.perDie = (nt >> 3) * a.slabs + ((nt & 7) * a.slabs + 7) / 8;
    const int ks = (K + 31) / 32;
    const dim3 grid((unsigned)(8 * a.perDie));
    const size_t lds = (size_t)ks * (B.pro == PRO_BNBWD ? 4608 : 4096);
#define MBK_CASE(KS_, RD_, PRO_, EPI_)                                                            \
    if (ks == KS_ && B.pro == PRO_) {                                                             \
        hipLaunchKernelGGL((conv_bw_kernel<KS_, RD_, PRO_, EPI_>), grid, dim3(256), lds, st, a);  \
        return hipGetLastError();                                                                 \
    }
    MBK_CASE(1, 1, PRO_NONE, EPI_STATS)
    MBK_CASE(2, 2, PRO_NONE, EPI_STATS)
    MBK_CASE(3, 3, PRO_NONE, EPI_STATS)
    MBK_CASE(4, 4, PRO_NONE, EPI_STATS)
    MBK_CASE(5, 5, PRO_NONE, EPI_STATS)
    MBK_CASE(6, 3, PRO_NONE, EPI_STATS)
    MBK_CASE(1, 1, PRO_BNBWD, EPI_NONE)
    MBK_CASE(2, 2, PRO_BNBWD, EPI_NONE)
    MBK_CASE(3, 1, PRO_BNBWD, EPI_NONE)
    MBK_CASE(4, 2, PRO_BNBWD, EPI_NONE)
    MBK_CASE(5, 1, PRO_BNBWD, EPI_NONE)
    MBK_CASE(6, 2, PRO_BNBWD, EPI_NONE)
#undef MBK_CASE
    return hipErrorInvalidValue;
}

} // namespace mbk
