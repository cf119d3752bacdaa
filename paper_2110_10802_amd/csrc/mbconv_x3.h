// fp32 contractions on the bf16 matrix cores: the three-plane operand split and its MFMA, and the
// weight images; shared by kernels_x3.hip (which derives them), kernels_xk.hip and kernels_misc.hip.
#pragma once
#include "mbconv_dev.h"
#include "mbconv_launch.h"

namespace mbk {

typedef float float16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct X3Operand {
    const float *p0, *p1;
    const float *c0, *c1, *c2, *gate;
};

// (x0, x1) -> three words, each the bf16 pair (plane value of x0 in bits 0-15, of x1 in 16-31)
__device__ __forceinline__ void x3_split2(float x0, float x1, uint32_t (&w)[3])
{
    w[0] = bf16_pack2(x0, x1);
    float r0 = x0 - __uint_as_float(w[0] << 16), r1 = x1 - __uint_as_float(w[0] & 0xffff0000u);
    w[1] = bf16_pack2(r0, r1);
    r0 -= __uint_as_float(w[1] << 16);
    r1 -= __uint_as_float(w[1] & 0xffff0000u);
    w[2] = bf16_pack2(r0, r1);
}
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

template <int PRO>
__device__ __forceinline__ float x3_apply(float v0, float v1, float k0, float k1, float k2)
{
    if (PRO == PRO_NONE)
        return v0;
    if (PRO == PRO_BNSWISH_GATE)
        return actf(fmaf(v0, k0, k1)) * k2;
    return fmaf(k0, v0, fmaf(k1, v1, k2));
}

__device__ __forceinline__ bf16x8 x3_lds8(const uint16_t *p)
{
    return *reinterpret_cast<const bf16x8 *>(p);
}

__device__ __forceinline__ f32x4 x3_mfma6_16(const bf16x8 (&a)[3], const bf16x8 (&b)[3], f32x4 acc)
{
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[2], b[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[2], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[1], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[1], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[0], acc, 0, 0, 0);
    return acc;
}

// eight values -> the three planes of an MFMA operand (value t in halfword t); p keeps the
// packed pairs (values 2t and 2t+1 of plane pl in p[t][pl])
__device__ __forceinline__ void x3_split8(const float (&v)[8], uint32_t (&p)[4][3], bf16x8 (&o)[3])
{
#pragma unroll
    for (int t = 0; t < 4; ++t)
        x3_split2(v[2 * t], v[2 * t + 1], p[t]);
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) {
        const u32x4 q = {p[0][pl], p[1][pl], p[2][pl], p[3][pl]};
        o[pl] = __builtin_bit_cast(bf16x8, q);
    }
}

// One tile (64 rows x 32 k) of a weight image, by 256 threads: thread -> (row tid/4, eight k at
// 8*(tid%4)).  The layout: kernels_x3.hip.
__device__ __forceinline__ void x3_prep_tile(const X3PrepArgs &a, int tile, int tid)
{
    int si = 0;
#pragma unroll
    for (int i = 1; i < 4; ++i)
        if (i < a.nsets && tile >= a.s[i].firstTile)
            si = i;
    const X3PrepSet S = a.s[si];
    const int local = tile - S.firstTile, mt = local / S.CH, ch = local % S.CH;
    const int r = tid >> 2, g = tid & 3;
    const int m = mt * 64 + r, k0 = ch * 32 + 8 * g;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = k0 + j;
        const size_t at = (size_t)m * S.sm + (size_t)k * S.sk;
        v[j] = (m < S.M && k < S.K) ? (a.bf16 ? ld<bf16_t>((const bf16_t *)S.w, at) : ((const float *)S.w)[at])
                                    : 0.f;
    }
    const int lane = (r & 15) + 16 * g;
    if (a.bf16) { // (uniform) the values are bf16 already: packing them rounds nothing
        *reinterpret_cast<uint4 *>(S.img + ((size_t)mt * S.CH + ch) * 2048 + ((r >> 4) * 64 + lane) * 8) =
            make_uint4(bf16_pack2(v[0], v[1]), bf16_pack2(v[2], v[3]), bf16_pack2(v[4], v[5]),
                       bf16_pack2(v[6], v[7]));
        return;
    }
    uint32_t w[4][3];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        x3_split2(v[2 * j], v[2 * j + 1], w[j]);
    uint16_t *dst = S.img + ((size_t)mt * S.CH + ch) * 3 * 2048 + ((r >> 4) * 3 * 64 + lane) * 8;
#pragma unroll
    for (int pl = 0; pl < 3; ++pl)
        *reinterpret_cast<uint4 *>(dst + pl * 512) = make_uint4(w[0][pl], w[1][pl], w[2][pl], w[3][pl]);
}

} // namespace mbk
