// Evaluation mode in the depthwise kernels (device side; DwEval in mbconv_launch.h).
#pragma once
#include <algorithm>
#include "mbconv_x3.h"

namespace mbk {

// The coefficients of a normalisation with fixed statistics, an affine map per channel (section
// "Background and Related Work", paragraph "Training vs. inference compilation": BN behaves differently
// in inference).  Two phases, as in mbconv_bnfin.h: the loads are requested ahead of the caller's own.
struct BnEvalRegs {
    float gm, bt, rm, rv;
};
__device__ __forceinline__ BnEvalRegs bn_eval_issue(const BnEval &b, int c)
{
    return {b.gamma[c], b.beta[c], b.run_mean[c], b.run_var[c]};
}
struct BnEvalCoef {
    float scale, shift, mean, rstd;
};
__device__ __forceinline__ BnEvalCoef bn_eval_coef(const BnEvalRegs &r, float eps)
{
    // 1/sqrt: the hardware estimate and one Newton step, in fp64 (as mbconv_bnfin.h)
    const double xv = (double)r.rv + (double)eps;
    double rstd = __builtin_amdgcn_rsq(xv);
    if (xv > 0.0 && xv < __builtin_inf())
        rstd = rstd * (1.5 - 0.5 * xv * rstd * rstd);
    const double scale = (double)r.gm * rstd;
    return {(float)scale, (float)((double)r.bt - (double)r.rm * scale), r.rm, (float)rstd};
}

// Workgroup `block` of those past the convolution's, `threads` threads.
__device__ __forceinline__ void dw_eval_extra(const DwEval &ev, int block, int threads)
{
    const int tid = threadIdx.x;
    if (block >= ev.coef) {
        // (uniform over the wavefront, which the compiler has to be told: the set's description then comes by scalar loads)
        const int tile = (block - ev.coef) * (threads / 256) + __builtin_amdgcn_readfirstlane(tid / 256);
        if (tile < ev.prep.tiles)
            x3_prep_tile(ev.prep, tile, tid & 255);
        return;
    }
    const int step = ev.coef * threads;
    for (size_t j = (size_t)block * threads + tid; j < ev.ones_count; j += step)
        ev.ones[j] = 1.0f;
    const auto one = [&](const BnEval &b, int c) __attribute__((always_inline)) {
        const BnEvalCoef k = bn_eval_coef(bn_eval_issue(b, c), ev.eps);
        b.bn[c] = k.scale;
        b.bn[b.C + c] = k.shift;
        b.bn[2 * b.C + c] = k.mean;
        b.bn[3 * b.C + c] = k.rstd;
    };
    const int C1 = ev.bn1.C, C2 = C1 + ev.bn2.C, C3 = C2 + ev.bn3.C;
    for (int i = block * threads + tid; i < C3; i += step) {
        if (i < C1)
            one(ev.bn1, i);
        else if (i < C2)
            one(ev.bn2, i - C1);
        else
            one(ev.bn3, i - C2);
    }
}

// Workgroups of `threads` threads that dw_eval_extra takes
inline unsigned dw_eval_blocks(DwEval &ev, int threads)
{
    // (the coefficients need a thread each; the ones, where there are any, eight to a thread)
    const size_t want = std::max((size_t)(ev.bn1.C + ev.bn2.C + ev.bn3.C), (ev.ones_count + 7) / 8);
    ev.coef = (int)std::min<size_t>((want + threads - 1) / threads, 1024);
    const int per = threads / 256;
    return (unsigned)(ev.coef + (ev.prep.tiles + per - 1) / per);
}

// Workgroups to append to a grid of `main` ones of `threads` threads.
inline unsigned dw_eval_extra_blocks(DwTrain &, unsigned, int) { return 0; }
inline unsigned dw_eval_extra_blocks(DwEval &ev, unsigned main, int threads)
{
    ev.main = (int)main;
    return dw_eval_blocks(ev, threads);
}

} // namespace mbk
