// Host-side launchers of the gfx950 kernels (internal to libmbconv).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace mbk {

// ---- operand of a 1x1 convolution with an elementwise prologue ------------------------
// The tensor is [N,C,HW] in the activation dtype.  What the GEMM consumes is
//   PRO_NONE         p0
//   PRO_BNSWISH_GATE swish(p0*c0[c]+c1[c]) * gate[n,c]       (Swish(BN(.)) times the SE gate)
//   PRO_BNBWD        c0[c]*p0 + c1[c]*p1 + c2[c]             (BN backward: p0 = dy, p1 = raw input)
enum { PRO_NONE = 0, PRO_BNSWISH_GATE = 1, PRO_BNBWD = 2 };
enum { EPI_NONE = 0, EPI_STATS = 1, EPI_RES = 2 };
constexpr int EPI_PARTIAL = 3; // internal: raw partial sums of a split contraction
// out = acc*scale[m] + shift[m] (+ res when res != NULL): a normalisation with fixed statistics
// folded into the epilogue (evaluation mode).  scale/shift travel in the psum/psq arguments of
// the internal launchers, read only.
constexpr int EPI_AFFINE = 4;

struct Operand {
    const void *p0 = nullptr;
    const void *p1 = nullptr;
    const float *c0 = nullptr, *c1 = nullptr, *c2 = nullptr;
    const float *gate = nullptr;
    int pro = PRO_NONE;
};

constexpr int kConvBQ = 128; // pixel columns per workgroup of the 1x1 conv kernel

inline int conv1x1_num_qtiles(int N, int HW) { return (int)(((long long)N * HW + kConvBQ - 1) / kConvBQ); }

// out[n,m,q] = sum_k A(m,k) * op(B)[n,k,q], A(m,k) = w[m*sAm + k*sAk] (dtype).
// epi: EPI_STATS writes partial sums of out and out^2 to psum/psq laid out
// [M][conv1x1_num_partials(...)]; EPI_RES adds res[n,m,q] before the store.
// sc_store (optional) receives the operand after its prologue (STORE policy).
// Long contractions with few output tiles are split over workgroups; `splitk_ws` then needs
// conv1x1_splitk_floats(...) floats (0 when the launch does not split).
// (`pro`, `epi`: the prologue and epilogue the launch will run with, where the caller knows
// them: some kernel families serve a shape only in certain roles; -1: not stated)
int conv1x1_num_partials(bool bf16, int N, int M, int K, int HW, bool stores_operand, int pro = -1,
                         int epi = -1);
// matrix-core instruction family of a launch: 1 fp32 MFMA, 2 bf16 MFMA on bf16 data, 3 bf16 MFMA
// on three-plane splits of fp32 data
int conv1x1_engine(bool bf16, int N, int M, int K, int HW, bool stores_operand, int pro = -1,
                   int epi = -1);
int wgrad1x1_engine(bool bf16, int Ma, int Mb, int N, int HW);
size_t conv1x1_splitk_floats(bool bf16, int N, int M, int K, int HW, bool stores_operand, int pro = -1,
                             int epi = -1);
//
// The convolutions of the wide blocks take their A operand from a weight image (bf16 planes in
// the order the kernels read them, see kernels_x3.hip): where
// conv1x1_uses_weight_image(...) says so, `wimg` must point to the image of this A (M rows, K
// contraction indices), x3_weight_image_bytes(M, K) bytes, written by launch_x3_prep beforehand;
// `w` is then read only for outputs that the image's planes cannot give (infinite operands).
bool conv1x1_uses_weight_image(bool bf16, int N, int M, int K, int HW, bool stores_operand,
                               int pro = -1, int epi = -1);
size_t x3_weight_image_bytes(bool bf16, int M, int K);
// Up to four images: set i is of A(m,k) = w[m*sm + k*sk], M x K (w in the activation dtype).  They are
// written by a launch of their own, or by extra workgroups of a launch that precedes their first
// reader anyway (launch_bn_finalize, launch_pool, launch_dw_fwd in evaluation mode).
struct X3PrepSet {
    const void *w;
    int M, K, sm, sk;
    uint16_t *img;
    int CH, firstTile;
};
struct X3PrepArgs {
    X3PrepSet s[4];
    int nsets, tiles; // tiles: workgroups of 256 threads it takes
    int bf16;         // the weights are stored as bf16: one plane
};
inline void x3_prep_add(X3PrepArgs &a, const void *w, int M, int K, int sm, int sk, void *img)
{
    const int CH = (K + 31) / 32;
    a.s[a.nsets++] = {w, M, K, sm, sk, (uint16_t *)img, CH, a.tiles};
    a.tiles += (M + 63) / 64 * CH;
}
hipError_t launch_x3_prep(const X3PrepArgs &a, hipStream_t st);
hipError_t launch_conv1x1(bool bf16, int N, int M, int K, int HW, const void *w, int sAm, int sAk,
                          const Operand &B, void *out, int epi, const void *res, float *psum,
                          float *psq, void *sc_store, float *splitk_ws, hipStream_t st,
                          const void *wimg = nullptr);

// The same convolution with out = acc*scale[m] + shift[m] (+ res if non-null) as its epilogue.
// Returns hipErrorNotSupported (nothing launched) when the kernel family that serves this
// shape has no such epilogue; the caller then runs the convolution and the affine map as two
// steps.
hipError_t launch_conv1x1_affine(bool bf16, int N, int M, int K, int HW, const void *w, int sAm,
                                 int sAk, const Operand &B, void *out, const void *res,
                                 const float *scale, const float *shift, hipStream_t st,
                                 const void *wimg = nullptr);

// Weight gradient of a 1x1 conv: dW[a,b] = sum_{n,q} op(U)[n,a,q] * op(V)[n,b,q].
// `partial` needs wgrad_splits(...)*Ma*Mb floats.
int wgrad_splits(bool bf16, int Ma, int Mb, int N, int HW);
// With `defer` non-null the second stage (the sum over the splits) is not launched: it is
// described in *defer, and the caller launches it later (launch_reduce_splits2, together with
// another one); `partial` must stay untouched until then.
struct SplitReduce {
    const float *in; // [S][count]
    int S;
    size_t count;    // 0: no reduction
    float *out;      // [count]
};
hipError_t launch_wgrad1x1(bool bf16, int N, int Ma, int Mb, int HW, const Operand &U,
                           const Operand &V, float *partial, float *dW, SplitReduce *defer,
                           hipStream_t st);
hipError_t launch_reduce_splits2(const SplitReduce &a, const SplitReduce &b, hipStream_t st);
// Two independent weight gradients (A, B) in one launch, for the shapes wgrad1x1_pair_supported
// names; their second stages come back in *ra and *rb.  hipErrorNotSupported: nothing launched.
bool wgrad1x1_pair_supported(bool bf16, int N, int MaA, int MbA, int HWA, int MaB, int MbB, int HWB);
hipError_t launch_wgrad1x1_pair(bool bf16, int N, int MaA, int MbA, int HWA, const Operand &UA,
                                const Operand &VA, float *partialA, float *dWA, SplitReduce *ra,
                                int MaB, int MbB, int HWB, const Operand &UB, const Operand &VB,
                                float *partialB, float *dWB, SplitReduce *rb, hipStream_t st);

// Both gradients of a 1x1 convolution from Cn (narrow) to Cw (wide) channels in one pass over
// de, the gradient at its output (PRO_BNBWD operand, [N,Cw,HW]):
//   dx[n,j,q] = sum_c w[c*Cn+j] * de[n,c,q] (+ res[n,j,q]),   dW[c][j] = sum_{n,q} de[n,c,q] * x[n,j,q]
// bwd1x1_fused_plan tells whether the shape is covered (Cn <= 32, Cn < Cw <= 256, HW % 4 == 0) and
// how many splits of dW land in `partial` ([splits][Cw*Cn] floats, the count wgrad_splits gives);
// the caller sums them (launch_reduce_splits2).
// The mirror image for a convolution from Cw (wide) to Cn (narrow) channels, whose input sc is a
// PRO_BNSWISH_GATE or PRO_NONE operand [N,Cw,HW] and whose output gradient dp is PRO_BNBWD [N,Cn,HW]:
//   G[n,c,q] = sum_j w[j*Cw+c] * dp[n,j,q],   dW[j][c] = sum_{n,q} dp[n,j,q] * sc[n,c,q]
// `fin` (optional): dp's BN-backward coefficients are not read from dp.c0/c1/c2 but derived in
// the kernel from the per-plane partial sums, as launch_bn_bwd_finalize would (psb/psr: [Cn][NP],
// inv_m: one over the elements per channel); workgroup 0 also stores dgamma, dbeta and the coefficient triple.
struct BnBwdFin {
    const float *psb, *psr, *gamma, *bn;
    float *dgamma, *dbeta, *coef;
    int NP;
    double inv_m;
};
bool projbwd_fused_plan(int N, int Cw, int Cn, int HW, int *splits);
hipError_t launch_projbwd_fused(bool bf16, int N, int Cw, int Cn, int HW, const Operand &dp,
                                const Operand &sc, const void *w, void *G, float *partial,
                                int *splits_out, const BnBwdFin *fin, hipStream_t st);
bool bwd1x1_fused_plan(int N, int Cw, int Cn, int HW, int *splits);
// 0: not fused; else the mbconv_engine value of the kernel launch_bwd1x1_fused picks
int bwd1x1_fused_engine(bool bf16, int N, int Cw, int Cn, int HW);
hipError_t launch_bwd1x1_fused(bool bf16, int N, int Cw, int Cn, int HW, const Operand &de,
                               const void *xin, const void *w, void *dx, const void *res,
                               float *partial, int *splits_out, hipStream_t st);

// ---- batch-norm statistics ---------------------------------------------------------------
// Training-mode statistics that the consuming kernel finalises itself (no launch for the finalise
// step): the partial sums of the producer, and what the finalise step needs besides.
struct BnFin {
    const float *psum, *psq;   // [C][NP] partial sums and sums of squares
    const float *gamma, *beta; // [C]
    float *run_mean, *run_var; // [C] running statistics to update, or null
    float *bn_out;             // {scale, shift, mean, rstd}[C], written once per channel
    int NP;
    float eps, momentum;
    double inv_m;              // 1 / elements per channel
    double unbias;             // m/(m-1) (1 when m == 1): biased -> unbiased variance
};
inline BnFin make_bn_fin(const float *psum, const float *psq, const float *gamma, const float *beta,
                         float *run_mean, float *run_var, float *bn_out, int NP, float eps,
                         float momentum, double m)
{
    return {psum, psq, gamma, beta, run_mean, run_var, bn_out, NP, eps, momentum,
            1.0 / m, m > 1.0 ? m / (m - 1.0) : 1.0};
}

// psum/psq: [C][NP] partial sums.  Writes bn = {scale[C], shift[C], mean[C], rstd[C]} and
// updates running statistics (if non-null) with momentum.  If ones is non-null the same launch
// also sets ones[0..ones_count) to 1; if prep is non-null it also writes those weight images.
hipError_t launch_bn_finalize(int C, int NP, double m, const float *psum, const float *psq,
                              const float *gamma, const float *beta, float eps, float momentum,
                              float *run_mean, float *run_var, float *bn, hipStream_t st,
                              float *ones = nullptr, size_t ones_count = 0,
                              const X3PrepArgs *prep = nullptr);

// Evaluation mode: a normalisation with its running statistics.
struct BnEval {
    int C; // 0: the block has none
    const float *gamma, *beta, *run_mean, *run_var;
    float *bn; // {scale, shift, mean, rstd}[C], for consumers that read the block
};
// What the depthwise launch of an evaluation-mode forward does besides the convolution: the kernel takes
// BN1's and BN2's coefficients from the running statistics and, where z is non-null, writes the SE stage's
// squeeze (the mean of each plane after BN2 and activation), and workgroups past the convolution's write
// what later kernels read: the blocks of BN2 and BN3 (and BN1's), the gate of ones of a block without SE, and
// weight images.  The launches these would be (coefficients, pool) are a few microseconds each, which is what a
// forward of one image consists of.
struct DwEval {
    static constexpr bool kEval = true;
    BnEval bn1, bn2, bn3;
    float eps;
    float *z;
    float inv_hw;
    float *ones;
    size_t ones_count;
    X3PrepArgs prep;
    int main, coef; // workgroups of the convolution and of the coefficients (the launcher's)
};
struct DwTrain { // training mode: no such work
    static constexpr bool kEval = false;
};

// Block without a squeeze-and-excitation stage (gate = 1, dz = 0): BN2's backward from the
// plane sums A1 = sum G*act'(y2), A2 = sum G*act'(y2)*dhat, both [N][C]:
//   dbeta = sum_n A1, dgamma = sum_n A2, coef as in launch_bn_bwd_finalize; dzs[N*C] is zeroed.
hipError_t launch_bn2_bwd_nose(int N, int C, double m, const float *A1, const float *A2,
                               const float *gamma, const float *bn, float *dgamma, float *dbeta,
                               float *coef, float *dzs, hipStream_t st);

// BN backward finalise from partial sums [C][NP] of dy (psb) and dy*xhat (psr):
//   dbeta = sum psb, dgamma = sum psr, and coef = {c0,c1,c2}[C] such that
//   dx = c0*dy + c1*raw + c2  equals  gamma*rstd*(dy - dbeta/m - xhat*dgamma/m).
hipError_t launch_bn_bwd_finalize(int C, int NP, double m, const float *psb, const float *psr,
                                  const float *gamma, const float *bn, float *dgamma,
                                  float *dbeta, float *coef, hipStream_t st);

// ---- depthwise chain ---------------------------------------------------------------------
struct DwShape {
    int N, C, H, W, Ho, Wo, k, s, p;
};
// Partial results per channel that launch_dw_fwd / launch_dw_bwd write (psum, psq, pdw, psb,
// psr are laid out [C][dw_num_partials]; forward and backward each with their own): one per image, or
// one per image range for the kernels that keep their accumulators across images.  `stores_a1`: the
// STORE policy is on.
int dw_num_partials(bool bf16, const DwShape &s, bool stores_a1, bool bwd);
size_t dw_fwd_lds_bytes(const DwShape &s);
size_t dw_bwd_lds_bytes(const DwShape &s);

// d = depthwise(swish(e*scale1+shift1)) (or depthwise(e) when bn1 == nullptr), plus per-plane
// partial sums of d and d^2 laid out [C][N].  a1_store (optional) receives swish(bn1(e)).
// With `fin` non-null (only when dw_fwd_finalizes_bn1 says so) the kernel derives bn1 from fin's
// partial sums and writes it to fin->bn_out; psum/psq must not overlap fin's partials.
// With `ev` non-null (evaluation mode) there are no partial sums, and of bn1 only whether it is null counts.
bool dw_fwd_finalizes_bn1(const DwShape &s, bool stores_a1);
// dw_eval_folds: whether evaluation mode should use `ev`.  Elsewhere launch_dw_eval_coef writes what the extra
// workgroups would, ahead of everything else (`coef_ahead`: a launch is due there anyway, for an image that the
// expansion conv reads), and the depthwise launch is that of training mode, its partial sums unread.
bool dw_eval_folds(bool bf16, const DwShape &s, bool se, bool coef_ahead);
hipError_t launch_dw_eval_coef(DwEval &ev, hipStream_t st);
hipError_t launch_dw_fwd(bool bf16, const DwShape &s, const void *e, const float *bn1,
                         const void *w_dw, void *d, float *psum, float *psq, void *a1_store,
                         const BnFin *fin, const DwEval *ev, hipStream_t st);

// Evaluation mode, fp32: the expansion conv, BN1, activation and the depthwise conv in one launch, e staying on the
// chip (kernels_evx.hip).  eval_expand_dw_plan: whether the shape is taken, and in how many strips of rows a plane is;
// the squeeze then comes as that many partial means, z[strip][n][c] (z null: none), or, where `q` is given, multiplied
// with W1 already, as eval_expand_dw_qparts partial sums q[n][part][Cse] (0: not available).  `act`: d is stored after BN2
// and the activation.
bool eval_expand_dw_plan(const DwShape &s, int K, int *strips);
int eval_expand_dw_qparts(const DwShape &s, int K, int Cse);
hipError_t launch_eval_expand_dw(const DwShape &s, int K, const void *x, const void *w_expand, const void *w_dw, void *d,
                                 float *z, float *q, int Cse, const float *w1, bool act, const DwEval &ev, hipStream_t st);

// Evaluation mode, fp32, a block without SE stage and with an expansion: all of it in one launch (ev: the normalisations).
bool eval_block_plan(const DwShape &s, int K, int M);
hipError_t launch_eval_block(const DwShape &s, int K, int M, const void *x, const void *w_expand, const void *w_dw,
                             const void *w_proj, const void *res, void *out, const DwEval &ev, hipStream_t st);

// Evaluation mode, fp32, small launches: out = BN3(W_p (act(BN2(d)) * gate)) (+ res) in one launch, the gate from
// the `parts` partial sums q of launch_eval_expand_dw, or (parts == 0) read from `gate`, or (that null) one.
// `act`: whether d is still to go through BN2 and the activation.
bool eval_proj_plan(int N, int M, int K, int HW, int Cse, bool act);
hipError_t launch_eval_proj(int N, int M, int K, int HW, int Cse, const void *w, const void *d, const float *bn2,
                            const float *bn3, const float *q, int parts, const float *b1, const float *w2,
                            const float *b2, const float *gate, bool act, const void *res, void *out, hipStream_t st);

// Per plane of d: z = mean swish(y2), s3 = sum swish'(y2), s4 = sum swish'(y2)*dhat.
// With `fin` non-null (only when plane_channel_form says so) the kernel derives bn2 from fin's partial
// sums and writes it to fin->bn_out, and writes the weight images of `prep` (may be null).
bool plane_channel_form(int N, int C, int HW);
hipError_t launch_pool(bool bf16, int N, int C, int HW, const void *d, const float *bn2, float *z,
                       float *s3, float *s4, const BnFin *fin, const X3PrepArgs *prep, hipStream_t st);

// SE excite: q = W1 z + b1, g = sigmoid(W2 swish(q) + b2); z is the sum of `nz` arrays [n][c], one behind the other.
hipError_t launch_se_fwd(int N, int C, int Cse, const float *z, int nz, const float *w1, const float *b1,
                         const float *w2, const float *b2, float *q, float *g, hipStream_t st);

// out = p*scale3+shift3 (+ x).
// With `fin` non-null (only where bn_apply_finalizes says so) the kernel derives bn3 from fin's partial
// sums and writes it to fin->bn_out.
bool bn_apply_finalizes(int N, int C, int HW);
hipError_t launch_bn_apply(bool bf16, int N, int C, int HW, const void *p, const float *bn3,
                           const void *res, void *out, const BnFin *fin, hipStream_t st);

// Per plane: sums of dy and dy*xhat with xhat = (raw-mean)*rstd, laid out [C][N].
hipError_t launch_plane_dot(bool bf16, int N, int C, int HW, const void *dy, const void *raw,
                            const float *bn, float *psb, float *psr, hipStream_t st);

// launch_plane_dot and launch_bn_bwd_finalize (f.coef, f.dgamma, f.dbeta) in one launch; f's partial sums
// are not used.
bool bn_bwd_chan_supported(int N, int HW);
hipError_t launch_bn_bwd_chan(bool bf16, int N, int C, int HW, const void *dy, const void *raw, const float *bn,
                              const BnBwdFin &f, hipStream_t st);

// Per plane of (G, d): dg = sum G*a2, A1 = sum G*swish'(y2), A2 = sum G*swish'(y2)*dhat.
hipError_t launch_gate_sums(bool bf16, int N, int C, int HW, const void *G, const void *d,
                            const float *bn2, float *dg, float *A1, float *A2, hipStream_t st);

// SE backward.  Step 1 (one workgroup per image): dt, dq, dzs = dz/HW.
// Step 2: the four FC gradients, and BN2's dgamma/dbeta/coef from the plane sums.
struct SeBwdArgs {
    int N, C, Cse, HW;
    const float *z, *g, *q, *w1, *w2;
    const float *dg, *A1, *A2, *s3, *s4;
    const float *gamma2, *bn2;
    double inv_m; // 1/(N*HW)
    float *dt, *dq, *dzs;
    float *dw1, *db1, *dw2, *db2, *dgamma2, *dbeta2, *coef2;
};
hipError_t launch_se_bwd(const SeBwdArgs &a, hipStream_t st);

// The fused depthwise backward (per plane):
//   dy2 = (G*g + dzs)*swish'(y2);  dd = c0*dy2 + c1*d + c2  (BN2 backward)
//   dw partial[c][n][k*k] = sum dd * a1(shifted);  da1 = depthwise-transpose(dd)
//   with expansion: dy1 = da1*swish'(y1) -> dy1_out, partial sums of dy1 and dy1*e -> [C][N]
//   without:        dx = da1 (+ dout)            -> dx_out
struct DwBwdArgs {
    DwShape s;
    const void *G, *d, *e; // e is x when there is no expansion
    const float *g, *dzs, *bn2, *coef2, *bn1; // bn1 == nullptr: no expansion
    const void *w_dw;
    const void *a1_saved; // optional (STORE policy): swish(bn1(e)) saved by forward
    void *dy1_out;        // or dx when there is no expansion
    const void *res;      // residual dout (no-expansion case only)
    float *pdw, *psb, *psr;
};
hipError_t launch_dw_bwd(bool bf16, const DwBwdArgs &a, hipStream_t st);

// out[i] = sum_{s<S} in[s*count+i]  /  out[c*inner+i] = sum_{n<N} in[(c*N+n)*inner+i]
hipError_t launch_reduce_splits(const float *in, int S, size_t count, float *out, hipStream_t st);
hipError_t launch_reduce_planes(const float *in, int C, int N, int inner, float *out,
                                hipStream_t st);
// launch_reduce_planes(pdw, C, NP, inner, dw) and launch_bn_bwd_finalize(C, NP, m, psb, ...)
// in one launch (both consume the partial results of the fused depthwise backward).
hipError_t launch_dw_bwd_finalize(const float *pdw, int C, int NP, int inner, float *dw, double m,
                                  const float *psb, const float *psr, const float *gamma,
                                  const float *bn, float *dgamma, float *dbeta, float *coef,
                                  hipStream_t st);

} // namespace mbk
