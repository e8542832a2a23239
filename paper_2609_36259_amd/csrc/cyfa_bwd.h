// Internal declarations of the backward pass (not part of the public ABI).
#pragma once

#include "cyfa_internal.h"

namespace cyfa {

constexpr int kBwdChunk = 16;       // chunk length a caller may name for the fp32 backward
constexpr int kBwdMfmaChunk = 32;   // tokens per chunk of the matrix-core backward kernels
constexpr int kBwdFinParts = 16;    // partial sums of the final-state loss per (b, h)

// Gradients of L = sum_t <do_t, o_t> + <dK_T, Kbar_T> + <dV_T, Vbar_T>.
struct BwdParams {
    int B, T, H, dk, dv, m;
    int nc;                         // chunks per sequence
    int Tpad;                       // nc times the chunk length: rows of the per-token workspace arrays
    int groups, cpg;                // chunk groups per sequence and chunks per group
    float scale;
    int dtype;
    const void *q, *k, *v, *dout;
    const float *delta, *log_alpha, *beta, *R;
    const int *lens;
    const int *cu;                  // packed sequences (the fp32 forward's front kernels only; see FwdParams)
    const float *K0, *V0;
    const double *clock0;
    const float *dK_T, *dV_T;
    void *gq, *gk, *gv;             // dtype of q
    float *gdelta, *glog_alpha, *gbeta, *gR, *gK0, *gV0;
    double *gclock0;
    // workspace
    float *U, *dP;                  // [BH][Tpad] readout output u_t and key-pass adjoint dp_t (fp32 backward)
    float *udu, *dlam, *dG;         // [BH][Tpad] <u_t, du_t>, dL/dlambda_t, dL/dG_t
    float *dMp;                     // [BH][groups][128][128] partial dL/dM
    double *fin;                    // [BH][kBwdFinParts] partial sums of <dK_T, Kbar_T> + <dV_T, Vbar_T>
};

// The last two kernels of either backward: reverse cumulative sums of p.dG and
// p.dlam (plus the final-state loss p.fin at the last token) into dlog_alpha,
// ddelta, dclock0; dR from the partial dM of every (b, h, group) in p.dMp.
hipError_t launch_bwd_tail(const BwdParams &p, int parts, hipStream_t s);
// fp32 backward (d_k, d_v in {64, 128} or both 256; m <= 127): its own chunks of 64 tokens.
size_t bwd_f32_workspace_bytes(int B, int T, int H, int dk, int dv);
hipError_t launch_bwd_f32(BwdParams p, void *ws, hipStream_t s);

// Matrix-core backward (bf16, d_k = d_v = 128, m <= 127, 32-token chunks, p.nc and
// p.Tpad counted in those chunks).
int bwd_mfma_auto_groups(int B, int T, int H);
size_t bwd_mfma_workspace_bytes(int B, int T, int H, int groups);
hipError_t launch_bwd_mfma(BwdParams p, void *ws, hipStream_t s);

}  // namespace cyfa
