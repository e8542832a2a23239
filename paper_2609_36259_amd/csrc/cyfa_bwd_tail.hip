// The last two kernels of either backward: reverse cumulative sums and dR.
#include "cyfa_bwd.h"
#include "cyfa_mfma_common.h"   // wave-level prefix sums (DPP)

namespace cyfa {

namespace {

constexpr int kNT = 512;            // threads per workgroup (two waves per SIMD)
constexpr int kLD = kStoreRows + 4; // padded row of the dM tile (16-byte rows)
constexpr int kCombBlocks = kBwdFinParts;

__device__ __forceinline__ int bwd_tokens(const BwdParams &p, int b) {
    if (p.cu) return min(max(p.cu[b + 1] - p.cu[b], 0), p.T);
    return p.lens ? min(max(p.lens[b], 0), p.T) : p.T;
}
// first row of sequence b in the [rows, H, ...] tensors
__device__ __forceinline__ size_t brow0(const BwdParams &p, int b) {
    return p.cu ? (size_t)p.cu[b] : (size_t)b * p.T;
}

// ---------------------------------------------------------------------------
// (5) reverse cumulative sums per sequence: dlog_alpha_t = sum_{tau >= t} dG_tau
// (with the final-state term at the last token), ddelta_t = sum_{tau >= t}
// dlambda_tau, dclock0 = sum_t dlambda_t, all in double.  Workgroup (b h, piece)
// handles one of kScanPieces consecutive pieces of the sequence: it sums the tokens
// after its piece itself (loads batched eight per thread), and within the piece each
// thread sums its own run of tokens; the sum of the later runs is the piece total
// minus an inclusive prefix over the threads (wave prefix sums, then one offset per
// wave).  The thread that ends at token 0 holds the whole sum, dclock0.
constexpr int kScanPieces = 8;
__global__ __launch_bounds__(kNT) void bwd_scan_kernel(BwdParams p) {
    constexpr int kW = kNT / 64;
    __shared__ double sG[kW], sL[kW];
    const int bh = blockIdx.x, pc = blockIdx.y, b = bh / p.H, h = bh % p.H, tid = threadIdx.x, lane = tid & 63,
              wv = tid >> 6;
    const int Tb = bwd_tokens(p, b);
    const float *dG = p.dG + (size_t)bh * p.Tpad;
    const float *dl = p.dlam + (size_t)bh * p.Tpad;
    double fin = 0.0;
    for (int u = 0; u < kCombBlocks; ++u) fin += p.fin[(size_t)bh * kCombBlocks + u];
    const int pp = (Tb + kScanPieces - 1) / kScanPieces;
    const int P0 = min(pc * pp, Tb), P1 = min(P0 + pp, Tb);
    // tokens after the piece
    double lG = 0.0, lL = 0.0;
    for (int t0 = P1; t0 < Tb; t0 += 8 * kNT) {
        float vg[8], vl[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int t = t0 + u * kNT + tid;
            vg[u] = t < Tb ? dG[t] : 0.f;
            vl[u] = t < Tb ? dl[t] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            lG += vg[u];
            lL += vl[u];
        }
    }
    if (P1 < Tb && tid == 0) lG += fin;
    for (int o = 32; o > 0; o >>= 1) {
        lG += __shfl_xor(lG, o);
        lL += __shfl_xor(lL, o);
    }
    if (lane == 0) {
        sG[wv] = lG;
        sL[wv] = lL;
    }
    __syncthreads();
    double LG = 0.0, LL = 0.0;
#pragma unroll
    for (int u = 0; u < kW; ++u) {
        LG += sG[u];
        LL += sL[u];
    }
    __syncthreads();
    const int per = (P1 - P0 + kNT - 1) / kNT;
    const int t_lo = min(P0 + tid * per, P1), t_hi = min(t_lo + per, P1);
    double aG = 0.0, aL = 0.0;
    for (int t = t_lo; t < t_hi; ++t) {
        aG += (double)dG[t] + (t == Tb - 1 ? fin : 0.0);
        aL += dl[t];
    }
    const double iG = mfma::wave_incl_scan(aG), iL = mfma::wave_incl_scan(aL);
    if (lane == 63) {
        sG[wv] = iG;
        sL[wv] = iL;
    }
    __syncthreads();
    double oG = 0.0, oL = 0.0, TG = 0.0, TL = 0.0;
#pragma unroll
    for (int u = 0; u < kW; ++u) {
        if (u < wv) {
            oG += sG[u];
            oL += sL[u];
        }
        TG += sG[u];
        TL += sL[u];
    }
    double rg = LG + (TG - (oG + iG)), rl = LL + (TL - (oL + iL));   // sums over the later tokens
    for (int t = t_hi - 1; t >= t_lo; --t) {
        rg += (double)dG[t] + (t == Tb - 1 ? fin : 0.0);
        rl += dl[t];
        const size_t si = (brow0(p, b) + t) * p.H + h;
        if (p.glog_alpha) p.glog_alpha[si] = (float)rg;
        p.gdelta[si] = (float)rl;
    }
    if (pc == 0 && tid == 0 && p.gclock0) p.gclock0[bh] = rl;       // t_lo = 0: every token
    for (int t = Tb + pc * kNT + tid; t < p.T; t += kScanPieces * kNT) {
        const size_t si = (brow0(p, b) + t) * p.H + h;
        if (p.glog_alpha) p.glog_alpha[si] = 0.f;
        p.gdelta[si] = 0.f;
    }
}

// ---------------------------------------------------------------------------
// (6) dR_h = (sum over sequences b and chunk groups of dM) Phi^T on the active
// m x m block (M = R Phi, Phi the real Fourier basis of App. A.1).  Workgroup
// (h, row block) handles kDRRows rows of dR, which need the same rows of dM only.
constexpr int kDRRows = 4;          // one element per thread (8: 16 us against 9 at H = 4, its chain of loads twice as long)
__global__ __launch_bounds__(kNT) void bwd_dR_kernel(BwdParams p, int nb) {
    __shared__ float dM[kDRRows][kLD];
    __shared__ float tab[2][kStoreRows];
    const int h = blockIdx.x, i0 = blockIdx.y * kDRRows, tid = threadIdx.x, m = p.m;
    for (int e = tid; e < kDRRows * kStoreRows; e += kNT) {
        const int ii = e >> 7, j = e & 127;
        float s[8] = {};                            // eight running sums, then a tree
        for (int u0 = 0; u0 < nb; u0 += 8) {
            float v[8];                             // eight loads in flight
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int u = u0 + k, b = u / p.groups, g = u % p.groups;
                v[k] = u < nb ? p.dMp[(((size_t)(b * p.H + h) * p.groups + g) * kStoreRows + i0 + ii) * kStoreRows + j]
                              : 0.f;
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) s[k] += v[k];
        }
        dM[ii][j] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    }
    if (tid < m) {
        double sn, cs;
        sincospi(2.0 * (double)tid / (double)m, &sn, &cs);
        tab[0][tid] = (float)cs;
        tab[1][tid] = (float)sn;
    }
    __syncthreads();
    const float dc = 1.f / sqrtf((float)m), ac = sqrtf(2.f / (float)m);
    for (int e = tid; e < kDRRows * m; e += kNT) {
        const int ii = e / m, s = e % m;
        if (i0 + ii >= m) continue;
        float acc = dM[ii][0] * dc;
        int n = 0;                                  // l s mod m, advanced by s per step
        for (int l = 1; 2 * l < m; ++l) {
            n += s;
            if (n >= m) n -= m;
            acc = fmaf(dM[ii][2 * l - 1], ac * tab[0][n], acc);
            acc = fmaf(dM[ii][2 * l], ac * tab[1][n], acc);
        }
        p.gR[((size_t)h * m + i0 + ii) * m + s] = acc;
    }
}

}  // namespace

hipError_t launch_bwd_tail(const BwdParams &p, int parts, hipStream_t s) {
    hipLaunchKernelGGL(bwd_scan_kernel, dim3(p.B * p.H, kScanPieces), dim3(kNT), 0, s, p);
    if (p.gR) hipLaunchKernelGGL(bwd_dR_kernel, dim3(p.H, kStoreRows / kDRRows), dim3(kNT), 0, s, p, parts);
    return hipGetLastError();
}

}  // namespace cyfa
